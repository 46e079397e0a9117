"""GPU <-> oracle parity of the BalanceKV hot path, through the C ABI (run with -m gpu).

Protocol (one halving): the GPU's signs are fed to the CPU oracle (teacher forcing); a decision may
differ only where |u_j - p_j| < 1e-4 (counted); the survivors must be exactly the output-step
function of the GPU's own signs; copied rows are bit-exact.  Attention outputs are compared with
the oracle's estimator on the GPU's cache within 1e-4 (fp32) / 2e-2 (bf16) relative L2.
"""
import math

import ctypes as C

import numpy as np
import pytest
import torch

from parity_utils import MARGIN, expected_survivors, f32, rel_l2, to_f64, verify_halving

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bk():
    import paper_2502_07861_amd as bkm
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    bkm.lib()          # raises if the HIP library is not built: there is no fallback
    return bkm


@pytest.fixture(scope="module")
def synth():
    from paper_2502_07861_amd import synth as s
    return s


def _blocks(synth, dtype, d, b, n_inst, seed):
    """K, V [n_inst, b, d] on the GPU with the structure of the benchmark workloads."""
    if dtype == torch.float32:
        t = synth.single_head_fp32(n=n_inst * b, d=d, nq=4, seed=seed, device="cpu")
        K, V = t["K"].view(n_inst, b, d), t["V"].view(n_inst, b, d)
    else:
        t = synth.gqa_layer_bf16(n_seq=n_inst, n=b, d=d, g=1, nq=1, seed=seed, device="cpu")
        K, V = t["K"], t["V"]
    return K.cuda().contiguous(), V.cuda().contiguous()


def _log_c_setting(oracle, kind, Kd, b, center):
    from oracle.tuning import tune_log_c
    if kind == "literal":
        return float("nan"), oracle.log_c_literal(b, 1e-6)
    if kind == "one":
        return 0.0, 0.0
    lc = f32(tune_log_c(Kd[: min(4, Kd.shape[0])], target=0.25, center=center))
    return lc, lc


# ------------------------------------------------------------------------------------------ a3/a4: kernel weights
@pytest.mark.parametrize("dtype,d,b,center", [
    (torch.float32, 64, 128, False), (torch.float32, 64, 256, True), (torch.bfloat16, 128, 192, True),
    (torch.bfloat16, 128, 1024, True), (torch.bfloat16, 64, 64, False), (torch.float32, 128, 320, True),
    (torch.float32, 128, 640, True), (torch.float32, 128, 1024, False),      # fp32, d=128: three and four chunks of 256 rows
])
def test_kernel_weights_match_definition(bk, synth, dtype, d, b, center):
    """g_ij = exp((<k_i,k_j> - r_key^2)/sqrt d - ln c) (Alg. 2 lines 2-8, v = 1), centred keys optional."""
    K, _ = _blocks(synth, dtype, d, b, 2, seed=101 + b)
    Kd = to_f64(K)
    Kc = Kd - Kd.mean(axis=1, keepdims=True) if center else Kd
    S = np.einsum("nid,njd->nij", Kc, Kc)
    A = np.max(np.einsum("nii->ni", S), axis=1)
    # choose ln c so that the largest off-diagonal weight is O(1): the comparison is then meaningful
    off = S - 1e30 * np.eye(b)[None]
    log_c = f32(float(np.mean((off.max(axis=(1, 2)) - A) / math.sqrt(d))))
    ref = np.exp((S - A[:, None, None]) / math.sqrt(d) - log_c)
    p = bk.make_params(d, b, 1, dtype, log_c=log_c, center=center)
    G = bk.kernel_weights(p, K).cpu().numpy().astype(np.float64)
    offd = ~np.eye(b, dtype=bool)[None].repeat(2, axis=0)
    assert np.isfinite(G[offd]).all()
    big = offd & (ref > 1e-30)             # below that the hardware exp2 flushes to zero
    assert big.sum() > 16 * b
    np.testing.assert_allclose(G[big], ref[big], rtol=5e-4)
    assert np.abs(G - ref)[offd].max() <= 5e-4 * ref[offd].max()
    diag_ok = np.eye(b, dtype=bool)[None].repeat(2, axis=0) & (ref < 1e30)
    np.testing.assert_allclose(G[diag_ok], ref[diag_ok], rtol=5e-4)
    np.testing.assert_allclose(G[offd], np.swapaxes(G, 1, 2)[offd], rtol=1e-4, atol=1e-30)


# ------------------------------------------------------------------------------------------ a3-a7: one halving
CASES = [
    # dtype, d, b, n_inst, center
    (torch.float32, 64, 256, 4, False),      # workload 1 shape
    (torch.bfloat16, 128, 512, 6, True),     # workload 2 shape
    (torch.bfloat16, 128, 1024, 3, True),    # workloads 3-5 shape: two LDS chunks
    (torch.bfloat16, 64, 128, 5, True),
    (torch.float32, 128, 320, 2, True),      # ragged: 5 panels, second chunk of one panel
    (torch.bfloat16, 128, 64, 9, False),     # a single panel
    (torch.float32, 128, 640, 2, True),      # fp32, d=128: chunks of 256 rows -> three chunks, the last of two panels
    (torch.float32, 128, 1024, 2, True),     # ... four full chunks (the counters are reset three times)
    (torch.bfloat16, 128, 960, 2, False),    # bf16: two chunks, the second of seven panels
    (torch.bfloat16, 128, 576, 2, True),     # ... the second of one panel (one slot brought in during the first pipeline)
    (torch.bfloat16, 128, 768, 2, True),     # ... of four
    (torch.float32, 64, 1024, 2, True),      # fp32 rows of 256 bytes: two full chunks
]


@pytest.mark.parametrize("dtype,d,b,n_inst,center", CASES)
@pytest.mark.parametrize("c_kind", ["literal", "one", "tuned"])
def test_compress_block_teacher_forced(bk, synth, oracle, dtype, d, b, n_inst, center, c_kind):
    K, V = _blocks(synth, dtype, d, b, n_inst, seed=7 + b + d)
    Kd, Vd = to_f64(K), to_f64(V)
    log_c_abi, log_c = _log_c_setting(oracle, c_kind, Kd, b, center)
    seed = 0xABCDEF + b
    p = bk.make_params(d, b, 1, dtype, log_c=log_c_abi, delta=1e-6, seed=seed, center=center)
    u = np.stack([oracle.uniform_fill(seed, t, 0, b) for t in range(n_inst)])
    out = bk.compress_block(p, K, V, w_in=2.0, uniforms=torch.from_numpy(u.astype(np.float32)).cuda())
    torch.cuda.synchronize()
    signs = out["signs"].cpu().numpy()
    assert set(np.unique(signs).tolist()) <= {-1, 1}
    v = verify_halving(oracle, Kd, u, signs, log_c=log_c, center=center)
    print("c=%s: %d decisions, %d within margin, %d margin flips, %d hard" % (c_kind, v["n"], v["near"], v["margin"], v["hard"]))
    assert v["hard"] == 0
    if c_kind == "tuned":          # the comparison is not vacuous: decisions depend on the weights
        assert np.abs(2 * v["res"]["p"] - 1).mean() > 0.1
    # output step: exact integer function of the GPU's own signs
    idx = out["idx"].cpu().numpy()
    np.testing.assert_array_equal(idx, expected_survivors(oracle, signs))
    # gathered rows are copies of the original rows; weights doubled
    gi = torch.from_numpy(idx.astype(np.int64)).cuda()
    assert torch.equal(out["K"], torch.gather(K, 1, gi[..., None].expand(-1, -1, d)))
    assert torch.equal(out["V"], torch.gather(V, 1, gi[..., None].expand(-1, -1, d)))
    assert torch.all(out["w"] == 4.0)
    # status / stats against the oracle's view of the same run
    status = out["status"].cpu().numpy()
    stats = out["stats"].cpu().numpy()
    marg = np.abs(u - v["res"]["p"]).min(axis=1)
    smax = np.abs(v["res"]["sigma"]).max(axis=1)
    np.testing.assert_allclose(stats[:, 0], marg, atol=2e-5)
    np.testing.assert_allclose(stats[:, 1], smax, rtol=1e-3, atol=1e-5)
    fail_gpu = (status & 1).astype(bool)
    fail_or = v["res"]["fails"] > 0
    clear = np.abs(smax - 1.0) > 1e-3
    np.testing.assert_array_equal(fail_gpu[clear], fail_or[clear])
    # free-running oracle: identical survivors unless a margin case occurred first
    free = oracle.softmax_balance_batch(Kd, u=u, log_c=log_c, center=center)
    for t in range(n_inst):
        if not np.array_equal(free["eta"][t], signs[t]):
            first = int(np.argmax(free["eta"][t] != signs[t]))
            assert abs(u[t, first] - free["p"][t, first]) < MARGIN


# panels dealt out as half columns (one to four at a time): single precision, and the value factor with the values in LDS
@pytest.mark.parametrize("dtype,d,b,value", [(torch.float32, d, b, False) for d in (64, 128) for b in (64, 128, 192, 256)] +
                         [(torch.float32, 128, 448, False), (torch.float32, 64, 192, True), (torch.float32, 128, 128, True),
                          (torch.bfloat16, 128, 128, True), (torch.bfloat16, 128, 192, True), (torch.bfloat16, 64, 256, True)])
def test_half_columns(bk, synth, oracle, dtype, d, b, value):
    n_inst = 3
    K, V = _blocks(synth, dtype, d, b, n_inst, seed=11 + b + d)
    Kd, Vd = to_f64(K), to_f64(V)
    _, log_c = _log_c_setting(oracle, "tuned", Kd, b, True)
    seed = 0x5EED + b
    p = bk.make_params(d, b, 1, dtype, log_c=log_c, seed=seed, center=True, value_gram=value)
    out = bk.compress_block(p, K, V)
    u = np.stack([oracle.uniform_fill(seed, t, 0, b) for t in range(n_inst)])
    signs = out["signs"].cpu().numpy()
    chk = oracle.softmax_balance_batch(Kd, Vd if value else None, u=u, log_c=log_c, center=True, forced=signs)
    hard = (chk["dec"] != signs) & (np.abs(u - chk["p"]) >= 1e-4)
    assert not hard.any()
    assert not (out["status"].cpu().numpy() & 2).any()         # BKV_STATUS_INTERNAL: a wait inside the block ran out
    np.testing.assert_array_equal(out["idx"].cpu().numpy(), expected_survivors(oracle, signs))


@pytest.mark.parametrize("dtype,d,b,center,r_key", [
    (torch.bfloat16, 128, 64, True, 0.0), (torch.bfloat16, 128, 256, False, 0.0), (torch.bfloat16, 128, 320, True, 0.0),     # one chunk: 1, 4, 5
    (torch.bfloat16, 128, 512, True, 9.0), (torch.float32, 64, 64, True, 0.0), (torch.float32, 64, 512, False, 9.0),         # ... and 8 panels
    (torch.bfloat16, 128, 576, True, 0.0), (torch.bfloat16, 128, 768, False, 0.0), (torch.bfloat16, 128, 832, True, 0.0),    # second chunk: 1, 4, 5
    (torch.bfloat16, 128, 1024, True, 0.0), (torch.bfloat16, 128, 1024, False, 9.0)])                                        # ... and 8 panels
def test_many_blocks_equal_few_blocks(bk, synth, dtype, d, b, center, r_key):
    """A launch with more blocks than compute units runs two blocks on each (another kernel); the same blocks in launches of
    at most one per compute unit are the reference (they are held against the oracle above).  Both form every sum in the
    same order, so nothing may differ: signs, survivors, rows, status and statistics bit for bit."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n_inst = n_cu + 9
    base_K, base_V = _blocks(synth, dtype, d, b, 8, seed=31 + b)
    perm = torch.randperm(8 * b, generator=torch.Generator().manual_seed(b)).cuda()
    K = torch.cat([base_K.view(-1, d)[(perm + 97 * k) % (8 * b)].view(8, b, d) for k in range((n_inst + 7) // 8)])[:n_inst].contiguous()
    V = torch.cat([base_V] * ((n_inst + 7) // 8))[:n_inst].contiguous()
    from oracle.tuning import tune_log_c
    lc = f32(tune_log_c(to_f64(K[:1]), target=0.25, center=center))
    p = bk.make_params(d, b, 1, dtype, log_c=lc, seed=77, center=center, r_key=r_key)
    ids = (torch.arange(n_inst, dtype=torch.int64) * 5 + 3).cuda()
    many = bk.compress_block(p, K, V, inst_ids=ids)
    torch.cuda.synchronize()
    for lo in range(0, n_inst, n_cu):
        few = bk.compress_block(p, K[lo:lo + n_cu].contiguous(), V[lo:lo + n_cu].contiguous(), inst_ids=ids[lo:lo + n_cu].contiguous())
        torch.cuda.synchronize()
        for name, x in few.items():
            assert torch.equal(many[name][lo:lo + n_cu], x), name
    assert (many["status"] & 2 == 0).all()


@pytest.mark.parametrize("dtype,d,b", [(torch.bfloat16, 128, 64), (torch.bfloat16, 128, 576), (torch.float32, 64, 256)])
def test_weights_that_overflow_decide_alike(bk, dtype, d, b):
    """A given r_key far below the keys' norms lets weights overflow: sums become infinite and then NaN, from which the two kernels
    (more blocks than compute units or fewer) must not decide differently."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    gen = torch.Generator().manual_seed(b)
    K = torch.randn(b, d, generator=gen)
    c = torch.randn(d, generator=gen)
    c *= math.sqrt(120 * math.sqrt(d)) / c.norm()
    for i in (3, 10, 20, 30, 37, 50):                                        # six keys a panel whose weights are e^120 among themselves
        K[i::64] = c * (1 + 1e-4 * i)
    K, V = K.to(dtype).cuda()[None], torch.randn(1, b, d, generator=gen).to(dtype).cuda()
    p = bk.make_params(d, b, 1, dtype, log_c=0.0, seed=5, center=False, r_key=1e-3)
    assert int(torch.isinf(bk.kernel_weights(p, K)).sum()) >= 36 * (b // 64)
    got = []
    for n in (2, n_cu + 9):
        out = bk.compress_block(p, K.repeat(n, 1, 1), V.repeat(n, 1, 1), inst_ids=torch.full((n,), 7, dtype=torch.int64, device="cuda"))
        assert (out["signs"] == out["signs"][:1]).all() and (out["idx"] == out["idx"][:1]).all()
        assert not (out["status"] & 2).any()
        got.append((out["signs"][0], out["idx"][0]))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


def _tuned(synth, dtype, d, b):
    from oracle.tuning import tune_log_c
    K, _ = _blocks(synth, dtype, d, b, 2, seed=5 + b)
    return f32(tune_log_c(to_f64(K), target=0.25, center=True))


@pytest.mark.parametrize("dtype,d,b,over", [(torch.bfloat16, 128, 1024, 1), (torch.bfloat16, 128, 896, 32), (torch.bfloat16, 128, 896, 33),
                                            (torch.bfloat16, 128, 512, 1), (torch.float32, 64, 320, 128)])
def test_a_few_more_than_two_blocks_per_compute_unit(bk, synth, dtype, d, b, over):
    """A few more large blocks than two on every compute unit (up to an eighth of them) stay with one at a time, the first of them
    started spread out (compress_kernel); others run two at a time: the blocks of small launches, bit for bit."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n_inst = 2 * n_cu + over
    K, V = _blocks(synth, dtype, d, b, 16, seed=b)
    K = torch.cat([K.roll(k, 0).roll(7 * k, 1) for k in range((n_inst + 15) // 16)])[:n_inst].contiguous()
    V = torch.cat([V.roll(k, 0) for k in range((n_inst + 15) // 16)])[:n_inst].contiguous()
    p = bk.make_params(d, b, 1, dtype, log_c=_tuned(synth, dtype, d, b), seed=9, center=True)
    ids = torch.arange(n_inst, dtype=torch.int64).cuda()
    many = bk.compress_block(p, K, V, inst_ids=ids)
    for lo in range(0, n_inst, n_cu):
        few = bk.compress_block(p, K[lo:lo + n_cu].contiguous(), V[lo:lo + n_cu].contiguous(), inst_ids=ids[lo:lo + n_cu].contiguous())
        for name, x in few.items():
            assert torch.equal(many[name][lo:lo + n_cu], x), name
    assert (many["status"] & 2 == 0).all()


@pytest.mark.parametrize("n_sink,n_recent", [(0, 0), (37, 101)])
@pytest.mark.parametrize("dtype,d,b,per_seq", [(torch.bfloat16, 128, 64, 4), (torch.bfloat16, 128, 128, 8), (torch.bfloat16, 128, 512, 8),
                                               (torch.bfloat16, 128, 1024, 4), (torch.float32, 64, 256, 8), (torch.float32, 64, 448, 4)])
def test_many_sequences_equal_few_in_a_tree(bk, synth, dtype, d, b, per_seq, n_sink, n_recent):
    """Two rounds over more blocks than compute units in each (two blocks per compute unit): survivors' indices, strided windows,
    draws by sequence and block, status words that several blocks share, against the same sequences in groups that
    stay below (seq_base), bit for bit."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n_seq = 3 * n_cu // per_seq + 5 if b <= 256 else 6 * n_cu // per_seq + 5           # (clear of a few more than two per unit)
    group = n_cu // per_seq
    n = b * per_seq + n_sink + n_recent
    base = _blocks(synth, dtype, d, n, 8, seed=b + n_sink)
    K, V = (torch.cat([x.roll(k, 0).roll(11 * k, 1) for k in range((n_seq + 7) // 8)])[:n_seq].contiguous() for x in base)
    p = bk.make_params(d, b, 2, dtype, log_c=_tuned(synth, dtype, d, b), seed=21, center=True)

    def call(lo, hi):
        if n_sink + n_recent:
            return bk.merge_reduce_protected(p, K[lo:hi].contiguous(), V[lo:hi].contiguous(), n_sink, n_recent, seq_base=40 + lo)
        return bk.merge_reduce(p, K[lo:hi].contiguous(), V[lo:hi].contiguous(), seq_base=40 + lo)

    many = call(0, n_seq)
    for lo in range(0, n_seq, group):
        for name, x in call(lo, min(n_seq, lo + group)).items():
            assert torch.equal(many[name][lo:lo + group], x), (name, lo)
    assert (many["status"] & 2 == 0).all()


@pytest.mark.parametrize("dtype,d,b", [(torch.bfloat16, 128, 64), (torch.bfloat16, 128, 128), (torch.float32, 64, 64)])
def test_many_sequences_equal_few_in_carries(bk, synth, dtype, d, b):
    """Carries of more sequences than compute units, with draws given: the same caches in two halves, bit for bit."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n_seq, T = n_cu + 24, 2
    half = n_seq // 2
    p = bk.make_params(d, b, T, dtype, log_c=_tuned(synth, dtype, d, b), seed=3, center=True)
    steps = 2 * b + 1
    K, V = _blocks(synth, dtype, d, steps, 8, seed=b + 1)
    K, V = (torch.cat([x.roll(k, 0).roll(5 * k, 1) for k in range((n_seq + 7) // 8)])[:n_seq].transpose(0, 1).contiguous() for x in (K, V))
    u = torch.rand(T, n_seq, b, generator=torch.Generator().manual_seed(8)).cuda()
    parts = [(0, n_seq), (0, half), (half, n_seq)]
    caches = [bk.Cache(p, hi - lo, 4 * b) for lo, hi in parts]
    status = [torch.zeros(hi - lo, T, dtype=torch.int32, device="cuda") for lo, hi in parts]
    signs = [torch.zeros(T, hi - lo, b, dtype=torch.int8, device="cuda") for lo, hi in parts]
    us = [u[:, lo:hi].contiguous() for lo, hi in parts]
    for j in range(steps):
        done = [c.append_token(K[j, lo:hi].contiguous(), V[j, lo:hi].contiguous(), status=st, uniforms=x, signs=sg)
                for c, (lo, hi), st, x, sg in zip(caches, parts, status, us, signs)]
        assert done[0] == done[1] == done[2] == {b: 1, 2 * b: 2}.get(j + 1, 0)
    n = caches[0].count
    whole = [x[:, :n] for x in caches[0].views()]
    for c, (lo, hi), st, sg in list(zip(caches, parts, status, signs))[1:]:
        assert c.count == n
        for x, y in zip(whole, c.views()):
            assert torch.equal(x[lo:hi], y[:, :n])
        assert torch.equal(status[0][lo:hi], st) and torch.equal(signs[0][:, lo:hi], sg)
    assert caches[0].error_word() == 0


@pytest.mark.parametrize("dtype,d,b", [(torch.bfloat16, 128, 512), (torch.bfloat16, 128, 1024), (torch.float32, 64, 256),
                                       (torch.float32, 128, 320)])
def test_large_common_key_mean(bk, synth, oracle, dtype, d, b):
    """Keys around a common mean of norm 40 (the case the key shift of App. B.5 item 1 exists for): <k_i,k_j> is about
    |mu|^2 = 1600 (more on the outlier channels) for every pair, e^{|mu|^2/sqrt d} is far beyond fp32, and only the
    centred exponent is small.  Kernel weights against the fp64 definition and a teacher-forced halving; no NaN, no
    status bit."""
    n_inst = 3
    t = synth.gqa_layer_bf16(n_seq=n_inst, n=b, d=d, g=1, nq=1, seed=4000 + b, device="cpu", dtype=dtype, mu_norm=40.0)
    K, V = t["K"].cuda().contiguous(), t["V"].cuda().contiguous()
    Kd = to_f64(K)
    assert np.linalg.norm(Kd.mean(axis=1), axis=1).min() > 35.0
    from oracle.tuning import tune_log_c
    log_c = f32(tune_log_c(Kd, target=0.25, center=True))
    p = bk.make_params(d, b, 1, dtype, log_c=log_c, seed=31, center=True)
    # the weights themselves
    Kc = Kd - Kd.mean(axis=1, keepdims=True)
    S = np.einsum("nid,njd->nij", Kc, Kc)
    A = np.max(np.einsum("nii->ni", S), axis=1)
    ref = np.exp((S - A[:, None, None]) / math.sqrt(d) - log_c)
    G = bk.kernel_weights(p, K).cpu().numpy().astype(np.float64)
    offd = ~np.eye(b, dtype=bool)[None].repeat(n_inst, axis=0)
    assert np.isfinite(G[offd]).all()
    big = offd & (ref > 1e-6 * ref[offd].max())
    np.testing.assert_allclose(G[big], ref[big], rtol=2e-3)
    # the walk
    u = np.stack([oracle.uniform_fill(31, s_, 0, b) for s_ in range(n_inst)])
    out = bk.compress_block(p, K, V, uniforms=torch.from_numpy(u.astype(np.float32)).cuda())
    torch.cuda.synchronize()
    signs = out["signs"].cpu().numpy()
    v = verify_halving(oracle, Kd, u, signs, log_c=log_c, center=True)
    print("common mean of norm 40: %d decisions, %d within margin, %d margin flips, %d hard" % (v["n"], v["near"], v["margin"], v["hard"]))
    assert v["hard"] == 0 and np.abs(2 * v["res"]["p"] - 1).mean() > 0.1
    status = out["status"].cpu().numpy()
    assert not np.any(status & 2)                       # no pipeline time-out
    smax = np.abs(v["res"]["sigma"]).max(axis=1)
    clear = np.abs(smax - 1.0) > 1e-3
    np.testing.assert_array_equal((status & 1).astype(bool)[clear], (v["res"]["fails"] > 0)[clear])      # FAIL events as the oracle sees them
    assert np.all(np.isfinite(out["stats"].cpu().numpy()))
    np.testing.assert_array_equal(out["idx"].cpu().numpy(), expected_survivors(oracle, signs))


VALUE_CASES = [
    # dtype, d, b, n_inst, center, r_value (0: measured per block)
    (torch.bfloat16, 128, 256, 4, True, 0.0),     # the largest block whose keys and values share LDS at d=128 bf16
    (torch.bfloat16, 128, 128, 5, True, 0.0),
    (torch.bfloat16, 128, 64, 7, False, 0.0),     # a single panel
    (torch.bfloat16, 64, 512, 3, True, 0.0),      # eight panels
    (torch.bfloat16, 64, 192, 4, False, 30.0),    # three panels, radius given
    (torch.float32, 64, 256, 3, False, 0.0),
    (torch.float32, 128, 128, 3, True, 25.0),
    # blocks whose values do not fit LDS next to the keys: value panels read tile by tile
    (torch.bfloat16, 128, 512, 3, True, 0.0),     # workload 2's block, one chunk of keys
    (torch.bfloat16, 128, 320, 2, False, 0.0),    # five panels
    (torch.bfloat16, 128, 1024, 2, True, 0.0),    # workloads 3-5: two chunks of keys
    (torch.float32, 128, 320, 2, True, 0.0),      # fp32, second chunk of one panel
    (torch.float32, 64, 512, 2, False, 12.0),     # radius given: no norm pass
    (torch.bfloat16, 64, 1024, 2, True, 0.0),
    (torch.float32, 128, 640, 2, True, 0.0),      # fp32, d=128: three chunks of keys
]


@pytest.mark.parametrize("dtype,d,b,n_inst,center,r_value", VALUE_CASES)
@pytest.mark.parametrize("c_kind", ["one", "tuned"])
def test_compress_block_with_value_factor(bk, synth, oracle, dtype, d, b, n_inst, center, r_value, c_kind):
    """Alg. 2 line 6 with its value factor: weights exp(...) <v_i,v_j> / r_value^2, teacher-forced against the oracle."""
    from oracle.tuning import tune_log_c
    K, V = _blocks(synth, dtype, d, b, n_inst, seed=311 + b + d)
    Kd, Vd = to_f64(K), to_f64(V)
    if r_value > 0.0:
        assert r_value ** 2 > (Vd ** 2).sum(-1).max() * 0.25          # a radius of the right order, not the measured one
    log_c = 0.0 if c_kind == "one" else f32(tune_log_c(Kd[:3], target=0.25, center=center, V_blocks=Vd[:3]))
    seed = 0x5EED + b
    p = bk.make_params(d, b, 1, dtype, log_c=log_c, seed=seed, center=center, value_gram=True, r_value=r_value)
    u = np.stack([oracle.uniform_fill(seed, t, 0, b) for t in range(n_inst)])
    out = bk.compress_block(p, K, V, uniforms=torch.from_numpy(u.astype(np.float32)).cuda())
    torch.cuda.synchronize()
    signs = out["signs"].cpu().numpy()
    assert set(np.unique(signs).tolist()) <= {-1, 1}
    assert not np.any(out["status"].cpu().numpy() & 2)                # no internal error
    v = verify_halving(oracle, Kd, u, signs, log_c=log_c, center=center, V_blocks=Vd, r_value=f32(r_value))
    print("c=%s: %d decisions, %d within margin, %d margin flips, %d hard" % (c_kind, v["n"], v["near"], v["margin"], v["hard"]))
    assert v["hard"] == 0
    if c_kind == "tuned":          # (tuned with the measured radius: a given, larger one lowers the activity)
        assert np.abs(2 * v["res"]["p"] - 1).mean() > 0.05
        # ... and they depend on the VALUE factor: the keys-only walk on the same draws decides differently
        keys_only = oracle.softmax_balance_batch(Kd, u=u, log_c=log_c, center=center)
        assert np.count_nonzero(keys_only["eta"] != signs) > 0.05 * signs.size
    idx = out["idx"].cpu().numpy()
    np.testing.assert_array_equal(idx, expected_survivors(oracle, signs))
    gi = torch.from_numpy(idx.astype(np.int64)).cuda()
    assert torch.equal(out["K"], torch.gather(K, 1, gi[..., None].expand(-1, -1, d)))
    assert torch.equal(out["V"], torch.gather(V, 1, gi[..., None].expand(-1, -1, d)))
    stats = out["stats"].cpu().numpy()
    np.testing.assert_allclose(stats[:, 0], np.abs(u - v["res"]["p"]).min(axis=1), atol=2e-5)
    smax = np.abs(v["res"]["sigma"]).max(axis=1)
    inside = smax < 1e25          # beyond: single weights leave the fp32 range the library states as its precondition (decisions still agree)
    np.testing.assert_allclose(stats[inside, 1], smax[inside], rtol=1e-3, atol=1e-5)


@pytest.mark.parametrize("dtype,d,b,n_inst,r_value", [
    (torch.bfloat16, 128, 256, 4, 0.0),       # keys and values in LDS together
    (torch.bfloat16, 128, 512, 3, 0.0),       # value panels from L2
    (torch.bfloat16, 128, 1024, 2, 16.0),     # two chunks of keys, a given radius
    (torch.float32, 64, 256, 3, 0.0),
])
def test_compress_block_with_augmented_value(bk, synth, oracle, dtype, d, b, n_inst, r_value):
    """BKV_VALUE_AUGMENT: the walk sees the value [v / r_value ; 1] (Alg. 2 takes values of any dimension), whose
    radius is sqrt 2.  The oracle is handed exactly those rows of dimension d + 1, so the device's factor
    (<v_i,v_j>/r_value^2 + 1) / 2 is checked against Alg. 2 as listed, teacher-forced.  One block has all-zero values:
    its augmented value is [0 ; 1] with radius 1 (the keys-only walk)."""
    from oracle.tuning import tune_log_c
    K, V = _blocks(synth, dtype, d, b, n_inst, seed=911 + b + d)
    V = V.clone()
    V[-1] = 0                                                      # the last block: no values at all
    Kd, Vd = to_f64(K), to_f64(V)
    radius = np.full(n_inst, r_value) if r_value > 0.0 else np.sqrt((Vd ** 2).sum(-1).max(axis=1))
    if r_value > 0.0:
        assert r_value ** 2 > (Vd ** 2).sum(-1).max()
    seed = 0xA06 + b
    u = np.stack([oracle.uniform_fill(seed, t, 0, b) for t in range(n_inst)])
    Vaug = np.concatenate([Vd / np.where(radius > 0, radius, 1.0)[:, None, None], np.ones((n_inst, b, 1))], axis=-1)
    log_c = f32(tune_log_c(Kd[:2], target=0.25, center=True, V_blocks=Vaug[:2]))      # (measured radius of these rows: sqrt 2)
    p = bk.make_params(d, b, 1, dtype, log_c=log_c, seed=seed, center=True, value_augment=True, r_value=r_value)
    out = bk.compress_block(p, K, V, uniforms=torch.from_numpy(u.astype(np.float32)).cuda())
    torch.cuda.synchronize()
    signs = out["signs"].cpu().numpy()
    stats = out["stats"].cpu().numpy()
    assert not np.any(out["status"].cpu().numpy() & 2)
    tot = dict(hard=0, near=0, n=0)
    for t in range(n_inst):                                        # the radius of the augmented rows differs for the empty block
        r_aug = math.sqrt(2.0) if radius[t] > 0 else 1.0
        v = verify_halving(oracle, Kd[t:t + 1], u[t:t + 1], signs[t:t + 1], log_c=log_c, center=True, V_blocks=Vaug[t:t + 1], r_value=r_aug)
        for k in tot:
            tot[k] += v[k]
        # the weights themselves, through the largest |sigma| of the walk (sensitive to the factor's scale and offset, which
        # the decisions alone need not be: most of them are saturated)
        smax = np.abs(v["res"]["sigma"]).max()
        if smax < 1e25:
            np.testing.assert_allclose(stats[t, 1], smax, rtol=1e-3, atol=1e-5)
        np.testing.assert_allclose(stats[t, 0], np.abs(u[t] - v["res"]["p"][0]).min(), atol=2e-5)
        if t == 0:
            assert np.abs(2 * v["res"]["p"] - 1).mean() > 0.05     # the decisions depend on the weights ...
            plain = oracle.softmax_balance_batch(Kd[:1], Vd[:1], u=u[:1], log_c=log_c, center=True)
            assert np.count_nonzero(plain["eta"] != signs[:1]) > 0  # ... and the factor is not the plain <v_i,v_j>/r^2
            keys_only = oracle.softmax_balance_batch(Kd[:1], u=u[:1], log_c=log_c, center=True)
            assert abs(np.abs(keys_only["sigma"]).max() / smax - 1.0) > 0.05      # ... nor 1
    print("%d decisions, %d within margin, %d hard" % (tot["n"], tot["near"], tot["hard"]))
    assert tot["hard"] == 0
    if r_value == 0.0:      # measured radius: the empty block decides as the keys-only walk does (factor 1; a given radius makes it 1/2)
        ko = oracle.softmax_balance_batch(Kd[-1:], u=u[-1:], log_c=log_c, center=True, forced=signs[-1:])
        assert np.count_nonzero((ko["dec"] != signs[-1:]) & (np.abs(u[-1:] - ko["p"]) >= MARGIN)) == 0
    np.testing.assert_array_equal(out["idx"].cpu().numpy(), expected_survivors(oracle, signs))


def test_merge_reduce_with_value_factor_workload2_blocks(bk, synth, oracle):
    """The tree with the value factor at workload 2's block size (values read from L2 by original index in round 1)."""
    from oracle.tuning import tune_log_c
    dtype, d, b, T, n_seq, n = torch.bfloat16, 128, 512, 2, 2, 4096
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n, d=d, g=1, nq=1, seed=808, device="cpu")
    K, V = t["K"].cuda().contiguous(), t["V"].cuda().contiguous()
    log_c = f32(tune_log_c(to_f64(K[0]).reshape(-1, b, d)[:2], center=True, V_blocks=to_f64(V[0]).reshape(-1, b, d)[:2]))
    p = bk.make_params(d, b, T, dtype, log_c=log_c, seed=3, center=True, value_gram=True)
    res = bk.merge_reduce(p, K, V, emit_signs=True)
    torch.cuda.synchronize()
    assert not np.any(res["status"].cpu().numpy() & 2)
    print("value-factor tree, block 512:", _verify_tree(bk, oracle, K, V, p, res))


def test_value_factor_with_zero_values_is_a_fair_coin(bk, synth, oracle):
    """All value rows zero: every weight is zero (r_value measured as 0 must not divide), p_j = 1/2."""
    dtype, d, b, n_inst = torch.bfloat16, 128, 128, 2
    K, V = _blocks(synth, dtype, d, b, n_inst, seed=5)
    V = torch.zeros_like(V)
    p = bk.make_params(d, b, 1, dtype, log_c=0.0, seed=9, center=True, value_gram=True)
    u = np.stack([oracle.uniform_fill(9, t, 0, b) for t in range(n_inst)])
    out = bk.compress_block(p, K, V, uniforms=torch.from_numpy(u.astype(np.float32)).cuda())
    np.testing.assert_array_equal(out["signs"].cpu().numpy(), np.where(u < 0.5, 1, -1).astype(np.int8))
    assert not np.any(out["status"].cpu().numpy() & 3)


def test_generator_on_device_equals_oracle_draws(bk, synth, oracle):
    """Internal draws (seed, stream = inst_id, ctr = j) == the same run fed the oracle's uniforms."""
    dtype, d, b, n_inst = torch.bfloat16, 128, 256, 5
    K, V = _blocks(synth, dtype, d, b, n_inst, seed=55)
    from oracle.tuning import tune_log_c
    log_c = f32(tune_log_c(to_f64(K)[:2], center=True))
    seed = 0x1234567890ABCDEF
    p = bk.make_params(d, b, 1, dtype, log_c=log_c, seed=seed, center=True)
    ids = torch.tensor([3, 2**40 + 1, 0, 77, 2**62], dtype=torch.int64, device="cuda")
    a = bk.compress_block(p, K, V, inst_ids=ids)
    u = np.stack([oracle.uniform_fill(seed, int(s), 0, b) for s in ids.cpu().tolist()])
    bres = bk.compress_block(p, K, V, uniforms=torch.from_numpy(u.astype(np.float32)).cuda())
    for k in ("signs", "idx", "K", "V", "status"):
        assert torch.equal(a[k], bres[k]), k
    # default streams 0..n_inst-1 and determinism
    c1 = bk.compress_block(p, K, V)
    c2 = bk.compress_block(p, K, V)
    u0 = np.stack([oracle.uniform_fill(seed, t, 0, b) for t in range(n_inst)])
    c3 = bk.compress_block(p, K, V, uniforms=torch.from_numpy(u0.astype(np.float32)).cuda())
    assert torch.equal(c1["signs"], c2["signs"]) and torch.equal(c1["signs"], c3["signs"])
    assert not torch.equal(c1["signs"], a["signs"])


def test_fail_branch_is_reported_not_fatal(bk, synth, oracle):
    """ln c = -40 forces |y^T eta| > c R^2 (Alg. 2 line 7): status bit set, p clamped, output produced."""
    dtype, d, b, n_inst = torch.float32, 64, 128, 3
    K, V = _blocks(synth, dtype, d, b, n_inst, seed=91)
    p = bk.make_params(d, b, 1, dtype, log_c=-40.0, seed=5)
    u = np.stack([oracle.uniform_fill(5, t, 0, b) for t in range(n_inst)])
    out = bk.compress_block(p, K, V, uniforms=torch.from_numpy(u.astype(np.float32)).cuda())
    signs = out["signs"].cpu().numpy()
    assert np.all(out["status"].cpu().numpy() & 1)
    v = verify_halving(oracle, to_f64(K), u, signs, log_c=-40.0, center=False)
    assert v["hard"] == 0 and np.all(v["res"]["fails"] > 0)
    np.testing.assert_array_equal(out["idx"].cpu().numpy(), expected_survivors(oracle, signs))


# ------------------------------------------------------------------------------------------ a8: merge-and-reduce tree
def _verify_tree(bk, oracle, K, V, p, res, seq_base=0, sample=None, rng=None):
    """Teacher-forced check of every round (or of `sample` blocks per round) + exact bookkeeping."""
    n_seq, n, d = K.shape
    b, T, seed = p.block, p.rounds, p.seed
    center = bool(p.flags & 1)
    log_c = float(p.log_c)
    Kd = None if sample else to_f64(K)
    cur = np.tile(np.arange(n, dtype=np.int64), (n_seq, 1))       # surviving original indices per sequence
    tot = dict(hard=0, margin=0, n=0, near=0)
    for r in range(T):
        signs = res["signs"][r].cpu().numpy()                        # [n_seq, n >> r]
        m = n >> r
        nb = m // b
        picks = [(s, blk) for s in range(n_seq) for blk in range(nb)]
        if sample and len(picks) > sample:
            sel = rng.choice(len(picks), size=sample, replace=False)
            picks = [picks[i] for i in sel]
        rows = np.stack([cur[s, blk * b:(blk + 1) * b] for s, blk in picks])
        if Kd is not None:
            Kb = np.stack([Kd[s][rows[i]] for i, (s, _) in enumerate(picks)])
        else:
            Kb = np.stack([to_f64(K[s][torch.from_numpy(rows[i]).cuda()]) for i, (s, _) in enumerate(picks)])
        u = np.stack([oracle.uniform_fill(seed, 64 * (seq_base + s) + r, blk * b, b) for s, blk in picks])
        sg = np.stack([signs[s, blk * b:(blk + 1) * b] for s, blk in picks])
        Vb = None
        if p.flags & bk.BKV_VALUE_GRAM:      # the value rows of the same surviving tokens
            Vb = np.stack([to_f64(V[s][torch.from_numpy(rows[i]).cuda()]) for i, (s, _) in enumerate(picks)])
        v = verify_halving(oracle, Kb, u, sg, log_c=log_c, center=center, V_blocks=Vb, r_value=float(p.r_value))
        for k in tot:
            tot[k] += v[k]
        # survivors of this round from the GPU's own signs (all blocks: integer work only)
        nxt = np.empty((n_seq, m // 2), dtype=np.int64)
        for s in range(n_seq):
            for blk in range(nb):
                keep = oracle.select_half(signs[s, blk * b:(blk + 1) * b], strict=True)
                nxt[s, blk * (b // 2):(blk + 1) * (b // 2)] = cur[s, blk * b + keep]
        cur = nxt
    assert tot["hard"] == 0, tot
    idx = res["idx"].cpu().numpy().astype(np.int64)
    np.testing.assert_array_equal(idx, cur)
    gi = torch.from_numpy(idx).cuda()
    assert torch.equal(res["K"], torch.gather(K, 1, gi[..., None].expand(-1, -1, d)))
    assert torch.equal(res["V"], torch.gather(V, 1, gi[..., None].expand(-1, -1, d)))
    assert torch.all(res["w"] == float(2 ** T))
    return tot


def test_merge_reduce_workload1_full(bk, synth, oracle):
    """Single head, d=64, n=1024 fp32, b=256, one round (keep 512), ln c in {literal, 1, tuned}."""
    from oracle.tuning import tune_log_c
    t = synth.make_workload("cfg1")
    K, V = t["K"].cuda(), t["V"].cuda()
    tuned = f32(tune_log_c(to_f64(K).reshape(4, 256, 64), center=False))
    for log_c in (f32(oracle.log_c_literal(256, 1e-6)), 0.0, tuned):
        p = bk.make_params(64, 256, 1, torch.float32, log_c=log_c, seed=t["cfg"]["seed"], center=False)
        res = bk.merge_reduce(p, K, V, emit_signs=True)
        tot = _verify_tree(bk, oracle, K, V, p, res)
        assert res["K"].shape == (1, 512, 64) and torch.all(res["w"] == 2.0)
        print("workload 1, ln c = %.3f: %s" % (log_c, tot))


def test_merge_reduce_workload2_full(bk, synth, oracle):
    """8 KV heads, d=128, n=16384 bf16, b=512, two rounds (4x), centred keys; every instance checked."""
    from oracle.tuning import tune_log_c
    t = synth.make_workload("cfg2", nq=1)
    K, V = t["K"].cuda(), t["V"].cuda()
    tuned = f32(tune_log_c(to_f64(K[:2, :1024]).reshape(4, 512, 128), center=True))
    p = bk.make_params(128, 512, 2, torch.bfloat16, log_c=tuned, seed=t["cfg"]["seed"], center=True)
    res = bk.merge_reduce(p, K, V, emit_signs=True)
    tot = _verify_tree(bk, oracle, K, V, p, res)
    print("workload 2 (tuned ln c = %.3f): %s" % (tuned, tot))
    assert res["K"].shape == (8, 4096, 128)
    st = res["status"].cpu().numpy()
    assert (st >> 8).sum() >= 0
    # merge_reduce == a chain of compress_block calls fed the tree's draws (checks stream/counter addressing)
    b = 512
    r0 = bk.compress_block(
        bk.make_params(128, b, 1, torch.bfloat16, log_c=tuned, seed=p.seed, center=True), K.view(-1, b, 128), None,
        uniforms=torch.from_numpy(np.stack([oracle.uniform_fill(p.seed, 64 * s + 0, blk * b, b)
                                            for s in range(8) for blk in range(16384 // b)]).astype(np.float32)).cuda())
    assert torch.equal(r0["signs"].view(8, -1), res["signs"][0])


def test_merge_reduce_three_rounds_and_seq_base(bk, synth, oracle):
    from oracle.tuning import tune_log_c
    t = synth.gqa_layer_bf16(n_seq=3, n=128 * 8 * 2, d=64, g=1, nq=1, seed=31, device="cpu")
    K, V = t["K"].cuda(), t["V"].cuda()
    tuned = f32(tune_log_c(to_f64(K[:1, :512]).reshape(4, 128, 64), center=True))
    p = bk.make_params(64, 128, 3, torch.bfloat16, log_c=tuned, seed=99, center=True)
    res = bk.merge_reduce(p, K, V, seq_base=10, emit_signs=True)
    _verify_tree(bk, oracle, K, V, p, res, seq_base=10)
    # sequences are independent: running sequence 1 alone with seq_base 11 gives the same survivors
    one = bk.merge_reduce(p, K[1:2].contiguous(), V[1:2].contiguous(), seq_base=11)
    assert torch.equal(one["idx"][0], res["idx"][1])
    # oracle's free-running offline tree agrees when the GPU met no margin case
    if int((res["status"].cpu().numpy() >> 8).sum()) == 0:
        from oracle.merge_reduce import merge_reduce_offline
        off = merge_reduce_offline(to_f64(K[1]), to_f64(V[1]), b=128, T=3, seed=99, seq=11, log_c=tuned, center=True)
        np.testing.assert_array_equal(off["idx"], res["idx"][1].cpu().numpy())


def test_merge_reduce_with_value_factor(bk, synth, oracle):
    """Three rounds with the value factor: from the second round on the value rows are found through the survivor
    indices.  Also through the protected-window entry point and the streaming cache (same kept set)."""
    from oracle.tuning import tune_log_c
    dtype, d, b, T, n_seq, n = torch.bfloat16, 128, 128, 3, 3, 2048
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n + 96, d=d, g=1, nq=1, seed=4242, device="cpu")
    Kall, Vall = t["K"].cuda().contiguous(), t["V"].cuda().contiguous()
    K, V = Kall[:, 32:32 + n].contiguous(), Vall[:, 32:32 + n].contiguous()
    log_c = f32(tune_log_c(to_f64(K[0]).reshape(-1, b, d)[:3], center=True, V_blocks=to_f64(V[0]).reshape(-1, b, d)[:3]))
    p = bk.make_params(d, b, T, dtype, log_c=log_c, seed=77, center=True, value_gram=True)
    res = bk.merge_reduce(p, K, V, seq_base=5, emit_signs=True)
    torch.cuda.synchronize()
    assert not np.any(res["status"].cpu().numpy() & 2)
    tot = _verify_tree(bk, oracle, K, V, p, res, seq_base=5)
    print("value-factor tree:", tot)
    # the keys-only tree keeps a different set
    res0 = bk.merge_reduce(bk.make_params(d, b, T, dtype, log_c=log_c, seed=77, center=True), K, V, seq_base=5)
    assert not torch.equal(res0["idx"], res["idx"])
    # protected windows around the same rows: identical choice in between (indices shifted by the sink window)
    prot = bk.merge_reduce_protected(p, Kall, Vall, 32, 64, seq_base=5)
    kept = n >> T
    assert torch.equal(prot["idx"][:, 32:32 + kept], res["idx"] + 32)
    assert torch.equal(prot["V"][:, 32:32 + kept], res["V"]) and torch.equal(prot["K"][:, 32:32 + kept], res["K"])


@pytest.mark.parametrize("dtype,d,b,T,n_seq,per_seq,value", [
    (torch.float32, 64, 64, 1, 3, 1, False), (torch.float32, 64, 64, 1, 2, 65, False), (torch.bfloat16, 128, 64, 1, 1, 200, False),
    (torch.bfloat16, 128, 128, 2, 5, 16, False), (torch.bfloat16, 64, 64, 3, 4, 64, True), (torch.bfloat16, 128, 1024, 1, 2, 4, False)])
def test_status_words_without_clearing(bk, synth, dtype, d, b, T, n_seq, per_seq, value):
    """The first round's blocks sum up their events through words of their own, whatever status and workspace held; a captured call, which
    clears the status first and adds to it, is the reference."""
    n = b * (-(-per_seq // (1 << T)) << T)
    t = synth.clustered_layer_bf16(n_seq=n_seq, n=n, d=d, g=1, nq=1, seed=9, device="cuda", dtype=dtype)
    K, V = t["K"], t["V"]
    V[0] = 0.0 if value else V[0]
    p = bk.make_params(d, b, T, dtype, log_c=-8.0, seed=4, center=True, value_gram=value)        # large weights: FAIL events
    need = bk.binding.merge_reduce_workspace_bytes(p, n_seq, n)
    ws = torch.randint(0, 256, (need,), device="cuda", dtype=torch.uint8)
    out = bk.merge_reduce(p, K, V, workspace=ws)
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    ref_ws = torch.zeros_like(ws)
    with torch.cuda.stream(side):
        ref = {k: torch.empty_like(v) for k, v in out.items()}
        with torch.cuda.graph(graph, stream=side):
            bk.merge_reduce(p, K, V, workspace=ref_ws, out=ref)
    graph.replay()
    torch.cuda.synchronize()
    assert (ref["status"] & 1).any() and not (ref["status"] & 2).any()
    for k in out:
        assert torch.equal(out[k], ref[k]), k
    for _ in range(3):                                                   # on what the call before has left
        out["status"].fill_(-1)
        bk.merge_reduce(p, K, V, workspace=ws, out=out)
        assert torch.equal(out["status"], ref["status"])


@pytest.mark.parametrize("dtype,d,b,per_seq,value", [
    (torch.bfloat16, 64, 64, 2, False), (torch.bfloat16, 64, 256, 64, False), (torch.bfloat16, 64, 256, 66, False), (torch.bfloat16, 64, 64, 256, False),
    (torch.bfloat16, 64, 64, 258, False), (torch.bfloat16, 64, 64, 3000, False),                              # (beyond the words: added up)
    (torch.float32, 128, 64, 130, False), (torch.bfloat16, 128, 64, 250, True), (torch.bfloat16, 128, 64, 1500, True)])
def test_status_is_the_sum_over_the_blocks(bk, oracle, dtype, d, b, per_seq, value):
    """One block of a sequence fails, another one in each (rows that are all alike in it, next to orthogonal elsewhere): the first, the last, the
    first of the last 64, the one before, none.  Near ties and the bit are those of the blocks one by one, through words in any state."""
    n_seq, n, seed = 5, per_seq * b, 77
    gen = torch.Generator(device="cuda").manual_seed(per_seq)
    K, V = (torch.randn(n_seq, per_seq, b, d, generator=gen, device="cuda") for _ in range(2))
    failing = [0, per_seq - 1, max(per_seq - 64, 0), max(per_seq - 65, 0)]
    for s, blk in enumerate(failing):
        K[s, blk], V[s, blk] = K[s, blk, :1], V[s, blk, :1]
    K, V = K.to(dtype).view(n_seq, n, d), V.to(dtype).view(n_seq, n, d)
    p = bk.make_params(d, b, 1, dtype, log_c=-0.5, seed=seed, value_gram=value)
    u = np.concatenate([oracle.uniform_fill(seed, 64 * s, 0, n) for s in range(n_seq)]).astype(np.float32).reshape(-1, b)
    blocks = bk.compress_block(p, K.view(-1, b, d), V.view(-1, b, d), uniforms=torch.from_numpy(u).cuda())["status"].view(n_seq, per_seq).cpu()
    assert [x.nonzero().flatten().tolist() for x in blocks & 1] == [[blk] for blk in failing] + [[]]
    near = blocks >> 8
    assert n_seq * n < 30000 or int((near > 0).sum(1).max()) > 1          # (2e-4 of the decisions)
    want = (near.sum(1) << 8) | (blocks & 1).amax(1)
    ws = torch.randint(0, 256, (bk.binding.merge_reduce_workspace_bytes(p, n_seq, n),), device="cuda", dtype=torch.uint8)
    out = bk.merge_reduce(p, K, V, workspace=ws)
    w = out["w"].clone()
    for _ in range(3):
        assert out["status"].flatten().tolist() == want.tolist()
        assert bool((out["w"] == 2.0).all()) and torch.equal(out["w"], w)
        out["status"].fill_(-1)
        bk.merge_reduce(p, K, V, workspace=ws, out=out)


@pytest.mark.parametrize("dtype,d,b,per_seq,sink,recent", [
    (torch.float32, 64, 256, 4, 0, 0), (torch.bfloat16, 64, 64, 130, 0, 0), (torch.bfloat16, 128, 64, 2, 0, 0), (torch.bfloat16, 128, 512, 600, 0, 0),
    (torch.bfloat16, 64, 64, 16, 3, 4), (torch.bfloat16, 64, 64, 16, 2, 4)])
def test_one_round_leaves_the_workspace_alone(bk, synth, dtype, d, b, per_seq, sink, recent):
    """With the indices given a call of one round neither needs nor touches the workspace: two that overlap may have been given the same.  Odd windows
    (weights that words do not fit) and even ones."""
    n = per_seq * b + sink + recent
    t = synth.clustered_layer_bf16(n_seq=3, n=n, d=d, g=1, nq=1, seed=3, device="cuda", dtype=dtype)
    p = bk.make_params(d, b, 1, dtype, log_c=-8.0, seed=4, center=True)
    pattern = torch.randint(0, 256, (bk.binding.merge_reduce_workspace_bytes(p, 3, per_seq * b) + 256,), device="cuda", dtype=torch.uint8)
    ws = pattern.clone()
    call = lambda w: bk.merge_reduce_protected(p, t["K"], t["V"], sink, recent, workspace=w) if sink else bk.merge_reduce(p, t["K"], t["V"], workspace=w)
    out, none = call(ws), call(torch.empty(0, device="cuda", dtype=torch.uint8))
    assert torch.equal(ws, pattern)
    assert (out["status"] & 1).all()
    for k in out:
        assert torch.equal(out[k], none[k]), k
    mid = out["w"][:, sink:out["w"].shape[1] - recent]
    assert bool((mid == 2.0).all()) and out["w"].sum() == 2 * mid.numel() + 3 * (sink + recent)


@pytest.mark.parametrize("dtype,d,b,T,n_sink,n_recent,n_mid", [
    (torch.bfloat16, 128, 512, 2, 256, 256, 4096),      # the paper's windows, workload-2 blocks
    (torch.float32, 64, 128, 1, 40, 7, 512),            # ragged windows
    (torch.bfloat16, 64, 64, 3, 0, 100, 1024),          # no sink
    (torch.bfloat16, 128, 256, 0, 16, 16, 256),         # no rounds: a plain copy
    (torch.bfloat16, 128, 256, 2, 300, 212, 0),         # nothing in between
])
def test_merge_reduce_protected_windows(bk, synth, oracle, dtype, d, b, T, n_sink, n_recent, n_mid):
    """First and recent tokens kept exactly, tree on the rows in between (Full Experimental Details, single-layer
    experiments).  The rows in between must equal bkv_merge_reduce on a copy of those rows (itself checked against the
    oracle above), shifted by the sink; the free-running oracle agrees unless a margin decision occurred."""
    from oracle.merge_reduce import merge_reduce_protected
    from oracle.tuning import tune_log_c
    n = n_sink + n_mid + n_recent
    n_seq = 3
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n, d=d, g=1, nq=1, seed=900 + n, device="cpu", dtype=dtype)
    K, V = t["K"].cuda(), t["V"].cuda()
    nb = min(2, n_mid // b)
    log_c = f32(tune_log_c(to_f64(K[:1, n_sink:n_sink + nb * b]).reshape(nb, b, d), center=True)) if nb else 0.0
    p = bk.make_params(d, b, T, dtype, log_c=log_c, seed=4242, center=True)
    res = bk.merge_reduce_protected(p, K, V, n_sink, n_recent, seq_base=5)
    kept_mid = n_mid >> T
    count = n_sink + kept_mid + n_recent
    idx = res["idx"].cpu().numpy().astype(np.int64)
    assert idx.shape == (n_seq, count)
    np.testing.assert_array_equal(idx[:, :n_sink], np.tile(np.arange(n_sink), (n_seq, 1)))
    np.testing.assert_array_equal(idx[:, count - n_recent:], np.tile(np.arange(n - n_recent, n), (n_seq, 1)))
    w = res["w"].cpu().numpy()
    assert np.all(w[:, :n_sink] == 1.0) and np.all(w[:, count - n_recent:] == 1.0)
    assert np.all(w[:, n_sink:count - n_recent] == float(2 ** T)) and np.all(w.sum(axis=1) == n)
    gi = torch.from_numpy(idx).cuda()
    assert torch.equal(res["K"], torch.gather(K, 1, gi[..., None].expand(-1, -1, d)))
    assert torch.equal(res["V"], torch.gather(V, 1, gi[..., None].expand(-1, -1, d)))
    if T > 0:
        assert int(res["status"].min()) >= 0                    # written by the library for every sequence and round
    if not n_mid:
        assert int(res["status"].abs().sum()) == 0
    if n_mid:
        alone = bk.merge_reduce(p, K[:, n_sink:n - n_recent].contiguous(), V[:, n_sink:n - n_recent].contiguous(), seq_base=5)
        if T > 0:
            np.testing.assert_array_equal(idx[:, n_sink:count - n_recent] - n_sink, alone["idx"].cpu().numpy())
            assert torch.equal(res["status"], alone["status"])
        else:
            np.testing.assert_array_equal(idx[:, n_sink:count - n_recent], np.tile(np.arange(n_sink, n - n_recent), (n_seq, 1)))
        assert torch.equal(res["K"][:, n_sink:count - n_recent], alone["K"])
        if T > 0 and int((res["status"].cpu().numpy() >> 8).sum()) == 0:
            for s in range(n_seq):
                off = merge_reduce_protected(to_f64(K[s]), to_f64(V[s]), b=b, T=T, n_sink=n_sink, n_recent=n_recent, seed=4242,
                                             seq=5 + s, log_c=log_c, center=True)
                np.testing.assert_array_equal(off["idx"], idx[s])
                np.testing.assert_array_equal(off["w"], w[s])


@pytest.mark.parametrize("dtype,d,n_sink,n_recent", [(torch.bfloat16, 64, 1, 0), (torch.float32, 128, 0, 1), (torch.bfloat16, 128, 0, 0),
                                                     (torch.bfloat16, 128, 257, 3)])
def test_protected_windows_of_single_rows(bk, synth, dtype, d, n_sink, n_recent):
    """One launch copies both windows and clears the status words: an empty window, windows of one row, an odd length."""
    n_seq, mid = 5, 256
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n_sink + mid + n_recent, d=d, g=1, nq=1, seed=77, device="cpu", dtype=dtype)
    K, V = t["K"].cuda(), t["V"].cuda()
    p = bk.make_params(d, 128, 1, dtype, log_c=-8.0, seed=3, center=True)
    res = bk.merge_reduce_protected(p, K, V, n_sink, n_recent)
    alone = bk.merge_reduce(p, K[:, n_sink:n_sink + mid].contiguous(), V[:, n_sink:n_sink + mid].contiguous())
    ends = list(range(n_sink)), list(range(n_sink + mid, n_sink + mid + n_recent))
    want = torch.cat([torch.tensor(ends[0], dtype=torch.int32).cuda().expand(n_seq, -1), alone["idx"] + n_sink,
                      torch.tensor(ends[1], dtype=torch.int32).cuda().expand(n_seq, -1)], dim=1)
    assert torch.equal(res["idx"], want) and torch.equal(res["status"], alone["status"])
    gi = want.long()[..., None].expand(-1, -1, d)
    assert torch.equal(res["K"], torch.gather(K, 1, gi)) and torch.equal(res["V"], torch.gather(V, 1, gi))
    w = torch.ones_like(res["w"])
    w[:, n_sink:n_sink + mid // 2] = 2.0
    assert torch.equal(res["w"], w)


def test_merge_reduce_rounds_zero_and_empty(bk, synth):
    t = synth.gqa_layer_bf16(n_seq=2, n=128, d=64, g=1, nq=1, seed=3, device="cpu")
    K, V = t["K"].cuda(), t["V"].cuda()
    p = bk.make_params(64, 64, 0, torch.bfloat16, log_c=0.0)
    res = bk.merge_reduce(p, K, V)
    assert torch.equal(res["K"], K) and torch.equal(res["V"], V) and torch.all(res["w"] == 1.0)
    p1 = bk.make_params(64, 64, 1, torch.bfloat16, log_c=0.0)
    empty = bk.merge_reduce(p1, K[:0].contiguous(), V[:0].contiguous())
    assert empty["K"].shape[0] == 0
    with pytest.raises(bk.BkvError) as e:
        bk.merge_reduce(bk.make_params(64, 64, 2, torch.bfloat16, log_c=0.0), K, V)   # 128 is not a multiple of 64*4
    assert e.value.code == -2


def test_merge_reduce_workload3_sampled(bk, synth, oracle):
    """32 layers x 8 KV heads, n=32768, d=128 bf16, b=1024, T=2, in the launch configuration the
    benchmark uses; 64 sampled instances per round are verified, bookkeeping on all of them."""
    from oracle.tuning import tune_log_c
    cfg = dict(synth.WORKLOADS["cfg3"])
    t = synth.gqa_layer_bf16(cfg["n_seq"], cfg["n"], cfg["d"], cfg["g"], cfg["nq"], seed=cfg["seed"], device="cuda")
    K, V = t["K"], t["V"]
    tuned = f32(tune_log_c(to_f64(K[:2, :2048]).reshape(4, 1024, 128), center=True))
    p = bk.make_params(128, 1024, 2, torch.bfloat16, log_c=tuned, seed=cfg["seed"], center=True)
    res = bk.merge_reduce(p, K, V, emit_signs=True)
    torch.cuda.synchronize()
    tot = _verify_tree(bk, oracle, K, V, p, res, sample=64, rng=np.random.default_rng(0))
    print("workload 3 sampled: %s" % tot)
    assert res["K"].shape == (256, 8192, 128)
    assert not np.any(res["status"].cpu().numpy() & 2)          # no pipeline time-out on any of the 12288 blocks
    # Determinism under load: the same launches once more give the same bytes (the panel pipeline hands data over
    # through counters without barriers; its results must not depend on timing).
    again = bk.merge_reduce(p, K, V, emit_signs=True)
    torch.cuda.synchronize()
    for r in range(2):
        assert torch.equal(again["signs"][r], res["signs"][r])
    assert torch.equal(again["idx"], res["idx"]) and torch.equal(again["status"], res["status"])
    assert torch.equal(again["K"], res["K"]) and torch.equal(again["V"], res["V"])


def test_merge_reduce_workload4_sampled(bk, synth, oracle):
    """64 layers x 8 KV heads, n=131072, d=128 bf16, b=1024, T=3 (the benchmark's default workload, in its launch
    configuration: grids of 65536 / 32768 / 16384 blocks, two on each compute unit): 64 sampled instances per round are
    teacher-forced against the oracle, the survivor bookkeeping is checked on every block."""
    cfg = dict(synth.WORKLOADS["cfg4"])
    t = synth.gqa_layer_bf16(cfg["n_seq"], cfg["n"], cfg["d"], cfg["g"], 1, seed=cfg["seed"], device="cuda")
    K, V = t["K"], t["V"]
    p = bk.make_params(128, 1024, 3, torch.bfloat16, log_c=-82.5617, seed=cfg["seed"], center=True)   # bench.py's ln c
    res = bk.merge_reduce(p, K, V, emit_signs=True)
    torch.cuda.synchronize()
    tot = _verify_tree(bk, oracle, K, V, p, res, sample=64, rng=np.random.default_rng(4))
    print("workload 4 sampled: %s" % tot)
    assert res["K"].shape == (512, 16384, 128)
    assert not np.any(res["status"].cpu().numpy() & 2)


# ------------------------------------------------------------------------------------------ a10: estimator
def _attend_ref(oracle, Kc, Vc, w, Q, count):
    n_seq, g, nq, d = Q.shape
    Kd, Vd, wd, Qd = to_f64(Kc), to_f64(Vc), to_f64(w), to_f64(Q)
    out = np.zeros((n_seq, g, nq, d))
    lse = np.zeros((n_seq, g, nq))
    for s in range(n_seq):
        for a in range(g):
            for i in range(nq):
                out[s, a, i], lse[s, a, i] = oracle.attend(Qd[s, a, i], Kd[s, :count], Vd[s, :count], wd[s, :count])
    return out, lse


@pytest.mark.parametrize("dtype,d,n_seq,count,stride,g,nq", [
    (torch.float32, 64, 1, 512, 512, 1, 16),        # workload 1 after one round
    (torch.bfloat16, 128, 3, 4096, 4096, 4, 2),     # workload 2 shape (fewer queries)
    (torch.bfloat16, 128, 2, 1000, 1024, 4, 1),     # ragged tail, stride > count
    (torch.bfloat16, 64, 2, 77, 80, 3, 1),          # g*nq not a multiple of the query tile
    (torch.float32, 128, 2, 1, 8, 2, 3),            # a single token
    (torch.bfloat16, 128, 1, 20000, 20000, 4, 1),   # many splits
    (torch.bfloat16, 128, 180, 300, 304, 12, 1),    # many sequences: one split each, no merge launch
    (torch.float32, 64, 140, 70, 70, 16, 1),        # the same in fp32
])
def test_attend_matches_oracle(bk, synth, oracle, dtype, d, n_seq, count, stride, g, nq):
    tol = 1e-4 if dtype == torch.float32 else 2e-2
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=stride, d=d, g=g, nq=nq, seed=17 + count, device="cpu", dtype=dtype)
    K, V, Q = t["K"].cuda(), t["V"].cuda(), t["Q"].cuda()
    gen = torch.Generator().manual_seed(count)
    w = (2.0 ** torch.randint(0, 4, (n_seq, stride), generator=gen)).float()
    if count > 8:
        w[:, 5] = 0.0                       # an absent slot in the middle
    w = w.cuda()
    p = bk.make_params(d, 64, 1, dtype, log_c=0.0)
    out, lse = bk.attend_kv(p, K, V, w, Q, count=count)
    torch.cuda.synchronize()
    ref, ref_lse = _attend_ref(oracle, K, V, w, Q, count)
    err = rel_l2(to_f64(out), ref)
    print("attend rel-L2 = %.3e" % err)
    assert err <= tol
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, atol=2e-3 if dtype == torch.bfloat16 else 1e-4)
    # equal weights cancel: plain softmax over the subset (Alg. 1 output line with one level)
    out2, _ = bk.attend_kv(p, K, V, torch.full_like(w, 4.0), Q, count=count)
    out1, _ = bk.attend_kv(p, K, V, torch.ones_like(w), Q, count=count)
    assert rel_l2(to_f64(out2), to_f64(out1)) <= (1e-6 if dtype == torch.float32 else 1e-2)


def test_attend_bf16_weight_rounding_is_bounded(bk, synth):
    """The bf16 path multiplies its value rows by weights of 17 bits (two bf16 numbers) and adds fp32 weights to the denominator;
    the fp32 path keeps fp32 throughout.  The same bf16 values through both paths: the outputs differ by the rounding of the
    output itself (2^-9 relative per element), and the log-denominator shows no bias (weights rounded to bf16 once were cut,
    which shifted it by about -2^-9 = -0.002)."""
    n_seq, count, d, g = 3, 8192, 128, 4
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=count, d=d, g=g, nq=1, seed=404, device="cpu")
    K, V, Q = t["K"].cuda(), t["V"].cuda(), t["Q"].cuda()
    gen = torch.Generator().manual_seed(3)
    w = (2.0 ** torch.randint(0, 4, (n_seq, count), generator=gen)).float().cuda()
    out_b, lse_b = bk.attend_kv(bk.make_params(d, 64, 1, torch.bfloat16, log_c=0.0), K, V, w, Q)
    out_f, lse_f = bk.attend_kv(bk.make_params(d, 64, 1, torch.float32, log_c=0.0), K.float(), V.float(), w, Q.float())
    torch.cuda.synchronize()
    err = rel_l2(to_f64(out_b), to_f64(out_f))
    dl = (lse_b - lse_f).cpu().numpy()
    print("bf16-weight path vs fp32-weight path: rel-L2 %.3e, lse difference mean %.2e max %.2e" % (err, dl.mean(), np.abs(dl).max()))
    assert err <= 4e-3
    assert np.abs(dl).max() <= 1e-3 and abs(dl.mean()) <= 3e-4


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("d,n_seq,count,g,nq", [(128, 8, 4357, 4, 4), (128, 4, 4096, 4, 16), (128, 1, 65536, 8, 2), (64, 8, 4357, 4, 4),
                                                (64, 2, 30000, 8, 5)])
def test_attend_error_against_64_bits(bk, synth, dtype, d, n_seq, count, g, nq):
    """What the attend may lose against a 64-bit evaluation of the same inputs.

    fp32: a dot product of d terms whose partial sums stay small (chains of four, then a tree), one rounding of the exponent's
    argument, one unit of exp2, the sums over the tokens: a few units of 2^-23 together, 7 allowed.  (One chain over the row
    rounds d times at the size of the whole sum; that alone is 8 to 19 units here.)
    bf16: weights carried to 2^-17, fp32 sums, and one rounding of the output to bf16.  So the output is the 64-bit result
    rounded to bf16, except where that lies within 2^-17 times a few of the middle between two bf16 numbers (spacing 2^-7 to 2^-8): at most
    2 % of the elements.  (Weights rounded to bf16 change a third of them.)  The logarithm of the denominator is fp32 all the way:
    a few units of 2^-24 of a logit of up to 64."""
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=count, d=d, g=g, nq=nq, seed=811, device="cuda", dtype=dtype)
    K, V, Q = t["K"], t["V"], t["Q"]
    w = torch.full((n_seq, count), 4.0, device="cuda")
    w[:, int(0.95 * count):] = 2.0
    w[:, int(0.98 * count):] = 1.0
    out, lse = bk.attend_kv(bk.make_params(d, 128, 2, dtype, log_c=0.0), K, V, w, Q)
    q = Q.double().reshape(n_seq, g * nq, d)
    ref = torch.empty_like(q)
    ref_lse = torch.empty(n_seq, g * nq, device="cuda", dtype=torch.float64)
    for s in range(n_seq):
        logit = torch.matmul(q[s], K[s].double().t().contiguous()) / math.sqrt(d) + torch.log(w[s].double())
        ref_lse[s] = torch.logsumexp(logit, -1)
        ref[s] = torch.matmul(torch.exp(logit - ref_lse[s][:, None]), V[s].double())
    out, lse = out.reshape(n_seq, g * nq, d), lse.reshape(n_seq, g * nq).double()
    lse_err = float((lse - ref_lse).abs().max())
    if dtype == torch.float32:
        err = float((out.double() - ref).norm() / ref.norm())
        print("rel-L2 %.2e = %.1f units, lse off by %.1e" % (err, err * 2 ** 23, lse_err))
        assert err <= 7 * 2.0 ** -23
    else:
        off = float((out != ref.to(torch.bfloat16)).double().mean())
        print("differs from the rounded result in %.2f %% of the elements, lse off by %.1e" % (100 * off, lse_err))
        assert off <= 0.02
    assert lse_err <= 8 * 2.0 ** -24 * 64


def _two_set_reference(K, V, w, Kd, wd, Q):
    """Float64: sum over (K, V, w) divided by the normaliser of (Kd, wd); returns (out, ln of the normaliser)."""
    d = K.shape[-1]
    Qf = Q.double().cpu().flatten(1, 2)
    num = w.double().cpu()[:, None] * torch.exp(Qf @ K.double().cpu().transpose(1, 2).contiguous() / d ** 0.5)
    den = (wd.double().cpu()[:, None] * torch.exp(Qf @ Kd.double().cpu().transpose(1, 2).contiguous() / d ** 0.5)).sum(-1)
    return ((num @ V.double().cpu()) / den[..., None]).view(*Q.shape), torch.log(den).view(*Q.shape[:-1])


@pytest.mark.parametrize("dtype,d,n_seq,count,g,nq", [
    (torch.bfloat16, 128, 1, 31, 1, 1), (torch.bfloat16, 128, 2, 32, 1, 15), (torch.bfloat16, 64, 3, 33, 4, 4),      # around one key group
    (torch.bfloat16, 128, 2, 8 * 32 * 3 + 1, 17, 1), (torch.bfloat16, 64, 9, 8 * 32, 33, 1),                         # two query tiles; by XCD
    (torch.bfloat16, 128, 40, 2048 + 16, 4, 1),                                                                      # several steps, four wavefronts
    (torch.bfloat16, 128, 1, 40000, 16, 1),                                                                          # splits merged by a second launch
    (torch.float32, 128, 2, 15, 1, 2), (torch.float32, 64, 3, 17, 16, 1), (torch.float32, 128, 9, 700, 33, 1)])
def test_attend_edges(bk, dtype, d, n_seq, count, g, nq):
    """Edges of the attend pass: key groups (32 / 16 keys), query tiles of 16, ranges split or not, runs of absent tokens, a
    set without a value sum; the workspace arrives with arbitrary content and is used again as the call left it.
    Bounds: fp32 sums of at most 40000 terms, relative 1e-5; bf16 outputs round to nearest (2^-9)."""
    gen = torch.Generator().manual_seed(count + g)
    K, V = torch.randn(n_seq, count, d, generator=gen).to(dtype).cuda(), torch.randn(n_seq, count, d, generator=gen).to(dtype).cuda()
    Q = torch.randn(n_seq, g, nq, d, generator=gen).to(dtype).cuda()
    w = (2.0 ** torch.randint(0, 4, (n_seq, count), generator=gen)).float()
    w[:, count // 3:count // 3 + count // 2] = 0.0                      # absent: whole groups where the range is long enough
    w[0, 0] = 0.0
    w[:, -1] = 2.0
    w = w.cuda()
    m = max(1, count // 2)
    p = bk.make_params(d, 64, 1, dtype, log_c=0.0)
    tol = 1e-5 if dtype == torch.float32 else 4e-3
    ws = torch.full((int(bk.lib().bkv_attend_sets_workspace_bytes(C.byref(p), n_seq, g, nq)),), 0xAB, dtype=torch.uint8, device="cuda")
    ref, ref_lse = _two_set_reference(K, V, w, K, w, Q)
    ref2, ref2_lse = _two_set_reference(K, V, w, K[:, :m], torch.ones(n_seq, m), Q)
    ones = torch.ones(n_seq, m, device="cuda")
    for _ in range(3):
        out, lse = bk.attend_kv(p, K, V, w, Q, workspace=ws)
        assert rel_l2(to_f64(out), ref.numpy()) <= tol
        np.testing.assert_allclose(lse.cpu().numpy(), ref_lse.numpy(), atol=1e-3 if dtype == torch.bfloat16 else 1e-5, rtol=1e-5)
        out, lse = bk.attend_sets(p, (K, V, w), (K[:, :m].contiguous(), ones), Q, workspace=ws)
        assert rel_l2(to_f64(out), ref2.numpy()) <= tol
        np.testing.assert_allclose(lse.cpu().numpy(), ref2_lse.numpy(), atol=1e-3 if dtype == torch.bfloat16 else 1e-5, rtol=1e-5)


@pytest.mark.parametrize("dtype,d,n_seq,count,stride,g", [
    (torch.bfloat16, 128, 64, 10301, 10310, 4), (torch.bfloat16, 128, 701, 999, 1000, 16), (torch.bfloat16, 64, 520, 2600, 2601, 5),      # more than the
    (torch.float32, 128, 41, 8193, 8200, 4), (torch.float32, 64, 90, 8190, 8192, 16),                                                     # caches hold
    (torch.bfloat16, 128, 256, 97, 100, 1), (torch.bfloat16, 128, 200, 1001, 1001, 4), (torch.bfloat16, 64, 64, 4100, 4111, 2)])          # less than that
def test_attend_of_many_sequences_equals_few(bk, dtype, d, n_seq, count, stride, g):
    """Rows read past the caches (those of as many sequences as are too much for them), and sequences enough for several to be on their way in
    a compute unit, against the same sequences eight at a time.  Only the order of the sums differs: outputs to their own rounding (bf16: 2^-9 each) or to that
    of fp32 sums, lse to that of fp32 sums."""
    gen = torch.Generator(device="cuda").manual_seed(count)
    K = torch.randn(n_seq, stride, d, generator=gen, device="cuda", dtype=torch.float32).mul_(2.0).to(dtype)
    V = torch.randn(n_seq, stride, d, generator=gen, device="cuda", dtype=torch.float32).to(dtype)
    Q = torch.randn(n_seq, g, 1, d, generator=gen, device="cuda", dtype=torch.float32).to(dtype)
    w = torch.tensor([0.0, 1.0, 2.0, 4.0], device="cuda")[torch.randint(0, 4, (n_seq, stride), generator=gen, device="cuda")]
    w[:, 64:96] = 0.0                                                    # a group without a live token
    p = bk.make_params(d, 128, 2, dtype, log_c=0.0)
    out, lse = bk.attend_kv(p, K, V, w, Q, count=count)
    for lo in range(0, n_seq, 8):
        s = slice(lo, lo + 8)
        ref, ref_lse = bk.attend_kv(p, K[s].contiguous(), V[s].contiguous(), w[s].contiguous(), Q[s].contiguous(), count=count)
        x, y = out[s].double(), ref.double()
        assert float((x - y).norm() / y.norm()) <= (1e-5 if dtype == torch.float32 else 4e-3)
        torch.testing.assert_close(lse[s], ref_lse, rtol=1e-6, atol=1e-5)


@pytest.mark.parametrize("d,n_seq,more,count,g", [(128, 64, 66, 4100, 4), (64, 64, 66, 4111, 1), (128, 32, 37, 8321, 4)])
def test_attend_cuts_decode_caches_as_ever(bk, d, n_seq, more, count, g):
    """A sequence's token range is cut by the steps that a wavefront takes over all sequences, and by nothing else: a decode attend gives the bits
    it gives among a few more sequences of as many steps (whatever part of the compute units either of them fills)."""
    steps = lambda n: -(-n * -(-count // 32) // 2048)
    assert steps(n_seq) == steps(more)
    gen = torch.Generator(device="cuda").manual_seed(count)
    rand = lambda *shape: torch.randn(*shape, generator=gen, device="cuda").to(torch.bfloat16)
    K, V, Q, w = rand(more, count, d), rand(more, count, d), rand(more, g, 1, d), torch.ones(more, count, device="cuda")
    p = bk.make_params(d, 128, 2, torch.bfloat16, log_c=0.0)
    ref, ref_lse = bk.attend_kv(p, K, V, w, Q)
    out, lse = bk.attend_kv(p, K[:n_seq].contiguous(), V[:n_seq].contiguous(), w[:n_seq].contiguous(), Q[:n_seq].contiguous())
    assert torch.equal(out, ref[:n_seq]) and torch.equal(lse, ref_lse[:n_seq])


@pytest.mark.parametrize("n_seq,count,g,nq", [(8, 4357, 4, 1), (3, 2000, 1, 1), (8, 4096, 4, 16)])
def test_attend_does_not_depend_on_what_the_workspace_holds(bk, n_seq, count, g, nq):
    """A call gives the same bytes on a fresh workspace and on one that holds what an earlier call left there, shifted by anything
    (what two overlapping calls can leave), and on one that replays of a captured call share with eager calls."""
    d = 128
    gen = torch.Generator(device="cuda").manual_seed(5)
    rand = lambda *shape: torch.randn(*shape, generator=gen, device="cuda").to(torch.bfloat16)
    p = bk.make_params(d, 64, 1, torch.bfloat16, log_c=0.0)
    sets = [(rand(n_seq, count, d), rand(n_seq, count, d), rand(n_seq, g, nq, d)) for _ in range(2)]
    w = torch.ones(n_seq, count, device="cuda")
    need = int(bk.lib().bkv_attend_workspace_bytes(C.byref(p), n_seq, count, g, nq))
    fresh = lambda: torch.zeros(need, dtype=torch.uint8, device="cuda")
    want = [bk.attend_kv(p, K, V, w, Q, workspace=fresh()) for K, V, Q in sets]
    ws = fresh()
    K, V, Q = sets[0]
    bk.attend_kv(p, K, V, w, Q, workspace=ws)
    left = ws.clone()
    words = left.view(torch.int64)[: min(left.numel() // 8, 8192)]           # (counters or labels in front of the partials)
    for shift in (0, 1, 2, 3, 5, 16, 17, 33, -1):
        ws.copy_(left)
        ws.view(torch.int64)[: words.numel()] = words + shift
        for k in (1, 0, 1):                                                   # other inputs than the partials there are of
            K, V, Q = sets[k]
            out, lse = bk.attend_kv(p, K, V, w, Q, workspace=ws)
            assert torch.equal(out, want[k][0]) and torch.equal(lse, want[k][1]), "shift %d" % shift
    # a captured call on the same workspace: its replays repeat whatever the launch was given
    K1 = sets[0][0].clone()
    out, lse = torch.empty_like(want[0][0]), torch.empty_like(want[0][1])
    bk.attend_kv(p, K1, sets[0][1], w, sets[0][2], workspace=ws)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out, lse = bk.attend_kv(p, K1, sets[0][1], w, sets[0][2], workspace=ws)
    ref1 = bk.attend_kv(p, sets[1][0], sets[0][1], w, sets[0][2], workspace=fresh())
    for k, shift in ((0, 0), (1, 1), (0, 2), (1, 5), (0, 0)):
        K1.copy_(sets[k][0])
        ws.view(torch.int64)[: words.numel()] += shift
        graph.replay()
        torch.cuda.synchronize()
        ref = ref1 if k else want[0]
        tol = dict(rtol=0, atol=0.01 * float(ref[0].float().abs().max()))     # (other order of the splits' sums: a bf16 unit, 2^-8, here and there)
        torch.testing.assert_close(out.float(), ref[0].float(), **tol)
        torch.testing.assert_close(lse, ref[1], rtol=0, atol=1e-4)
        K, V, Q = sets[1]
        got = bk.attend_kv(p, K, V, w, Q, workspace=ws)
        assert torch.equal(got[0], want[1][0])


@pytest.mark.parametrize("count", [40, 4000])                                     # one split and several
@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.float32, 64)])
def test_attend_shows_what_is_not_finite(bk, dtype, d, count):
    """A NaN in a key, an infinite value and a denominator set without mass are visible in the outputs of their sequence and in no
    other; rows of absent tokens may hold any key."""
    n_seq, g = 3, 2
    gen = torch.Generator(device="cuda").manual_seed(count)
    rand = lambda *shape: torch.randn(*shape, generator=gen, device="cuda").to(dtype)
    p = bk.make_params(d, 64, 1, dtype, log_c=0.0)
    K, V, Kd, Q = rand(n_seq, count, d), rand(n_seq, count, d), rand(n_seq, count, d), 0.1 * rand(n_seq, g, 1, d)
    w, wd = torch.ones(n_seq, count, device="cuda"), torch.ones(n_seq, count, device="cuda")
    at = count - 3
    bad = lambda x, i, v: x.clone().index_put_((torch.tensor(1), torch.tensor(at), torch.tensor(i)), torch.tensor(v, dtype=dtype, device="cuda"))
    ok = [0, 2]
    base, _ = bk.attend_kv(p, K, V, w, Q)
    base2, _ = bk.attend_sets(p, (K, V, w), (Kd, wd), Q)
    assert torch.isfinite(base.float()).all() and torch.isfinite(base2.float()).all()
    # a NaN in a key of the only set, of the numerator set, of the denominator set
    out, _ = bk.attend_kv(p, bad(K, 5, float("nan")), V, w, Q)
    assert torch.equal(out[ok], base[ok]) and torch.isnan(out[1].float()).all()
    out, _ = bk.attend_sets(p, (bad(K, 5, float("nan")), V, w), (Kd, wd), Q)
    assert torch.equal(out[ok], base2[ok]) and torch.isnan(out[1].float()).all()
    out, lse = bk.attend_sets(p, (K, V, w), (bad(Kd, 5, float("nan")), wd), Q)
    assert torch.equal(out[ok], base2[ok]) and not torch.isfinite(out[1].float()).any() and not torch.isfinite(lse[1]).any()
    # a denominator set without mass
    none = wd.clone()
    none[1] = 0.0
    out, lse = bk.attend_sets(p, (K, V, w), (Kd, none), Q)
    assert torch.equal(out[ok], base2[ok]) and not torch.isfinite(out[1].float()).any() and (lse[1] == -math.inf).all()
    # an infinite value: its column is infinite, the others are what they were
    for sign in (1.0, -1.0):
        for call, ref in ((lambda v: bk.attend_kv(p, K, v, w, Q)[0], base), (lambda v: bk.attend_sets(p, (K, v, w), (Kd, wd), Q)[0], base2)):
            out = call(bad(V, 7, sign * math.inf))
            assert (out[1, ..., 7].float() == sign * math.inf).all()
            keep = torch.arange(d, device="cuda") != 7
            assert torch.equal(out[..., keep], ref[..., keep]) and torch.equal(out[ok], ref[ok])
    # an absent token's key may hold anything
    gone = w.clone()
    gone[1, at] = 0.0
    ref, _ = bk.attend_kv(p, K, V, gone, Q)
    assert torch.equal(bk.attend_kv(p, bad(K, 5, float("nan")), V, gone, Q)[0], ref)


@pytest.mark.parametrize("n_seq,count,g,nq", [(511, 40, 1, 1), (512, 700, 2, 1), (513, 700, 1, 16), (128, 1000, 8, 8), (127, 1000, 8, 8), (85, 3000, 1, 5),
                                              (1, 40000, 1, 1), (3, 9000, 17, 1), (2, 31, 1, 1)])
@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 64), (torch.float32, 128)])
def test_attend_stays_within_the_published_workspace(bk, dtype, d, n_seq, count, g, nq):
    """Around the sizes at which ranges are no longer split: the call works with exactly the published bytes and writes nothing behind."""
    gen = torch.Generator(device="cuda").manual_seed(7)
    rand = lambda *shape: torch.randn(*shape, generator=gen, device="cuda").to(dtype)
    K, V, Q = rand(n_seq, count, d), rand(n_seq, count, d), rand(n_seq, g, nq, d)
    w = torch.ones(n_seq, count, device="cuda")
    p = bk.make_params(d, 64, 1, dtype, log_c=0.0)
    want, _ = bk.attend_kv(p, K.float(), V.float(), w, Q.float()) if dtype == torch.float32 else bk.attend_kv(
        bk.make_params(d, 64, 1, torch.float32, log_c=0.0), K.float(), V.float(), w, Q.float())
    tol = 1e-5 if dtype == torch.float32 else 4e-3
    for need, call in ((int(bk.lib().bkv_attend_workspace_bytes(C.byref(p), n_seq, count, g, nq)), lambda ws: bk.attend_kv(p, K, V, w, Q, workspace=ws)[0]),
                       (int(bk.lib().bkv_attend_sets_workspace_bytes(C.byref(p), n_seq, g, nq)),
                        lambda ws: bk.attend_sets(p, (K, V, w), (K, w), Q, workspace=ws)[0])):
        ws = torch.full((need + 65536,), 0xAB, dtype=torch.uint8, device="cuda")
        out = call(ws[:need])
        assert bool((ws[need:] == 0xAB).all())
        assert rel_l2(to_f64(out), to_f64(want)) <= tol


def test_attend_with_as_many_query_groups_as_the_limits_allow(bk):
    """n_seq = 65535 sequences and 129 groups of 32 queries each: 2^23 workgroups of 512 threads and more, which one dimension of a
    grid does not hold.  Queries of zero: the output is the weighted mean of the values, 34 GB of it."""
    n_seq, nq, d, count = 65535, 4097, 64, 3
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("needs 90 GB of device memory")
    gen = torch.Generator(device="cuda").manual_seed(3)
    K = torch.randn(n_seq, count, d, generator=gen, device="cuda").to(torch.bfloat16)
    V = torch.randn(n_seq, count, d, generator=gen, device="cuda").to(torch.bfloat16)
    w = torch.tensor([1.0, 2.0, 4.0], device="cuda").repeat(n_seq, 1)
    Q = torch.zeros(n_seq, 1, nq, d, dtype=torch.bfloat16, device="cuda")
    out = torch.full_like(Q, 7.0)
    ws = torch.empty(int(bk.lib().bkv_attend_workspace_bytes(C.byref(bk.make_params(d, 64, 1, torch.bfloat16, log_c=0.0)), n_seq, count, 1, nq)),
                     dtype=torch.uint8, device="cuda")
    bk.attend_kv(bk.make_params(d, 64, 1, torch.bfloat16, log_c=0.0), K, V, w, Q, workspace=ws, out=out, lse=False)
    want = ((V.double() * w.double()[..., None]).sum(1) / 7.0).to(torch.bfloat16)
    first = out[:, 0, 0]
    off = (first.float() - want.float()).abs().max()
    assert float(off) <= 2.0 ** -7 * float(want.float().abs().max())           # a bf16 unit at a tie
    for s in range(0, n_seq, 4096):                                            # all queries of a sequence alike
        part = out[s:s + 4096, 0]
        assert torch.equal(part.amax(1), first[s:s + 4096]) and torch.equal(part.amin(1), first[s:s + 4096])
    del Q, out, ws
    torch.cuda.empty_cache()


def test_attend_empty_cache(bk, synth):
    t = synth.gqa_layer_bf16(n_seq=2, n=64, d=64, g=2, nq=1, seed=1, device="cpu")
    K, V, Q = t["K"].cuda(), t["V"].cuda(), t["Q"].cuda()
    w = torch.ones(2, 64, device="cuda")
    p = bk.make_params(64, 64, 1, torch.bfloat16, log_c=0.0)
    out, lse = bk.attend_kv(p, K, V, w, Q, count=0)
    assert torch.all(out == 0) and torch.all(torch.isinf(lse) & (lse < 0))


def test_end_to_end_workload1_error_vs_exact(bk, synth, oracle):
    """Compressed-cache attention against Eq. 1 on workload 1: reports eps of Eq. 2 and the relative
    error of App. B.1; asserts the constant-free certificate for the softmax denominator instead of a
    hidden-constant bound."""
    from oracle.tuning import tune_log_c
    t = synth.make_workload("cfg1")
    K, V, Q = t["K"].cuda(), t["V"].cuda(), t["Q"].cuda()
    Kd, Vd, Qd = to_f64(K)[0], to_f64(V)[0], to_f64(Q)[0, 0]
    d = 64
    tuned = f32(tune_log_c(Kd.reshape(4, 256, 64), center=False))
    p = bk.make_params(64, 256, 1, torch.float32, log_c=tuned, seed=1)
    res = bk.merge_reduce(p, K, V, emit_signs=True)
    out, lse = bk.attend_kv(p, res["K"], res["V"], res["w"], Q)
    outd, lsed = to_f64(out)[0, 0], lse.cpu().numpy().astype(np.float64)[0, 0]
    idx = res["idx"].cpu().numpy()[0]
    sgn = -np.ones(1024)
    sgn[idx] = 1.0
    cert = 0.0
    for blk in range(4):
        sl = slice(blk * 256, (blk + 1) * 256)
        Gb = np.exp(Kd[sl] @ Kd[sl].T / math.sqrt(d))
        cert += math.sqrt(sgn[sl] @ Gb @ sgn[sl])
    eps, rel = [], []
    for i in range(Qd.shape[0]):
        q = Qd[i]
        exact = oracle.exact_attention(q, Kd, Vd)
        e = np.exp(Kd @ q / math.sqrt(d))
        assert abs(math.exp(lsed[i]) - e.sum()) <= cert * math.exp(q @ q / (2 * math.sqrt(d))) * (1 + 1e-3)
        sm = e / e.sum()
        eps.append(np.linalg.norm(outd[i] - exact) / (np.linalg.norm(sm) * np.linalg.norm(Vd)))
        rel.append(np.linalg.norm(outd[i] - exact) / np.linalg.norm(exact))
    print("workload 1 vs exact attention: eps(Eq.2) mean %.3f, relative error mean %.3f" % (np.mean(eps), np.mean(rel)))
    assert np.mean(eps) < 1.0


# ------------------------------------------------------------------------------------------ a9: streaming
@pytest.mark.parametrize("value_gram", [False, True])
def test_streaming_cache_equals_offline_tree_and_oracle(bk, synth, oracle, value_gram):
    """Alg. 3 on the device: sum of weights = tokens seen at every step; at multiples of b*2^T the
    state equals the offline tree (same draws); the oracle's stream agrees when no margin case arose.
    Keys-only weights and weights with the value factor of Alg. 2 line 6."""
    from oracle.merge_reduce import MergeAndReduceStream
    from oracle.tuning import tune_log_c
    d, b, T, n_seq = 64, 64, 2, 3
    n = b * 4 * 2 + 37
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n, d=d, g=2, nq=1, seed=77, device="cpu", dtype=torch.float32)
    K, V, Q = t["K"].cuda(), t["V"].cuda(), t["Q"].cuda()
    tuned = f32(tune_log_c(to_f64(K[:, :256]).reshape(-1, 64, 64), center=True,
                           V_blocks=to_f64(V[:, :256]).reshape(-1, 64, 64) if value_gram else None))
    p = bk.make_params(d, b, T, torch.float32, log_c=tuned, seed=4242, center=True, value_gram=value_gram)
    cache = bk.Cache(p, n_seq, max_tokens=512)
    status = torch.zeros(n_seq, T, dtype=torch.int32, device="cuda")
    streams = [MergeAndReduceStream(d, d, t=b, T=T, seed=4242, seq=s, log_c=tuned, center=True, value_gram=value_gram)
               for s in range(n_seq)]
    Kd, Vd = to_f64(K), to_f64(V)
    Kv, Vv, wv = cache.views()
    n_carry = 0
    for j in range(n):
        h = cache.append_token(K[:, j].contiguous(), V[:, j].contiguous(), status)
        exp_h = 0
        if (j + 1) % b == 0:
            pn = (j + 1) // b
            while exp_h < T and pn % (1 << exp_h) == 0:
                exp_h += 1
        assert h == exp_h
        n_carry += h
        for s in range(n_seq):
            streams[s].append(Kd[s, j], Vd[s, j])
        cnt = cache.count
        assert cnt == sum(l.shape[0] for l in streams[0].levels)
        if (j + 1) % 16 == 0 or h:
            assert torch.all(wv[:, :cnt].sum(dim=1) == float(j + 1))
            assert torch.all(wv[:, cnt:] == 0)
    torch.cuda.synchronize()
    assert cache.tokens_seen == n
    margins = int((status.cpu().numpy() >> 8).sum())
    cnt = cache.count
    if margins == 0:
        for s in range(n_seq):
            idx, w = streams[s].flat()
            np.testing.assert_array_equal(to_f64(Kv[s, :cnt]), Kd[s][idx])
            np.testing.assert_array_equal(to_f64(Vv[s, :cnt]), Vd[s][idx])
            np.testing.assert_array_equal(wv[s, :cnt].cpu().numpy(), w)
    # offline tree on the first b*2^T*2 tokens == the level-T part of the stream
    n_full = b * 4 * 2
    off = bk.merge_reduce(p, K[:, :n_full].contiguous(), V[:, :n_full].contiguous())
    assert torch.equal(off["K"], Kv[:, :n_full >> T])
    assert torch.equal(off["V"], Vv[:, :n_full >> T])
    # estimator over all levels == oracle's estimator over the device's own state
    out, lse = cache.attend(Q)
    ref, ref_lse = _attend_ref(oracle, Kv, Vv, wv, Q, cnt)
    assert rel_l2(to_f64(out), ref) <= 1e-4
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, atol=1e-4)
    cache.close()


def test_append_token_uniforms_hook_equals_generator(bk, synth, oracle):
    """The decision-level hooks of bkv_append_token: draws passed in as `uniforms` give the same signs, survivors and
    weights as the generator with the same seed; `signs` carries eta of every carry."""
    d, b, T, n_seq = 64, 64, 2, 2
    n = b * 4
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n, d=d, g=1, nq=1, seed=78, device="cpu")
    K, V = t["K"].cuda(), t["V"].cuda()
    p = bk.make_params(d, b, T, torch.bfloat16, log_c=-20.0, seed=99, center=True)
    caches = [bk.Cache(p, n_seq, max_tokens=2 * n) for _ in range(2)]
    for j in range(n):
        k, v = K[:, j].contiguous(), V[:, j].contiguous()
        carry = (j + 1) % b == 0
        sg = [torch.zeros(T, n_seq, b, dtype=torch.int8, device="cuda") for _ in range(2)] if carry else [None, None]
        u = None
        if carry:      # what the generator would draw: level i, block number (j+1)/b/2^i - 1
            u = torch.zeros(T, n_seq, b, dtype=torch.float32)
            for i in range(T):
                if ((j + 1) // b) % (1 << i) == 0:
                    for s in range(n_seq):
                        u[i, s] = torch.from_numpy(oracle.uniform_fill(99, 64 * s + i, ((j + 1) // b // (1 << i) - 1) * b, b)).float()
            u = u.cuda()
        h0 = caches[0].append_token(k, v, signs=sg[0])
        h1 = caches[1].append_token(k, v, uniforms=u, signs=sg[1])
        assert h0 == h1
        if carry:
            assert torch.equal(sg[0][:h0], sg[1][:h0]) and bool(torch.all(sg[0][:h0].abs() == 1))
            assert bool(torch.all(sg[0][h0:] == 0))                     # levels that did not carry are not written
    v0, v1 = caches[0].views(), caches[1].views()
    for a, c in zip(v0, v1):
        assert torch.equal(a, c)
    for c in caches:
        c.close()


def test_decode_workload_carries_teacher_forced(bk, synth, oracle):
    """The streaming-decode workload at its real per-sequence size, one session (256 KV sequences, d=128 bf16): a
    32768-token prefill (block 1024, two rounds) straight into the cache, then 1024 appended tokens with block 512
    and two levels.  On 64 sampled sequences every carry (two at level 0, one at level 1) is teacher-forced against
    the oracle from the device's own signs, the region behind the prefill's survivors must hold exactly the rows
    and weights that follow from those signs, the free-running oracle stream must agree where the device reported no
    margin decision, and the decode attend is compared with the oracle's estimator on the device's own cache."""
    from oracle.merge_reduce import MergeAndReduceStream
    n_seq, n, d, bd, n_dec = 256, 32768, 128, 512, 1024
    cfg = dict(synth.WORKLOADS["cfg5"])
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n, d=d, g=4, nq=1, seed=cfg["seed"], device="cuda", tail=n_dec)
    K, V, Q = t["K"], t["V"], t["Q"].contiguous()
    Kt, Vt = t["K_tail"], t["V_tail"]
    log_c_pre, log_c_dec, seed_dec = -82.5617, -73.5768, 2
    pre = bk.make_params(d, 1024, 2, torch.bfloat16, log_c=log_c_pre, seed=1, center=True)
    dec = bk.make_params(d, bd, 2, torch.bfloat16, log_c=log_c_dec, seed=seed_dec, center=True)
    cache = bk.Cache(dec, n_seq, max_tokens=(n >> 2) + n_dec + bd)
    st_pre = torch.zeros(n_seq, 2, dtype=torch.int32, device="cuda")
    cache.prefill(pre, K, V, status=st_pre)
    base = cache.count
    assert base == n >> 2
    del K, V
    status = torch.zeros(n_seq, 2, dtype=torch.int32, device="cuda")
    signs = {}
    kt, vt = Kt.transpose(0, 1).contiguous(), Vt.transpose(0, 1).contiguous()
    for j in range(n_dec):
        sg = torch.zeros(2, n_seq, bd, dtype=torch.int8, device="cuda") if (j + 1) % bd == 0 else None
        h = cache.append_token(kt[j], vt[j], status, signs=sg)
        if sg is not None:
            signs[j + 1] = (h, sg)
    out, lse = cache.attend(Q)
    torch.cuda.synchronize()
    assert signs[512][0] == 1 and signs[1024][0] == 2 and cache.count == base + 256
    assert int((st_pre & 2).sum()) == 0 and int((status & 2).sum()) == 0          # no pipeline time-outs
    assert cache.error_word() == 0                                                # ... and the cache's own word agrees
    Kv, Vv, wv = cache.views()
    assert bool(torch.all(wv[:, :base] == 4.0)) and bool(torch.all(wv[:, base:base + 256] == 4.0))
    assert bool(torch.all(wv[:, base + 256:] == 0.0))
    rng = np.random.default_rng(5)
    picks = np.sort(rng.choice(n_seq, size=64, replace=False))
    sel = torch.from_numpy(picks).cuda()
    Ktd, Vtd = to_f64(Kt[sel]), to_f64(Vt[sel])                                   # [64, 1024, d]
    sa = signs[512][1][0][sel].cpu().numpy()
    sb0 = signs[1024][1][0][sel].cpu().numpy()
    sb1 = signs[1024][1][1][sel].cpu().numpy()
    st = status[sel].cpu().numpy()
    tot = dict(hard=0, margin=0, n=0, near=0)
    def check(Kb, u, sg):
        v = verify_halving(oracle, Kb, u, sg, log_c=log_c_dec, center=True)
        for k in tot:
            tot[k] += v[k]
    # level 0, blocks 0 and 1 of each sequence's stream
    check(Ktd[:, :bd], np.stack([oracle.uniform_fill(seed_dec, 64 * int(s), 0, bd) for s in picks]), sa)
    check(Ktd[:, bd:], np.stack([oracle.uniform_fill(seed_dec, 64 * int(s), bd, bd) for s in picks]), sb0)
    keep_a, keep_b = expected_survivors(oracle, sa), expected_survivors(oracle, sb0)
    lvl1 = np.concatenate([keep_a, bd + keep_b], axis=1)                          # [64, 512] positions in the tail, older half first
    check(np.stack([Ktd[i][lvl1[i]] for i in range(64)]),
          np.stack([oracle.uniform_fill(seed_dec, 64 * int(s) + 1, 0, bd) for s in picks]), sb1)
    assert tot["hard"] == 0, tot
    keep_1 = expected_survivors(oracle, sb1)
    final = np.stack([lvl1[i][keep_1[i]] for i in range(64)])                     # [64, 256]
    Kc, Vc = to_f64(Kv[sel, base:base + 256]), to_f64(Vv[sel, base:base + 256])
    free = 0
    for i in range(64):
        np.testing.assert_array_equal(Kc[i], Ktd[i][final[i]])
        np.testing.assert_array_equal(Vc[i], Vtd[i][final[i]])
        if int((st[i] >> 8).sum()) == 0:       # no margin decision: the oracle's own stream keeps the same tokens
            stream = MergeAndReduceStream(d, d, t=bd, T=2, seed=seed_dec, seq=int(picks[i]), log_c=log_c_dec, center=True)
            for j in range(n_dec):
                stream.append(Ktd[i, j], Vtd[i, j])
            idx, w = stream.flat()
            np.testing.assert_array_equal(idx, final[i])
            assert np.all(w == 4.0)
            free += 1
    print("decode workload, 64 sampled sequences: %s, free-running oracle stream compared on %d of them" % (tot, free))
    # the decode attend over the device's own cache (prefill survivors + the streamed region), 64 sequences x 4 heads
    cnt = cache.count
    ref, ref_lse = _attend_ref(oracle, Kv[sel], Vv[sel], wv[sel], Q[sel], cnt)
    err = rel_l2(to_f64(out[sel]), ref)
    print("decode attend rel-L2 = %.3e" % err)
    assert err <= 2e-2
    np.testing.assert_allclose(lse[sel].cpu().numpy(), ref_lse, atol=2e-3)
    cache.close()


def test_cache_load_then_stream(bk, synth, oracle):
    """A prefill result adopted as final survivors, then a fresh Alg. 3 counter with another block size."""
    d, n_seq = 128, 2
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=1024 + 200, d=d, g=4, nq=1, seed=5, device="cpu")
    K, V, Q = t["K"].cuda(), t["V"].cuda(), t["Q"].cuda()
    pre = bk.merge_reduce(bk.make_params(d, 256, 2, torch.bfloat16, log_c=-30.0, seed=1, center=True),
                          K[:, :1024].contiguous(), V[:, :1024].contiguous())
    p = bk.make_params(d, 64, 2, torch.bfloat16, log_c=-30.0, seed=2, center=True)
    cache = bk.Cache(p, n_seq, max_tokens=1024)
    cache.load(pre["K"], pre["V"], pre["w"])
    assert cache.count == 256
    for j in range(200):
        cache.append_token(K[:, 1024 + j].contiguous(), V[:, 1024 + j].contiguous())
    Kv, Vv, wv = cache.views()
    cnt = cache.count
    assert cnt == 256 + 32 + 32 + 8           # 128 -> level 2 (32), 64 -> level 1 (32), 8 raw
    assert torch.all(wv[:, :cnt].sum(dim=1) == 1224.0)
    assert torch.equal(Kv[:, :256], pre["K"])
    out, _ = cache.attend(Q)
    ref, _ = _attend_ref(oracle, Kv, Vv, wv, Q, cnt)
    assert rel_l2(to_f64(out), ref) <= 2e-2
    # capacity is enforced
    small = bk.Cache(p, n_seq, max_tokens=64)
    for j in range(64):
        small.append_token(K[:, j].contiguous(), V[:, j].contiguous())
    assert small.count == 32
    cache.close()
    small.close()


def test_cache_prefill_equals_merge_reduce(bk, synth):
    """Prefill straight into the cache == bkv_merge_reduce followed by bkv_cache_load (one and two rounds)."""
    d, n_seq, n = 128, 3, 2048
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n, d=d, g=4, nq=1, seed=8, device="cpu")
    K, V, Q = t["K"].cuda(), t["V"].cuda(), t["Q"].cuda()
    for T in (1, 2):
        pre = bk.make_params(d, 256, T, torch.bfloat16, log_c=-60.0, seed=3, center=True)
        ref = bk.merge_reduce(pre, K, V)
        dec = bk.make_params(d, 64, 2, torch.bfloat16, log_c=-60.0, seed=4, center=True)
        cache = bk.Cache(dec, n_seq, max_tokens=n)
        status = torch.zeros(n_seq, T, dtype=torch.int32, device="cuda")
        cache.prefill(pre, K, V, status=status)
        Kv, Vv, wv = cache.views()
        cnt = cache.count
        assert cnt == n >> T
        assert torch.equal(Kv[:, :cnt], ref["K"]) and torch.equal(Vv[:, :cnt], ref["V"])
        assert torch.all(wv[:, :cnt] == float(2 ** T)) and torch.all(wv[:, cnt:] == 0)
        assert torch.equal(status, ref["status"])
        o1, _ = cache.attend(Q)
        o2, _ = bk.attend_kv(pre, ref["K"], ref["V"], ref["w"], Q)
        assert torch.equal(o1, o2)
        cache.close()
    with pytest.raises(bk.BkvError) as e:
        small = bk.Cache(dec, n_seq, max_tokens=256)
        small.prefill(bk.make_params(d, 256, 1, torch.bfloat16, log_c=0.0), K, V)
    assert e.value.code == -5


def test_prefill_and_attend_replay_from_a_captured_graph(bk, synth):
    """The launches behind bkv_cache_prefill and bkv_attend are plain kernels (no memset nodes, no allocation, no
    synchronisation), so a caller may capture them: every replay, with unrelated eager work and synchronisations in
    between, must reproduce the eager result bit for bit."""
    d, n_seq, n = 128, 4, 4096
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n, d=d, g=4, nq=1, seed=77, device="cpu")
    K, V, Q = t["K"].cuda(), t["V"].cuda(), t["Q"].cuda()
    pre = bk.make_params(d, 512, 2, torch.bfloat16, log_c=-70.0, seed=5, center=True)
    dec = bk.make_params(d, 512, 2, torch.bfloat16, log_c=-70.0, seed=6, center=True)
    cache = bk.Cache(dec, n_seq, max_tokens=n)
    ws = torch.empty(int(bk.lib().bkv_cache_prefill_workspace_bytes(cache.h, pre, n)), device="cuda", dtype=torch.uint8)
    out = torch.empty(n_seq, 4, 1, d, device="cuda", dtype=torch.bfloat16)

    def step():
        cache.prefill(pre, K, V, workspace=ws)
        cache.attend(Q, out=out, lse=False)

    step()                                          # eager: sets up the attend workspace, function attributes, reference
    torch.cuda.synchronize()
    ref = out.clone()
    Kc_ref = cache.views()[0].clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                   # warm-up on the capture stream, as torch asks
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    other = torch.randn(1 << 20, device="cuda")
    for rep in range(4):
        out.zero_()
        cache.views()[0].zero_()                   # the replay must rebuild the cache and the output
        (other * 2).sum().item()                    # unrelated eager work and a synchronisation between replays
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref), rep
        assert torch.equal(cache.views()[0], Kc_ref), rep
    cache.close()


# ------------------------------------------------------------------------------------------ ablation grid
@pytest.mark.parametrize("recipe", ["clustered", "iid"])
def test_ablation_grid_cell_against_oracle(bk, synth, oracle, recipe):
    """The single-layer ablation (grid of block size x rate, uniform-sampling comparator) on a small instance: the
    per-query errors behind a cell's figures are recomputed by the oracle from the kept sets of the cell's first seed
    (Alg. 1 output line in fp64 against Eq. 1 in fp64), for BalanceKV and for the comparator."""
    from paper_2502_07861_amd import ablation
    r = ablation.run(seeds=1, blocks=(64,), rounds=(1, 2), n_mid=1024, n_seq=2, nq=4, keep_outputs=True, recipe=recipe)
    K, V, Q = to_f64(r["K"]), to_f64(r["V"]), to_f64(r["Q"])
    n = K.shape[1]
    # the yardstick of the study is Eq. 1 itself
    ex = r["exact"].cpu().numpy()
    for s in range(K.shape[0]):
        for a in range(Q.shape[1]):
            np.testing.assert_allclose(ex[s, a, 0], oracle.exact_attention(Q[s, a, 0], K[s], V[s]), rtol=0, atol=1e-9)
    assert [c["rate"] for c in r["cells"]] == ["1/2", "1/4"]
    for c in r["cells"]:
        f = c["first"]
        T = c["rounds"]
        assert c["kept"] == 256 + (1024 >> T) + 256 and c["compress_ms"] > 0
        for idx_t, w_t, z_t, key in ((f["idx"], f["w"], f["z"], "balancekv_rel_err"),
                                     (f["idx_uniform"], f["w_uniform"], f["z_uniform"], "uniform_rel_err")):
            idx, w, z = idx_t.cpu().numpy().astype(np.int64), w_t.cpu().numpy().astype(np.float64), to_f64(z_t)
            errs = []
            for s in range(K.shape[0]):
                assert np.all(np.diff(idx[s]) > 0) and idx[s, 0] == 0 and idx[s, -1] == n - 1 and w[s].sum() == n
                for a in range(Q.shape[1]):
                    for j in range(Q.shape[2]):
                        exact = oracle.exact_attention(Q[s, a, j], K[s], V[s])
                        est = oracle.attend(Q[s, a, j], K[s][idx[s]], V[s][idx[s]], w[s])[0]
                        np.testing.assert_allclose(z[s, a, j], est, rtol=0, atol=2e-2 * np.linalg.norm(est))
                        errs.append(np.linalg.norm(est - exact) / np.linalg.norm(exact))
            # one counted seed: the cell's figure is the mean of exactly these per-query errors, up to the bf16 rounding
            # of the kernel's output (2^-9 relative per element, against |exact|)
            bf16 = 2.0 ** -8 * np.mean([np.linalg.norm(to_f64(z_t)[s]) / np.linalg.norm(ex[s]) for s in range(K.shape[0])])
            assert abs(c[key] - np.mean(errs)) <= 0.02 * np.mean(errs) + bf16
        # the comparator keeps the windows and a duplicate-free sample of the right size in between
        iu = f["idx_uniform"].cpu().numpy()
        assert np.all(iu[:, :256] == np.arange(256)) and np.all(iu[:, -256:] == np.arange(n - 256, n))
        mid = iu[:, 256:-256]
        assert mid.shape[1] == 1024 >> T and np.all((mid >= 256) & (mid < n - 256))


def test_ablation_shows_the_method_on_repeating_keys(bk):
    """On the recipe with repeating keys (norms as App. B.5 reports them) the kept set of BalanceKV answers better than
    a uniform sample of the same size, as Section 4.1 reports for real activations: the softmax normaliser, which
    the keys-only walk balances directly, clearly, and the attention output at rates 1/2 and 1/4."""
    from paper_2502_07861_amd import ablation
    r = ablation.run(seeds=4, blocks=(256,), rounds=(1, 2), recipe="clustered")
    for c in r["cells"]:
        print(c["rate"], "BalanceKV %.4f +- %.4f, uniform %.4f +- %.4f; normaliser %.4f vs %.4f"
              % (c["balancekv_rel_err"], c["balancekv_std"], c["uniform_rel_err"], c["uniform_std"],
                 c["balancekv_normaliser_err"], c["uniform_normaliser_err"]))
        assert c["balancekv_normaliser_err"] < 0.85 * c["uniform_normaliser_err"]
        assert c["balancekv_rel_err"] < c["uniform_rel_err"] - max(c["balancekv_std"], c["uniform_std"])
        assert c["balancekv_rel_err"] < 0.5                      # far from answering zero


# ------------------------------------------------------------------------------------------ Alg. 1: buckets, two instances
def _heavy_tailed_values(V, seed, zero_rows=3, tiny_rows=0):
    """Value rows scaled by 2^U(-3.5, 3.5) per token (several norm buckets), a few zero rows, a few negligible ones."""
    g = torch.Generator().manual_seed(seed)
    n_seq, n, _ = V.shape
    scale = torch.exp2(torch.rand(n_seq, n, generator=g) * 7.0 - 3.5)
    for s in range(n_seq):
        pick = torch.randperm(n, generator=g)
        scale[s, pick[:zero_rows]] = 0.0
        scale[s, pick[zero_rows:zero_rows + tiny_rows]] *= 2.0 ** -40
    return (V.float() * scale[..., None]).to(V.dtype)


def _verify_sets(bk, oracle, which, p, K, V, res, seq_base, eps, r):
    """Teacher-forced check of every halving of bkv_balancekv_sets and exact check of its bookkeeping: buckets, erase
    rule, slot order, the level structure Alg. 3 leaves behind, weights, gathered rows."""
    from oracle.balancekv import bucket_index
    n_seq, n, d = K.shape
    b, T, seed = p.block, p.rounds, p.seed
    center, log_c = bool(p.flags & 1), float(p.log_c)
    Kd, Vd = to_f64(K), to_f64(V)
    slot = res["slot"].cpu().numpy()
    count = res["count"].cpu().numpy()
    idx_out, w_out = res["idx"].cpu().numpy(), res["w"].cpu().numpy()
    cap = idx_out.shape[1]
    tot = dict(hard=0, margin=0, n=0, near=0, borderline=0, segments=0, erased=0)
    for s in range(n_seq):
        if which == bk.BKV_SET_NUMERATOR:
            norms = np.sqrt((Vd[s] ** 2).sum(-1))
            thr = eps / (2.0 * n) * math.exp(-r * r / math.sqrt(d)) * norms.max() if eps > 0 else 0.0
            for t in range(n):
                i = bucket_index(float(norms[t]))
                want = 511 if (i is None or 2.0 ** i <= thr) else 256 + i
                if slot[s, t] != want:          # only a norm on a bucket boundary (or on the erase threshold) may differ
                    near_pow2 = i is not None and abs(math.log2(norms[t]) - round(math.log2(norms[t]))) < 1e-5
                    near_thr = i is not None and thr > 0 and abs(2.0 ** i / thr - 1.0) < 1e-5
                    assert near_pow2 or near_thr, (s, t, norms[t], slot[s, t], want)
                    tot["borderline"] += 1
                tot["erased"] += int(i is not None and slot[s, t] == 511)
        else:
            assert np.all(slot[s] == 0)
        order = np.argsort(slot[s], kind="stable")
        exp_idx, exp_w = [], []
        for sl in np.unique(slot[s]):
            if sl == 511:
                continue
            start = int(np.count_nonzero(slot[s] < sl))
            cur = order[start:start + int(np.count_nonzero(slot[s] == sl))]
            tot["segments"] += 1
            rv = 2.0 ** (int(sl) - 256) if which == bk.BKV_SET_NUMERATOR else 0.0
            left = []                                  # (level, original indices) left behind below level T
            for rd in range(T):
                nb = cur.shape[0] // b
                if nb == 0:
                    break
                blocks = cur[:nb * b].reshape(nb, b)
                sg = res["signs"][rd][s].cpu().numpy()[(start >> rd):(start >> rd) + nb * b].reshape(nb, b)
                assert set(np.unique(sg).tolist()) <= {-1, 1}
                u = np.stack([oracle.uniform_fill(seed, 64 * ((seq_base + s) * 512 + int(sl)) + rd, blk * b, b) for blk in range(nb)])
                v = verify_halving(oracle, Kd[s][blocks], u, sg, log_c=log_c, center=center,
                                   V_blocks=Vd[s][blocks] if which == bk.BKV_SET_NUMERATOR else None, r_value=rv)
                for k in ("hard", "margin", "n", "near"):
                    tot[k] += v[k]
                left.append((rd, cur[nb * b:]))
                cur = np.concatenate([blocks[i][oracle.select_half(sg[i], strict=True)] for i in range(nb)])
            else:
                rd = T
            # `cur` is what reached level rd (= T unless the blocks ran out earlier)
            exp_idx.append(cur); exp_w.append(np.full(cur.shape[0], float(2 ** rd)))
            for lv, rest in reversed(left):
                exp_idx.append(rest); exp_w.append(np.full(rest.shape[0], float(2 ** lv)))
        exp_idx = np.concatenate(exp_idx) if exp_idx else np.zeros(0, dtype=np.int64)
        exp_w = np.concatenate(exp_w) if exp_w else np.zeros(0)
        assert count[s] == exp_idx.shape[0] <= cap
        np.testing.assert_array_equal(idx_out[s, :count[s]], exp_idx)
        np.testing.assert_array_equal(w_out[s, :count[s]], exp_w)
        assert np.all(w_out[s, count[s]:] == 0)
        gi = torch.from_numpy(exp_idx).cuda()
        assert torch.equal(res["K"][s, :count[s]], K[s][gi]) and torch.equal(res["V"][s, :count[s]], V[s][gi])
        assert not res["K"][s, count[s]:].any() and not res["V"][s, count[s]:].any()
        if which == bk.BKV_SET_NUMERATOR:
            kept_w = exp_w.sum()
            assert kept_w == np.count_nonzero(slot[s] != 511)
        else:
            assert exp_w.sum() == n
    assert tot["hard"] == 0, tot
    assert not np.any(res["status"].cpu().numpy() & 2)
    return tot


@pytest.mark.parametrize("dtype,d,b,T,n,n_seq,eps", [
    (torch.bfloat16, 128, 64, 2, 3001, 3, 0.0),
    (torch.bfloat16, 128, 128, 3, 4100, 2, 1e-3),      # with erased buckets
    (torch.float32, 64, 64, 3, 2500, 2, 0.0),
    (torch.bfloat16, 64, 256, 1, 1111, 2, 0.0),
    (torch.bfloat16, 128, 64, 2, 50, 2, 0.0),          # no full block anywhere: nothing is halved
    (torch.bfloat16, 128, 256, 2, 16384, 8, 0.0),      # the sequences of workload 2 at the largest block the value factor takes
    (torch.bfloat16, 64, 64, 2, 333, 300, 0.0),        # many short sequences
    (torch.bfloat16, 128, 512, 2, 9000, 2, 0.0),       # blocks whose values do not fit LDS: value panels from L2, keys through the permutation
    (torch.bfloat16, 128, 1024, 1, 20000, 2, 0.0),     # multi-chunk blocks: keys copied into slot order first
])
def test_balancekv_sets_against_oracle(bk, synth, oracle, dtype, d, b, T, n, n_seq, eps):
    """Alg. 1: bucketed numerator instances (value factor, r_value = 2^i, erase rule) and the keys-only denominator
    instance, each brought to the state of Alg. 3 after the last token, for a ragged n."""
    from oracle.tuning import tune_log_c
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n, d=d, g=2, nq=3, seed=31 + n, device="cpu", dtype=dtype)
    K = t["K"].cuda().contiguous()
    V = _heavy_tailed_values(t["V"], seed=n, tiny_rows=40 if eps > 0 else 0).cuda().contiguous()
    nb = max(1, min(3, n // b))
    Kt = to_f64(K[0, :nb * b]).reshape(nb, -1, d) if n >= b else to_f64(K[:1, :n])
    log_c = f32(tune_log_c(Kt, center=True))
    radius = 1.0          # the radius of the erase rule is an input of Alg. 1; a small one so that the rule has an effect here
    p = bk.make_params(d, b, T, dtype, log_c=log_c, seed=2024, center=True)
    den = bk.balancekv_sets(p, bk.BKV_SET_DENOMINATOR, K, V, seq_base=2, emit_signs=True)
    torch.cuda.synchronize()
    tot_d = _verify_sets(bk, oracle, bk.BKV_SET_DENOMINATOR, p, K, V, den, 2, 0.0, 0.0)
    # the value factor lowers the weights: its own ln c so that decisions still depend on them
    Vt = to_f64(V[0, :nb * b]).reshape(nb, -1, d) if n >= b else to_f64(V[:1, :n])
    pn = bk.make_params(d, b, T, dtype, log_c=f32(tune_log_c(Kt, center=True, V_blocks=Vt)), seed=2024, center=True)
    num = bk.balancekv_sets(pn, bk.BKV_SET_NUMERATOR, K, V, seq_base=2, eps=eps, r=radius, emit_signs=True, max_buckets=12)
    torch.cuda.synchronize()
    tot_n = _verify_sets(bk, oracle, bk.BKV_SET_NUMERATOR, pn, K, V, num, 2, eps, radius)
    print("denominator:", tot_d, "numerator:", tot_n)
    assert tot_n["segments"] >= 5 * n_seq                     # several buckets per sequence
    if eps > 0:
        assert tot_n["erased"] >= 40 * n_seq
    if n >= 8 * b:
        assert tot_n["n"] > 0 and tot_d["n"] > 0
    # Alg. 1 output line over the two sets == the same ratio in fp64 from the device's own sets
    Q = t["Q"].cuda().contiguous()
    out, lse = bk.attend_sets(p, (num["K"], num["V"], num["w"]), (den["K"], den["w"]), Q)
    torch.cuda.synchronize()
    Kn, Vn, wn = to_f64(num["K"]), to_f64(num["V"]), num["w"].cpu().numpy().astype(np.float64)
    Kdn, wd = to_f64(den["K"]), den["w"].cpu().numpy().astype(np.float64)
    Qd = to_f64(Q)
    ref = np.zeros_like(Qd)
    ref_lse = np.zeros(Qd.shape[:3])
    for s in range(n_seq):
        for a in range(Qd.shape[1]):
            for j in range(Qd.shape[2]):
                q = Qd[s, a, j]
                ln, ld = Kn[s] @ q / math.sqrt(d), Kdn[s] @ q / math.sqrt(d)
                m = max(ln.max(), ld.max())
                den_sum = (wd[s] * np.exp(ld - m)).sum()
                ref[s, a, j] = (wn[s] * np.exp(ln - m)) @ Vn[s] / den_sum
                ref_lse[s, a, j] = m + math.log(den_sum)
    assert rel_l2(to_f64(out), ref) <= (1e-4 if dtype == torch.float32 else 2e-2)
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, atol=1e-3 if dtype == torch.float32 else 2e-2)


@pytest.mark.parametrize("n_seq,group,n,eps", [(40, 4, 32768, 0.0), (11, 1, 32767, 0.0), (72, 9, 12000, 3e3)])
def test_balancekv_sets_many_sequences_equal_few(bk, n_seq, group, n, eps):
    """Many sequences of many chunks have the counts of the chunks summed by a launch of its own; the same sequences in small groups
    (seq_base) do not: the same sets, bit for bit."""
    d, b, T = 64, 64, 2
    gen = torch.Generator(device="cuda").manual_seed(n)
    K = torch.randn(n_seq, n, d, generator=gen, device="cuda").to(torch.bfloat16)
    V = (torch.randn(n_seq, n, d, generator=gen, device="cuda") *
         torch.exp2(torch.rand(n_seq, n, 1, generator=gen, device="cuda") * 5 - 2.5)).to(torch.bfloat16)
    V[:, 17] = 0.0                                                            # a row of no bucket
    p = bk.make_params(d, b, T, torch.bfloat16, log_c=-57.0, seed=11, center=True, value_gram=True)
    call = lambda lo, hi: bk.balancekv_sets(p, bk.BKV_SET_NUMERATOR, K[lo:hi].contiguous(), V[lo:hi].contiguous(), seq_base=lo, eps=eps,
                                            max_buckets=12)
    whole = call(0, n_seq)
    for lo in range(0, n_seq, group):
        part = call(lo, min(n_seq, lo + group))
        for name in ("K", "V", "w", "idx", "count", "slot", "status"):
            assert torch.equal(whole[name][lo:lo + group], part[name]), (name, lo)


@pytest.mark.parametrize("dtype,d,b,per_seq,T", [
    (torch.bfloat16, 128, 64, 8, 2), (torch.bfloat16, 128, 512, 4, 2), (torch.bfloat16, 128, 576, 4, 2), (torch.bfloat16, 128, 1024, 4, 2),
    (torch.bfloat16, 128, 128, 8, 3), (torch.float32, 64, 64, 8, 3), (torch.float32, 64, 512, 4, 2)])
def test_balancekv_sets_denominator_many_sequences_equal_few(bk, synth, dtype, d, b, per_seq, T):
    """An instance table of more blocks than compute units runs two blocks on each (another kernel), in the first round and in later
    ones (rows found through the indices of the round before, no rows stored in the last); the same sequences in groups whose
    tables have at most one block per compute unit: the same signs and the same bits."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n_seq, group, n = n_cu // (per_seq // 2) + 5, n_cu // per_seq, b * per_seq + 37
    assert n_seq * (per_seq // 2) > n_cu >= group * per_seq
    K, _ = _blocks(synth, dtype, d, 64, 32, seed=b + d)
    base = K.view(-1, d)
    at = torch.arange(n_seq * n, dtype=torch.int64)
    K = base[((at * 1009 + at // n * 37 + at // 2048) % base.shape[0]).cuda()].view(n_seq, n, d).contiguous()
    V = K.roll(1, 2).contiguous()
    p = bk.make_params(d, b, T, dtype, log_c=_tuned(synth, dtype, d, b), seed=41, center=True)
    call = lambda lo, hi: bk.balancekv_sets(p, bk.BKV_SET_DENOMINATOR, K[lo:hi].contiguous(), V[lo:hi].contiguous(), seq_base=lo, emit_signs=True)
    whole = call(0, n_seq)
    assert not (whole["status"] & 2).any()
    for lo in range(0, n_seq, group):
        hi = min(n_seq, lo + group)
        part = call(lo, hi)
        torch.cuda.synchronize()
        for name in ("K", "w", "idx", "count", "status"):
            assert torch.equal(whole[name][lo:hi], part[name]), (name, lo)
        for r in range(T):                                                    # the halvings' rows of the level-r buffers
            rows = (per_seq >> r) * b
            assert rows and torch.equal(whole["signs"][r][lo:hi, :rows], part["signs"][r][:, :rows]), (r, lo)


def test_balancekv_sets_replay_from_a_captured_graph(bk, synth):
    """Both set builds and the two-set output line are plain kernel launches without host round trips (grids are upper
    bounds, counts stay on the device): captured once, every replay reproduces the eager result bit for bit."""
    dtype, d, b, T, n, n_seq = torch.bfloat16, 128, 128, 2, 3000, 3
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n, d=d, g=2, nq=2, seed=123, device="cpu", dtype=dtype)
    K, Q = t["K"].cuda().contiguous(), t["Q"].cuda().contiguous()
    V = _heavy_tailed_values(t["V"], seed=9).cuda().contiguous()
    p = bk.make_params(d, b, T, dtype, log_c=-62.0, seed=77, center=True)

    def step():
        num = bk.balancekv_sets(p, bk.BKV_SET_NUMERATOR, K, V, eps=1e-4, r=1.0, max_buckets=12)
        den = bk.balancekv_sets(p, bk.BKV_SET_DENOMINATOR, K, V)
        out, lse = bk.attend_sets(p, (num["K"], num["V"], num["w"]), (den["K"], den["w"]), Q)
        return num, den, out, lse

    num0, den0, out0, lse0 = step()
    torch.cuda.synchronize()
    assert int(num0["count"].min()) > 0 and not bool(torch.isnan(out0.float()).any())
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        num, den, out, lse = step()
    other = torch.randn(1 << 20, device="cuda")
    for rep in range(3):
        for tns in (num["idx"], num["w"], num["K"], num["count"], den["idx"], den["w"], out, lse):
            tns.zero_()
        (other * 2).sum().item()
        graph.replay()
        torch.cuda.synchronize()
        for k in ("idx", "w", "K", "V", "count", "slot", "status"):
            assert torch.equal(num[k], num0[k]), (rep, "numerator", k)
            assert torch.equal(den[k], den0[k]), (rep, "denominator", k)
        assert torch.equal(out, out0) and torch.equal(lse, lse0), rep


def test_balancekv_sets_equal_the_oracle_stream(bk, synth, oracle):
    """Small instance against the oracle's Alg. 1 run token by token (free-running): identical sets per bucket and
    identical denominator set unless a near-tie decision or a norm on a bucket boundary occurred; the estimate over
    the device's sets equals the oracle's output line."""
    from oracle.balancekv import BalanceKVStream
    dtype, d, b, T, n, n_seq = torch.float32, 64, 64, 2, 777, 5
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n, d=d, g=1, nq=2, seed=99, device="cpu", dtype=dtype)
    K = t["K"].cuda().contiguous()
    V = _heavy_tailed_values(t["V"], seed=5).cuda().contiguous()
    p = bk.make_params(d, b, T, dtype, log_c=-30.0, seed=31337, center=True)
    num = bk.balancekv_sets(p, bk.BKV_SET_NUMERATOR, K, V, seq_base=1)
    den = bk.balancekv_sets(p, bk.BKV_SET_DENOMINATOR, K, V, seq_base=1)
    Q = t["Q"].cuda().contiguous()
    out, _ = bk.attend_sets(p, (num["K"], num["V"], num["w"]), (den["K"], den["w"]), Q)
    torch.cuda.synchronize()
    near = (num["status"].cpu().numpy() >> 8).sum(axis=1) + (den["status"].cpu().numpy() >> 8).sum(axis=1)
    Kd, Vd, Qd = to_f64(K), to_f64(V), to_f64(Q)
    compared = 0
    for s in range(n_seq):
        st = BalanceKVStream(d, d, t=b, T=T, n_total=n, seed=31337, seq=1 + s, log_c=f32(-30.0), center=True)
        for j in range(n):
            st.append(Kd[s, j], Vd[s, j])
        if near[s]:           # a decision within 1e-4 of its draw may legitimately go the other way: no set comparison
            continue
        cnt = int(num["count"][s])
        idx, w, slot = num["idx"][s, :cnt].cpu().numpy(), num["w"][s, :cnt].cpu().numpy(), num["slot"][s].cpu().numpy()
        sets = st.numerator_sets()
        assert sorted(256 + i for i in sets) == sorted(set(slot.tolist()) - {511})
        pos = 0
        for i in sorted(sets):
            ei, ew = sets[i]
            np.testing.assert_array_equal(idx[pos:pos + ei.shape[0]], ei)
            np.testing.assert_array_equal(w[pos:pos + ei.shape[0]], ew)
            pos += ei.shape[0]
        assert pos == cnt
        di, dw = st.denominator_set()
        cd = int(den["count"][s])
        np.testing.assert_array_equal(den["idx"][s, :cd].cpu().numpy(), di)
        np.testing.assert_array_equal(den["w"][s, :cd].cpu().numpy(), dw)
        for j in range(Qd.shape[2]):
            assert rel_l2(to_f64(out[s, 0, j]), st.estimate(Qd[s, 0, j])) <= 1e-4
        compared += 1
    print("near-tie decisions per sequence: %s, sequences compared with the oracle stream: %d" % (near.tolist(), compared))
    assert compared >= 2


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.float32, 64)])
@pytest.mark.parametrize("n,eps", [(1, 0.0), (255, 0.0), (257, 1e-4), (513, 0.0), (33001, 0.0), (70000, 1e-4)])
def test_balancekv_sets_keep_every_token_in_slot_order(bk, dtype, d, n, eps):
    """Without rounds the kept set is the stable partition itself: chunks of one token, of a remainder, of more than 256 tokens, more
    tokens than 128 chunks of 256.  Slots against the norms in fp64 (rows near a power of two may go either way)."""
    n_seq = 2
    gen = torch.Generator().manual_seed(n)
    scale = torch.exp2(torch.rand(n_seq, n, 1, generator=gen) * 6 - 3)
    V = (torch.randn(n_seq, n, d, generator=gen) * scale)
    V[:, n // 2] = 0.0                                                       # a row of no bucket
    V, K = V.to(dtype).cuda(), torch.randn(n_seq, n, d, generator=gen).to(dtype).cuda()
    p = bk.make_params(d, 64, 0, dtype, log_c=0.0, seed=1, center=True)
    num = bk.balancekv_sets(p, bk.BKV_SET_NUMERATOR, K, V, capacity=n, eps=eps, r=0.0)
    norm = V.double().norm(dim=-1)
    want = torch.where(norm > 0, 256 + torch.ceil(torch.log2(norm.clamp_min(1e-30))).int(), 511)
    if eps > 0:
        gone = torch.exp2(2.0 * (want - 256)) <= (eps / (2 * n)) ** 2 * norm.max(dim=1, keepdim=True).values ** 2
        want = torch.where(gone, 511, want)
    near = (torch.log2(norm.clamp_min(1e-30)) - torch.round(torch.log2(norm.clamp_min(1e-30)))).abs() < 1e-5
    assert torch.all((num["slot"] == want) | near)
    for s in range(n_seq):
        order = torch.argsort(num["slot"][s], stable=True)
        order = order[: int((num["slot"][s] != 511).sum())]
        c = int(num["count"][s])
        assert c == order.numel() and torch.equal(num["idx"][s, :c].long(), order)
        assert torch.equal(num["K"][s, :c], K[s, order]) and torch.equal(num["V"][s, :c], V[s, order])
        assert torch.all(num["w"][s, :c] == 1.0) and torch.all(num["w"][s, c:] == 0.0) and torch.all(num["K"][s, c:] == 0)
    den = bk.balancekv_sets(p, bk.BKV_SET_DENOMINATOR, K, V, capacity=n)
    assert torch.equal(den["idx"], torch.arange(n, dtype=torch.int32, device="cuda").expand(n_seq, -1)) and torch.equal(den["K"], K)


def test_balancekv_sets_degenerate_cases(bk, synth, oracle):
    """No rounds (everything kept with weight 1: the two-set output line is exact attention, Eq. 1), a capacity below
    the count (the surplus is not written, the count is still reported), all value rows zero (empty numerator set:
    the output is zero), and an erase threshold that leaves only the top buckets."""
    dtype, d, n, n_seq = torch.float32, 64, 700, 2
    t = synth.gqa_layer_bf16(n_seq=n_seq, n=n, d=d, g=2, nq=2, seed=4, device="cpu", dtype=dtype)
    K, Q = t["K"].cuda().contiguous(), t["Q"].cuda().contiguous()
    V = _heavy_tailed_values(t["V"], seed=1, zero_rows=5).cuda().contiguous()
    Kd, Vd, Qd = to_f64(K), to_f64(V), to_f64(Q)
    # T = 0
    p0 = bk.make_params(d, 64, 0, dtype, log_c=0.0, seed=1, center=True)
    num = bk.balancekv_sets(p0, bk.BKV_SET_NUMERATOR, K, V, capacity=n)
    den = bk.balancekv_sets(p0, bk.BKV_SET_DENOMINATOR, K, V, capacity=n)
    assert num["count"].tolist() == [n - 5] * n_seq and den["count"].tolist() == [n] * n_seq
    assert torch.all(num["w"][:, :n - 5] == 1.0) and torch.all(num["w"][:, n - 5:] == 0.0) and torch.all(den["w"] == 1.0)
    for s in range(n_seq):       # every row with a non-zero value exactly once, bucket by bucket in arrival order
        idx = num["idx"][s, :n - 5].cpu().numpy()
        assert sorted(idx.tolist()) == np.flatnonzero((Vd[s] ** 2).sum(-1) > 0).tolist()
        slot = num["slot"][s].cpu().numpy()
        assert np.all(np.diff(slot[idx]) >= 0) and np.all(np.diff(idx)[np.diff(slot[idx]) == 0] > 0)
    out, _ = bk.attend_sets(p0, (num["K"], num["V"], num["w"]), (den["K"], den["w"]), Q)
    ref = np.stack([[[oracle.exact_attention(Qd[s, a, j], Kd[s], Vd[s]) for j in range(Qd.shape[2])] for a in range(Qd.shape[1])]
                    for s in range(n_seq)])
    assert rel_l2(to_f64(out), ref) <= 1e-4
    # capacity below the count
    p2 = bk.make_params(d, 64, 2, dtype, log_c=-20.0, seed=1, center=True)
    full = bk.balancekv_sets(p2, bk.BKV_SET_NUMERATOR, K, V, max_buckets=16)
    cut = bk.balancekv_sets(p2, bk.BKV_SET_NUMERATOR, K, V, capacity=100)
    assert torch.equal(cut["count"], full["count"]) and int(full["count"].min()) > 100
    assert torch.equal(cut["idx"], full["idx"][:, :100]) and torch.equal(cut["K"], full["K"][:, :100])
    # all values zero: nothing in the numerator, output zero; the denominator is unaffected
    Vz = torch.zeros_like(V)
    numz = bk.balancekv_sets(p2, bk.BKV_SET_NUMERATOR, K, Vz, max_buckets=16)
    assert numz["count"].tolist() == [0] * n_seq and not numz["w"].any() and bool(torch.all(numz["slot"] == 511))
    den2 = bk.balancekv_sets(p2, bk.BKV_SET_DENOMINATOR, K, Vz)
    outz, lsez = bk.attend_sets(p2, (numz["K"], numz["V"], numz["w"]), (den2["K"], den2["w"]), Q, count_n=0)
    assert not outz.any() and bool(torch.isfinite(lsez).all())
    # an erase threshold just below the largest norm's bucket: only buckets above it survive
    norms = np.sqrt((Vd ** 2).sum(-1))
    eps = 2.0 * n * 0.3                      # threshold = 0.3 * v_max with r = 0
    er = bk.balancekv_sets(p2, bk.BKV_SET_NUMERATOR, K, V, eps=eps, r=0.0, max_buckets=16)
    for s in range(n_seq):
        slot = er["slot"][s].cpu().numpy()
        thr = 0.3 * norms[s].max()
        kept = slot != 511
        assert kept.any() and np.all(2.0 ** (slot[kept] - 256) > thr) and np.all(2.0 ** np.ceil(np.log2(norms[s][~kept & (norms[s] > 0)])) <= thr * (1 + 1e-6))


def test_decode_workload_one_session(bk):
    """The streaming-decode workload at its real per-sequence size (32768-token prefill, 1024 appended tokens, carries
    after every 512th, GQA-4 attends) for one session = 256 KV sequences: the module checks at nine points of the stream
    that the weights of every sequence add up to the tokens seen, that nothing beyond the count carries weight, that the
    attend output is finite, and at the end the number of halvings and the stored count."""
    from paper_2502_07861_amd import decode_workload
    assert decode_workload.main(["--sessions", "1"]) == 0
