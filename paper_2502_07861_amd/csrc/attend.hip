// Decode attention against the compressed, weighted cache (Alg. 1 output line of arXiv 2502.07861):
//   z = sum_i w_i e^{<k_i,q>/sqrt d} v_i / sum_i w_i e^{<k_i,q>/sqrt d},  w_i = 2^level(i).
// w_i e^x = 2^{x log2(e) + log2 w_i}: a softmax with logit bias log2 w_i, evaluated with a running reference exponent.
// Optionally numerator and denominator run over two sets of their own (Alg. 1 as listed).
//
// Both contractions run on the matrix cores in 16x16 tiles and nothing is staged through LDS: a wavefront takes groups
// of kKeys keys (32 bf16, 16 fp32) straight from memory into operand registers.  With lane = 16 kg + n:
//   S^T = K Q^T   rows = keys, columns = queries.  Lane (n, kg) holds piece kg of every 64 bytes of key row n (A) and of
//                 query n (B): the same pieces, so the contraction meets every column once.  Result: query n, keys 4 kg + r.
//   O^T += V^T P  the weights are already where the next product wants them (column = query n, the lane's own keys), if the
//                 lane loads the value rows of exactly those keys.  It takes columns d = kEpn n + e, e < kEpn, of each (16
//                 lanes cover a row; of fp32 rows of 512 bytes 4 n + e and 64 + 4 n + e, e < 4, so that a load covers 256 bytes
//                 without gaps): element e is operand row n of product e.  bf16 pairs two keys per register by a byte
//                 permute; fp32 elements are operands as they are.
// So the pass needs no transposes, and a query's weights, running reference and sums stay in its own lanes.
// What bounds it: with few queries per sequence the stream over K, V, w (1024 sequences x 8321 tokens x 4 queries, bf16:
// 631 to 649 us from box to box = 6.7 to 6.9 TB/s, 707 to 712 with the rows kept in the caches); with many (16 or 32 queries share every load) the latency of the loads from L2 and the merge (8 x 4096
// tokens x 256 queries: 25 us; 114 us on the vector units, four queries per pass); short ranges the sum of two memory
// round trips and the hand-over between workgroups (8 x 4357 tokens: 11.3 us in one launch; 14 us as pass + merge launches).
#include <unistd.h>

#include <atomic>
#include <chrono>
#include <utility>

#include "bkv_device.h"
#include "bkv_host.h"

namespace bkv {

constexpr int kOneGroups = 128;              // groups of a set that one workgroup looks through (attend_in_one)
constexpr int kTargetWaves = 2048;           // wavefronts of the pass when token ranges are split (see attend_plan)
constexpr int kRowPad = 4;                   // floats behind the D sums of a partial row: [0] reference exponent, [1] denominator
constexpr float kNeg = -1.0e30f;             // "minus infinity" that stays finite under subtraction
constexpr float kSlack = 6.f;                // weights may exceed the running reference by 2^6 before it moves

typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4)));     // four consecutive weights, any alignment
typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------------------------------------------------
// "Is everybody's partial there?", without anybody having cleared anything before: the workspace is the caller's, arrives with
// any content, and nothing that a call leaves in it means anything to a later one.  Every workgroup stores the launch's number,
// which no other launch of the process has, into a word of its own behind its partial, waits until that has arrived, and then
// reads the words of its group.  The workgroup whose word arrives last finds them all and merges.  (Workgroups that arrive
// together may all find them: they merge the same partials in the same order and store the same bytes.)  A call that overlaps
// another one on the same memory may find its words overwritten; the next call does not look at them.  Replays of a captured
// launch would repeat its number, so a captured call merges in a launch of its own.
// Called by one wavefront after the workgroup's partial has arrived.
__device__ __forceinline__ bool all_arrived(unsigned long long* words, unsigned int mine, unsigned int total, unsigned long long label) {
    const unsigned int lane = threadIdx.x & 63u;
    if (lane == 0) __hip_atomic_store(words + mine, label, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    bool there = true;
    for (unsigned int w = lane; w < total; w += 64u)
        there &= __hip_atomic_load(words + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == label;
    return __ballot(!there) == 0ull;
}

// Partial rows travel between workgroups (other XCDs, other L2s) past the caches, two floats at a time: device-scope
// accesses, ordered by waiting for them.  A release fence per workgroup would write back its XCD's whole L2 instead, which
// made a pass of 500 workgroups twice as long.
__device__ __forceinline__ void put2(float* p, float x, float y) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), __builtin_bit_cast(unsigned long long, floatx2{x, y}), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ floatx2 get2(const float* p) {
    return __builtin_bit_cast(floatx2, __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ float log2_or(float l, float m) { return m + __builtin_amdgcn_logf(l); }      // v_log_f32 = log2

template <typename T> __device__ __forceinline__ void store4(char* out, size_t i, const floatx4& z) {
    if constexpr (sizeof(T) == 2) {
        const uintx2 p = {f32_to_bf16_bits(z[0]) | (f32_to_bf16_bits(z[1]) << 16), f32_to_bf16_bits(z[2]) | (f32_to_bf16_bits(z[3]) << 16)};
        *reinterpret_cast<uintx2*>(out + i * 2) = p;
    } else {
        *reinterpret_cast<floatx4*>(out + i * 4) = z;
    }
}

// Sum the partial rows of `nq` consecutive queries over the splits of the numerator set, divide by the denominator (of
// the same set, or of the second one), store.  part: row 0 of split 0; consecutive splits are `sstride` floats apart; splits
// ns0 .. ns0 + ns1 - 1 belong to the second set.  Whole workgroup of NTH threads; a thread owns four columns of a query and
// every SR-th split, with a running reference of its own, so that one pass of independent loads is all the latency there is;
// the order of all sums is fixed.
template <typename T, int D, int NTH>
__device__ __forceinline__ void merge_rows(const float* part, size_t sstride, int nq, int ns0, int ns1, char* out, float* lse_out,
                                           size_t row0, float* red /*[NTH * 8]*/) {
    constexpr int P = D + kRowPad, CG = D / 4;
    const int tid = threadIdx.x;
    const int C = nq * CG, SR = C < NTH ? NTH / C : 1;            // splits summed side by side
    for (int c0 = 0; c0 < C; c0 += NTH) {
        const int sg = SR > 1 ? tid / C : 0, c = SR > 1 ? tid - sg * C : c0 + tid;
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        float M = kNeg, L = 0.f, Md = kNeg, Ld = 0.f;
        const int q = c / CG, col = 4 * (c - q * CG);
        const float* row = part + (size_t)q * P;
        if (sg < SR && c < C) {
            // All of a thread's splits are requested before the first is used (device-scope loads are not reordered by the
            // compiler), up to twelve at a time: each is a trip past the caches for the whole wavefront, so batches are of 2, 4, 6 or 12
            // (denominator 4 or 12), the places behind the last split taken by that split again.  The products that are rounded and those
            // that are fused are written out: left to the compiler they differed between the batches.
            auto numerator = [&](auto u_c) {
                constexpr int U = decltype(u_c)::value;
                for (int s = sg; s < ns0; s += U * SR) {
                    floatx2 ml[U], x[U], y[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const float* r = row + (size_t)min(s + u * SR, ns0 - 1) * sstride;
                        ml[u] = get2(r + D); x[u] = get2(r + col); y[u] = get2(r + col + 2);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (s + u * SR >= ns0) break;
                        const float mn = fmaxf(M, ml[u][0]), f0 = fast_exp2(M - mn), f1 = fast_exp2(ml[u][0] - mn);
                        M = mn; L = fmaf(L, f0, ml[u][1] * f1);
                        acc[0] = fmaf(acc[0], f0, x[u][0] * f1); acc[1] = fmaf(acc[1], f0, x[u][1] * f1);
                        acc[2] = fmaf(acc[2], f0, y[u][0] * f1); acc[3] = fmaf(acc[3], f0, y[u][1] * f1);
                    }
                }
            };
            auto denominator = [&](auto u_c) {
                constexpr int U = decltype(u_c)::value;
                for (int s = ns0 + sg; s < ns0 + ns1; s += U * SR) {
                    floatx2 ml[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) ml[u] = get2(row + (size_t)min(s + u * SR, ns0 + ns1 - 1) * sstride + D);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (s + u * SR >= ns0 + ns1) break;
                        const float mn = fmaxf(Md, ml[u][0]);
                        Ld = fmaf(ml[u][1], fast_exp2(ml[u][0] - mn), Ld * fast_exp2(Md - mn));
                        Md = mn;
                    }
                }
            };
            const int per = (ns0 + SR - 1) / SR;                      // splits of a thread
            if (per <= 2) numerator(std::integral_constant<int, 2>{});
            else if (per <= 4) numerator(std::integral_constant<int, 4>{});
            else if (per <= 6) numerator(std::integral_constant<int, 6>{});
            else numerator(std::integral_constant<int, 12>{});
            if (ns1 > 0) {
                if (ns1 <= 4 * SR) denominator(std::integral_constant<int, 4>{});
                else denominator(std::integral_constant<int, 12>{});
            }
        }
        if (SR > 1) {
            float* mine = red + tid * 8;
            *reinterpret_cast<floatx4*>(mine) = acc;
            *reinterpret_cast<floatx4*>(mine + 4) = floatx4{M, L, Md, Ld};
            __syncthreads();
            if (tid >= C) return;
            for (int r = 1; r < SR; ++r) {
                const floatx4 x = *reinterpret_cast<const floatx4*>(red + (r * C + tid) * 8), k = *reinterpret_cast<const floatx4*>(red + (r * C + tid) * 8 + 4);
                const float mn = fmaxf(M, k[0]), f0 = fast_exp2(M - mn), f1 = fast_exp2(k[0] - mn);
                M = mn; L = fmaf(L, f0, k[1] * f1);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] = fmaf(acc[e], f0, x[e] * f1);
                const float dn = fmaxf(Md, k[2]);
                Ld = fmaf(Ld, fast_exp2(Md - dn), k[3] * fast_exp2(k[2] - dn));
                Md = dn;
            }
        }
        if (c < C) {
            float f = L > 0.f ? 1.f / L : 0.f;
            if (ns1 > 0) {
                // a denominator of 0 or NaN (no mass, a broken row) gives infinities, not zeros that look like a result
                f = L > 0.f ? (Ld > 0.f ? fast_exp2(M - Md) / Ld : INFINITY) : 0.f;
                M = Md; L = Ld;
            }
            store4<T>(out, (row0 + q) * D + col, acc * f);
            if (lse_out && col == 0) lse_out[row0 + q] = L > 0.f ? log2_or(L, M) * 0.6931471805599453f : -INFINITY;
        }
    }
}

// One workgroup of W wavefronts: NQT x 16 queries of one sequence against one range of keys; its wavefronts take the
// key groups of the range in turn.  Registers (NQT = 1, bf16, d = 128): 64 for the K and V rows in flight, 16 queries, 32
// sums.  The rows of the next group are requested as soon as the registers of the current one are free (keys after S^T,
// values after O^T), so that about 12 KB per wavefront are under way at any time.
// STREAM: K and V are read past the caches (see attend_streams).
// ONE: a workgroup takes both sets of a sequence as a whole, nothing is merged behind it (see attend_in_one).
template <typename T, int D, int NQT, int W, bool STREAM = false, bool ONE = false>
__global__ __launch_bounds__(W * 64) void attend_kernel(const AttendArgs a) {
    constexpr bool B16 = sizeof(T) == 2;
    constexpr int ROWB = D * (int)sizeof(T);
    constexpr int KEYS = B16 ? 32 : 16;        // keys per step of a wavefront
    constexpr int NT = KEYS / 16;              // key tiles of a step
    constexpr int KC = ROWB / 64;              // 16-byte pieces of a lane's quarter of a row
    constexpr int VR = KEYS / 4;               // value rows (= weights) per lane and step
    constexpr int EPN = D / 16;                // columns per lane of a value row
    constexpr int VD = EPN * (int)sizeof(T) / 4;   // ... in dwords
    constexpr int RQ = 16 * NQT;
    constexpr int P = D + kRowPad;

    // the wavefronts' sums meet here
    __shared__ __align__(16) float lds[W * RQ * P];
    __shared__ int last_flag;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kg = lane >> 4;

    // workgroup -> (sequence, query group, split).  Where several query groups read the same rows, the workgroups of a
    // sequence go to one XCD (blocks are dealt to the eight XCDs in turn, x fastest), whose L2 then serves all but the first
    // read: a row of the grid holds the workgroups of eight sequences, else those of one.
    const unsigned int ns = ONE ? 1u : (unsigned int)(a.ns[0] + a.ns[1]);
    const unsigned int seq_u = a.by_xcd ? blockIdx.y * 8u + (blockIdx.x & 7u) : blockIdx.y;
    const unsigned int rest = a.by_xcd ? blockIdx.x >> 3 : blockIdx.x;
    if (seq_u >= (unsigned int)a.n_seq) return;
    const int qg = (int)(rest % (unsigned int)a.n_qg);
    const int split = (int)(rest / (unsigned int)a.n_qg);
    const int64_t seq = seq_u;
    int which = split >= a.ns[0] ? 1 : 0;
    // ONE: the groups with a live token of each set, dealt out to wavefronts that take one set each (of W as many as their share of the
    // rows; a numerator's group has two)
    __shared__ int order[ONE ? 2 : 1][ONE ? kOneGroups : 1];
    __shared__ int n_live[2];
    int w0_waves = W, mine = 0, stride = 1, listed = 0;
    if constexpr (ONE) {
        constexpr int GPL = 64 / KEYS, U = 8;                 // groups per weight load of a wavefront; loads under way
        __shared__ int live[2][kOneGroups + 64 / KEYS];
        const int chunks0 = (int)((a.set[0].count + 63) / 64), chunks = chunks0 + (int)((a.set[1].count + 63) / 64);
        for (int c0 = wave; c0 < chunks; c0 += W * U) {
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c0 + u * W, k = c >= chunks0 ? 1 : 0;
                const int64_t key = 64ll * (k ? c - chunks0 : c) + lane;
                const AttendSet& Z = a.set[k];
                x[u] = c < chunks && key < Z.count ? Z.w[(size_t)seq * Z.stride + key] : 0.f;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c0 + u * W, k = c >= chunks0 ? 1 : 0;
                const unsigned long long m = __ballot(x[u] > 0.f);
                if (c < chunks && lane < GPL)
                    live[k][(k ? c - chunks0 : c) * GPL + lane] = ((m >> (lane * KEYS)) & ((1ull << KEYS) - 1ull)) != 0ull ? 1 : 0;
            }
        }
        __syncthreads();
        if (wave < 2) {
            const int groups = (int)((a.set[wave].count + KEYS - 1) / KEYS);
            int n_so_far = 0;
            for (int g = lane; g < (groups + 63) / 64 * 64; g += 64) {
                const bool is = g < groups && live[wave][g] != 0;
                const unsigned long long m = __ballot(is);
                if (is) order[wave][n_so_far + (int)__popcll(m & ((1ull << lane) - 1ull))] = g;
                n_so_far += (int)__popcll(m);
            }
            if (lane == 0) n_live[wave] = n_so_far;
        }
        __syncthreads();
        const int l0 = __builtin_amdgcn_readfirstlane(n_live[0]), l1 = __builtin_amdgcn_readfirstlane(n_live[1]);
        const int w1 = l1 == 0 ? 0 : l0 == 0 ? W : min(max((W * l1 + l0) / (2 * l0 + l1), 1), W - 1);
        w0_waves = W - w1;
        which = wave >= w0_waves ? 1 : 0;
        mine = which ? wave - w0_waves : wave; stride = which ? w1 : w0_waves; listed = which ? l1 : l0;
    }
    const AttendSet S = which ? a.set[1] : a.set[0];
    const bool has_v = S.V != nullptr;
    const int64_t groups = (S.count + KEYS - 1) / KEYS, full = S.count / KEYS;
    const int64_t g0 = ONE ? 0 : (int64_t)(split - (which ? a.ns[0] : 0)) * S.groups_per_split;
    const int64_t g1 = ONE ? 0 : min(groups, g0 + S.groups_per_split), gf = min(full, g1);

    const char* Kb = S.K + (size_t)seq * S.stride * ROWB;
    const char* Vb = has_v ? S.V + (size_t)seq * S.stride * ROWB : nullptr;
    const float* wb = S.w + (size_t)seq * S.stride;

    uintx4 kf[NT][KC];
    unsigned int vf[VR][VD];
    float w0[VR], w1[VR];
    const int koff = n * ROWB + kg * 16, vcol = n * (VD < 4 ? VD : 4) * 4, voff = 4 * kg * ROWB + vcol;
    auto load_w = [&](float (&w)[VR], int64_t g) {
        const float* p = wb + g * KEYS + 4 * kg;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const floatx4_u x = *reinterpret_cast<const floatx4_u*>(p + 16 * t);
#pragma unroll
            for (int r = 0; r < 4; ++r) w[4 * t + r] = x[r];
        }
    };
    auto fetch = [](const auto* p) { return STREAM ? __builtin_nontemporal_load(p) : *p; };
    auto load_v_row = [&](int j, const char* p) {
        if constexpr (VD == 2) {
            const uintx2 x = fetch(reinterpret_cast<const uintx2*>(p));
            vf[j][0] = x[0]; vf[j][1] = x[1];
        } else {
#pragma unroll
            for (int c = 0; c < VD / 4; ++c) {
                const uintx4 x = fetch(reinterpret_cast<const uintx4*>(p + 256 * c));
#pragma unroll
                for (int i = 0; i < 4; ++i) vf[j][4 * c + i] = x[i];
            }
        }
    };
    auto load_k = [&](int64_t g) {
        const char* p = Kb + (size_t)g * (KEYS * ROWB) + koff;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int c = 0; c < KC; ++c) kf[t][c] = fetch(reinterpret_cast<const uintx4*>(p + 16 * t * ROWB + 64 * c));
    };
    auto load_v = [&](int64_t g) {
        const char* p = Vb + (size_t)g * (KEYS * ROWB) + voff;
#pragma unroll
        for (int j = 0; j < VR; ++j) load_v_row(j, p + ((j & 3) + 16 * (j >> 2)) * ROWB);
    };

    // the sequence's last group, if it is not full: rows past the end repeat the last row with weight 0
    const int left = (int)(S.count - full * KEYS) - 1;           // its last valid row
    auto load_w_end = [&](float (&w)[VR]) {
#pragma unroll
        for (int j = 0; j < VR; ++j) {
            const int row = 4 * kg + (j & 3) + 16 * (j >> 2);
            const float x = wb[full * KEYS + min(row, left)];
            w[j] = row <= left ? x : 0.f;
        }
    };
    auto load_k_end = [&]() {
        const char* kp = Kb + (size_t)full * (KEYS * ROWB) + kg * 16;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int c = 0; c < KC; ++c) kf[t][c] = *reinterpret_cast<const uintx4*>(kp + min(16 * t + n, left) * ROWB + 64 * c);
    };
    auto load_v_end = [&]() {
#pragma unroll
        for (int j = 0; j < VR; ++j) {
            const int row = 4 * kg + (j & 3) + 16 * (j >> 2);
            load_v_row(j, Vb + (size_t)full * (KEYS * ROWB) + min(row, left) * ROWB + vcol);
        }
    };
    int64_t g = g0 + wave;
    const bool any_full = !ONE && g < gf;
    if (any_full) {
        load_w(w0, g);
        load_k(g);
        if (has_v) load_v(g);
    }
    if constexpr (ONE) {
        if (mine < listed) {
            const int x = __builtin_amdgcn_readfirstlane(order[which][mine]);
            if (x < full) { load_w(w0, x); load_k(x); if (has_v) load_v(x); }
            else { load_w_end(w0); load_k_end(); if (has_v) load_v_end(); }
        }
    }
    // queries: lane (n, kg) holds its quarter of query n of each tile (queries past the end repeat the last one)
    uintx4 qf[NQT][KC];
#pragma unroll
    for (int t = 0; t < NQT; ++t) {
        const int q = min(qg * RQ + 16 * t + n, a.n_q - 1);
        const char* p = a.Q + ((size_t)seq * a.n_q + q) * ROWB + kg * 16;
#pragma unroll
        for (int c = 0; c < KC; ++c) qf[t][c] = *reinterpret_cast<const uintx4*>(p + 64 * c);
    }
    if (any_full && g + W < gf) load_w(w1, g + W);

    float m[NQT], l[NQT];
    floatx4 o[NQT][EPN];
    const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NQT; ++t) {
        m[t] = kNeg; l[t] = 0.f;
#pragma unroll
        for (int e = 0; e < EPN; ++e) o[t][e] = zero4;
    }
    floatx4 s[NQT][NT];
    auto qk = [&]() {
        if constexpr (B16) {
#pragma unroll
            for (int t = 0; t < NQT; ++t)
#pragma unroll
                for (int kt = 0; kt < NT; ++kt) s[t][kt] = zero4;
#pragma unroll
            for (int c = 0; c < KC; ++c)
#pragma unroll
                for (int kt = 0; kt < NT; ++kt)
#pragma unroll
                    for (int t = 0; t < NQT; ++t)
                        s[t][kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kf[kt][c]), __builtin_bit_cast(bf16x8_t, qf[t][c]),
                                                                           s[t][kt], 0, 0, 0);
        } else {
            // Chains of two matrix instructions (eight columns), their results added in a tree: one chain over the row rounds d
            // times at the size of the whole sum, 1.3e-6 off the 64-bit output (d = 128, 8321 tokens), this 5.3e-7.  With 16
            // queries a piece is added while the next one is in the matrix cores; with 32 there are no registers for that.
#pragma unroll
            for (int t = 0; t < NQT; ++t) {
                constexpr int LAG = NQT == 1 ? 1 : 0;
                floatx4 level[4], y[LAG + 1][2];
#pragma unroll
                for (int c = 0; c < KC + LAG; ++c) {
                    if (c < KC) {
                        asm volatile("" : "+v"(qf[t][c < KC ? c : 0]));       // (registers: pieces start one after the other)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int j = 2 * (i & 1) + (i >> 1);
                            const unsigned int ka = kf[0][c < KC ? c : 0][j], qa = qf[t][c < KC ? c : 0][j];
                            y[c & LAG][i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(ka), __uint_as_float(qa), i < 2 ? zero4 : y[c & LAG][i & 1], 0, 0, 0);
                        }
                    }
                    const int p = c - LAG;
                    if (p < 0) continue;
                    floatx4 x = y[p & LAG][0] + y[p & LAG][1];
                    int l = 0;
#pragma unroll
                    for (int k = p; k & 1; k >>= 1) x = level[l++] + x;
                    asm volatile("" : "+v"(x));
                    level[l] = x;
                }
                s[t][0] = level[KC == 8 ? 3 : 2];
            }
        }
    };
    // logits -> weights 2^(logit - m), the difference rounded once (a logit rounded for itself is off by 2^-24 of its size,
    // which is what the weight is off by).  The denominator adds the fp32 weights.  On the bf16 path the values meet them as
    // two bf16 numbers each, the upper bits and what they leave (17 bits; one number each is off by up to 2^-9, and a peaked
    // softmax shows it: 1.96e-3 instead of 1.66e-3 off the 64-bit result over 8321 tokens, where rounding the output makes
    // 1.65e-3; the second product costs 716 -> 718 us with 1024 sequences, 27.8 -> 28.7 with 256 queries).  The second
    // number of a weight that has one is never 0: an infinite value stays infinite.
    // The reference m moves only when a logit passes it by more than kSlack (then to the largest one, for all lanes of the
    // query): the weights are floating-point numbers, so a reference that is 2^6 too small costs nothing.
    bf16x8_t pb[NQT], pl[NQT];
    auto softmax = [&](const float (&w)[VR]) {
        float bias[VR];
        bool dead = false;
#pragma unroll
        for (int x = 0; x < VR; ++x) {
            const bool live = w[x] > 0.f;
            dead |= !live;
            bias[x] = live ? __builtin_amdgcn_logf(w[x]) : 2.f * kNeg;        // below every reference: weight 0
        }
        if (__builtin_amdgcn_ballot_w64(dead) != 0ull) {                      // (whatever an absent token's row holds)
#pragma unroll
            for (int t = 0; t < NQT; ++t)
#pragma unroll
                for (int x = 0; x < VR; ++x) s[t][x >> 2][x & 3] = w[x] > 0.f ? s[t][x >> 2][x & 3] : 0.f;
        }
        bool grew = false;
        float mx[NQT];
#pragma unroll
        for (int t = 0; t < NQT; ++t) {
            mx[t] = 2.f * kNeg;
#pragma unroll
            for (int x = 0; x < VR; ++x) {
                const float lg = fmaf(s[t][x >> 2][x & 3], a.scale_log2, bias[x]);
                mx[t] = fmaxf(mx[t], lg);
            }
            grew |= mx[t] > m[t] + kSlack;
        }
        if (__builtin_amdgcn_ballot_w64(grew) != 0ull) {
#pragma unroll
            for (int t = 0; t < NQT; ++t) {
                float mm = fmaxf(mx[t], __shfl_xor(mx[t], 16));
                mm = fmaxf(mm, __shfl_xor(mm, 32));
                const float mnew = fmaxf(m[t], mm);
                const float sc = fast_exp2(m[t] - mnew);
                m[t] = mnew;
                l[t] *= sc;
#pragma unroll
                for (int e = 0; e < EPN; ++e) o[t][e] *= sc;
            }
        }
#pragma unroll
        for (int t = 0; t < NQT; ++t) {
#pragma unroll
            for (int x = 0; x < VR; ++x) s[t][x >> 2][x & 3] = fast_exp2(fmaf(s[t][x >> 2][x & 3], a.scale_log2, bias[x] - m[t]));
            if constexpr (B16) {
                uintx4 hi, lo;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const floatx2 pf = {s[t][i >> 1][2 * (i & 1)], s[t][i >> 1][2 * (i & 1) + 1]};
                    const unsigned int b0 = __float_as_uint(pf[0]), b1 = __float_as_uint(pf[1]);
                    hi[i] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
                    const floatx2 rest = {fmaf(pf[0], 0x1p-40f, pf[0] - __uint_as_float(b0 & 0xffff0000u)),
                                          fmaf(pf[1], 0x1p-40f, pf[1] - __uint_as_float(b1 & 0xffff0000u))};
                    lo[i] = __builtin_bit_cast(unsigned int, __builtin_convertvector(rest, bf16x2_t));
                    l[t] += pf[0] + pf[1];
                }
                pb[t] = __builtin_bit_cast(bf16x8_t, hi); pl[t] = __builtin_bit_cast(bf16x8_t, lo);
            } else {
#pragma unroll
                for (int x = 0; x < VR; ++x) l[t] += s[t][x >> 2][x & 3];
            }
        }
    };
    auto pv = [&]() {
#pragma unroll
        for (int e = 0; e < EPN; ++e) {
            if constexpr (B16) {
                uintx4 f;
#pragma unroll
                for (int i = 0; i < 4; ++i)       // element e of the rows of keys 2i, 2i + 1 of this lane
                    f[i] = __builtin_amdgcn_perm(vf[2 * i + 1][e >> 1], vf[2 * i][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
                for (int t = 0; t < NQT; ++t) {
                    o[t][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f), pb[t], o[t][e], 0, 0, 0);
                    o[t][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, f), pl[t], o[t][e], 0, 0, 0);
                }
            } else {
#pragma unroll
                for (int t = 0; t < NQT; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        o[t][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(vf[j][e]), s[t][0][j], o[t][e], 0, 0, 0);
            }
        }
    };

    if (any_full) {
        for (;;) {
            // the next group with a live key (places without a token are not read); its weights arrived a step ago
            int64_t gn = g + W;
            bool more = false;
            while (gn < gf) {
                bool live = false;
#pragma unroll
                for (int x = 0; x < VR; ++x) live |= w1[x] > 0.f;
                if (__builtin_amdgcn_ballot_w64(live) != 0ull) { more = true; break; }
                gn += W;
                if (gn < gf) load_w(w1, gn);
            }
            float wc[VR];
#pragma unroll
            for (int x = 0; x < VR; ++x) { wc[x] = w0[x]; w0[x] = w1[x]; }
            if (more && gn + W < gf) load_w(w1, gn + W);
            qk();
            if (more) load_k(gn);
            softmax(wc);
            if (has_v) {
                pv();
                if (more) load_v(gn);
            }
            if (!more) break;
            g = gn;
        }
    }
    if constexpr (ONE) {
        for (int i = mine; i < listed; i += stride) {
            const bool more = i + stride < listed;
            const int x = more ? __builtin_amdgcn_readfirstlane(order[which][i + stride]) : 0;
            float wc[VR];
#pragma unroll
            for (int y = 0; y < VR; ++y) wc[y] = w0[y];
            if (more) { if (x < full) load_w(w0, x); else load_w_end(w0); }
            qk();
            if (more) { if (x < full) load_k(x); else load_k_end(); }
            softmax(wc);
            if (has_v) {
                pv();
                if (more) { if (x < full) load_v(x); else load_v_end(); }
            }
        }
    }
    // (the last group: one wavefront)
    if (!ONE && g1 > full && (int)((full - g0) % W) == wave) {
        float wt[VR];
        load_k_end();
        load_w_end(wt);
        if (has_v) load_v_end();
        qk();
        softmax(wt);
        if (has_v) pv();
    }
#pragma unroll
    for (int t = 0; t < NQT; ++t) {
        l[t] += __shfl_xor(l[t], 16);
        l[t] += __shfl_xor(l[t], 32);
    }

    // ---- the wavefronts meet in LDS; a thread then owns four columns of a query
    const int q0 = qg * RQ, nqv = min(RQ, a.n_q - q0);
#pragma unroll
    for (int t = 0; t < NQT; ++t)
        if (16 * t + n < nqv) {
            float* row = lds + (wave * RQ + 16 * t + n) * P;
            if (has_v) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int e = 0; e < EPN; e += 4) {
                        const floatx4 x = {o[t][e][r], o[t][e + 1][r], o[t][e + 2][r], o[t][e + 3][r]};
                        *reinterpret_cast<floatx4*>(row + (VD > 4 ? 16 * e + 4 * (4 * kg + r) : EPN * (4 * kg + r) + e)) = x;
                    }
            }
            if (kg == 0) *reinterpret_cast<floatx2*>(row + D) = floatx2{m[t], l[t]};
        }
    __syncthreads();
    const size_t row0 = (size_t)seq * a.n_q + q0;
    // partial rows: [sequence][query group][split][row], a.rows rows of P floats each
    const size_t grp = (size_t)seq * a.n_qg + qg, sstride = (size_t)a.rows * P;
    float* part = a.partial + grp * ns * sstride;
    for (int c = tid; c < nqv * (D / 4); c += W * 64) {
        const int q = c / (D / 4), col = 4 * (c - q * (D / 4));
        const float* row = lds + q * P;
        if constexpr (ONE) {
            float M = kNeg, L = 0.f, Md = kNeg, Ld = 0.f;
            for (int w = 0; w < W; ++w) {
                const float x = row[w * RQ * P + D];
                if (w < w0_waves) M = fmaxf(M, x); else Md = fmaxf(Md, x);
            }
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
            for (int w = 0; w < W; ++w) {
                const floatx2 x = *reinterpret_cast<const floatx2*>(row + w * RQ * P + D);
                if (w < w0_waves) {
                    const float f = fast_exp2(x[0] - M);
                    L = fmaf(x[1], f, L);
                    acc += *reinterpret_cast<const floatx4*>(row + w * RQ * P + col) * f;
                } else Ld = fmaf(x[1], fast_exp2(x[0] - Md), Ld);
            }
            // (as in merge_rows: a denominator of 0 or NaN shows)
            const float f = L > 0.f ? (Ld > 0.f ? fast_exp2(M - Md) / Ld : INFINITY) : 0.f;
            store4<T>(a.out, (row0 + q) * D + col, acc * f);
            if (col == 0 && a.lse_out) a.lse_out[row0 + q] = Ld > 0.f ? log2_or(Ld, Md) * 0.6931471805599453f : -INFINITY;
            continue;
        }
        floatx2 ml[W];
        float M = kNeg, L = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) { ml[w] = *reinterpret_cast<const floatx2*>(row + w * RQ * P + D); M = fmaxf(M, ml[w][0]); }
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float f = fast_exp2(ml[w][0] - M);
            L = fmaf(ml[w][1], f, L);
            if (has_v) acc += *reinterpret_cast<const floatx4*>(row + w * RQ * P + col) * f;
        }
        if (ns == 1) {                          // the whole range was one split: normalise and store
            store4<T>(a.out, (row0 + q) * D + col, acc * (L > 0.f ? 1.f / L : 0.f));
            if (col == 0 && a.lse_out) a.lse_out[row0 + q] = L > 0.f ? log2_or(L, M) * 0.6931471805599453f : -INFINITY;
        } else {
            float* dst = part + split * sstride + q * P;
            if (has_v) { put2(dst + col, acc[0], acc[1]); put2(dst + col + 2, acc[2], acc[3]); }
            if (col == 0) put2(dst + D, M, L);
        }
    }
    if (ONE || ns == 1 || !a.fused) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // this wavefront's share of the partial has reached memory ...
    __syncthreads();                                            // ... and so has everybody else's
    if (wave == 0) {
        const bool last = all_arrived(a.arrivals + grp * ns, (unsigned int)split, ns, a.label);
        if (lane == 0) last_flag = last ? 1 : 0;
    }
    __syncthreads();
    if (!last_flag) return;
    merge_rows<T, D, W * 64>(part, sstride, nqv, a.ns[0], a.ns[1], a.out, a.lse_out, row0, lds);
}

// Partials of many splits per query: one workgroup per (sequence, query) merges them (spread over the chip, where the last
// workgroup of a group would have to read them all by itself).
constexpr int kMergeThreads = 256;
template <typename T, int D>
__global__ __launch_bounds__(kMergeThreads) void attend_merge_kernel(const AttendArgs a, int rq) {
    __shared__ __align__(16) float red[kMergeThreads * 8];
    const int64_t seq = blockIdx.y;
    const int q = blockIdx.x, qg = q / rq, ns = a.ns[0] + a.ns[1];
    const size_t sstride = (size_t)a.rows * (D + kRowPad);
    const float* part = a.partial + ((size_t)seq * a.n_qg + qg) * ns * sstride + (size_t)(q - qg * rq) * (D + kRowPad);
    merge_rows<T, D, kMergeThreads>(part, sstride, 1, a.ns[0], a.ns[1], a.out, a.lse_out, (size_t)seq * a.n_q + q, red);
}

// ---------------------------------------------------------------------------------------------------------------------
struct AttendPlan {
    int nqt, waves, n_qg, rows;   // query tiles and wavefronts per workgroup, query groups, rows of a partial
    int ns[2], gps[2];            // splits and key groups per split of each set
    bool fused;                   // the last workgroup of a query group merges (never in a captured launch)
    size_t arrive_bytes, partial_bytes;
};

// Splits: eight wavefronts per compute unit, each at least one key group (twice as many: the merge takes longer than the
// pass gains, 27.8 against 23.3 us with 256 queries, decode of 64 sequences 3 % slower); the steps of a wavefront decide a
// workgroup's time, so the ranges are cut into equal numbers of steps.
static AttendPlan attend_plan(int d, int elem, int64_t n_seq, int64_t count0, int64_t count1, int n_q, size_t max_bytes) {
    AttendPlan p;
    const int keys = elem == 2 ? 32 : 16;
    p.nqt = n_q > 16 ? 2 : 1;
    const int rq = 16 * p.nqt;
    p.n_qg = (n_q + rq - 1) / rq;
    p.rows = n_q < rq ? n_q : rq;
    const int64_t wgs = n_seq * p.n_qg;
    const int64_t cnt[2] = {count0, count1};
    const int64_t all = (count0 + keys - 1) / keys + (count1 + keys - 1) / keys;
    // bf16: four wavefronts per workgroup let three workgroups share a compute unit (registers); eight mean half the splits
    // where a wavefront has a single group anyway.  fp32: eight, four take more registers and fewer of them are resident
    // (1024 x 2000 tokens, d = 64: 184 us against 196; 256 x 1000, d = 128: 43 against 47; one sequence of 65536, d = 64: 16.7
    // against 15.9).  32 queries take eight (one workgroup per compute unit, LDS).
    // (Eight also where workgroups of eight fill the compute units once, 64 sequences x 4100 tokens 24.5 us for 25.1, 256 x 1000 21.6 for 24.2, would cut
    // the ranges, and with them the order of the sums and the last bits of a decode, by how much of the chip a batch happens to fill.)
    p.waves = elem == 2 && p.nqt == 1 && all * wgs > kTargetWaves ? 4 : 8;
    const size_t row_bytes = (size_t)p.rows * (d + kRowPad) * sizeof(float);
    int64_t most = (int64_t)(max_bytes / ((size_t)wgs * row_bytes));          // splits whose partials fit the buffer
    int64_t steps = (all * wgs + kTargetWaves - 1) / kTargetWaves;             // per wavefront
    if (steps < 1) steps = 1;
    for (int k = 0; k < 2; ++k) {
        const int64_t groups = (cnt[k] + keys - 1) / keys;
        int64_t ns = (groups + steps * p.waves - 1) / (steps * p.waves);
        const int64_t lim = k == 0 ? (count1 > 0 ? (most + 1) / 2 : most) : most / 2;
        if (ns > lim) ns = lim;
        if (ns < 1 && groups > 0) ns = 1;
        const int64_t gps = ns > 0 ? (groups + ns - 1) / ns : 1;
        p.ns[k] = groups > 0 ? (int)((groups + gps - 1) / gps) : 0;
        p.gps[k] = (int)gps;
    }
    const int ns = p.ns[0] + p.ns[1];
    p.partial_bytes = ns > 1 ? (size_t)wgs * ns * row_bytes : 0;
    p.arrive_bytes = ns > 1 ? ((size_t)wgs * ns * 8 + 255) / 256 * 256 : 0;
    // one workgroup reads ns * rows partial rows at the end: up to 128 KB of them that is faster than one more launch (by
    // 2 us with 18 splits of 4 rows, equal with 4 splits of 32)
    p.fused = ns > 1 && (size_t)ns * row_bytes <= (size_t)128 * 1024;
    return p;
}

// Upper bounds for any token count.  One set is cut into at most S = ceil(kTargetWaves / (wavefronts per workgroup * wgs))
// splits, two sets together into at most S + 1 (each rounds up once); one split in all needs no memory.
size_t attend_workspace_bytes(int d, int64_t n_seq, int n_q, int sets) {
    const int rq = n_q > 16 ? 32 : 16;
    const int64_t wgs = n_seq * ((n_q + rq - 1) / rq);
    const int64_t wg_target = kTargetWaves / (n_q > 16 ? 8 : 4);
    int64_t splits = wgs > 0 ? (wg_target + wgs - 1) / wgs + sets - 1 : 0;
    if (splits == 1) splits = 0;
    const size_t row_bytes = (size_t)(n_q < rq ? n_q : rq) * (d + kRowPad) * sizeof(float);
    return (size_t)(wgs * splits) * (row_bytes + 8) + 512;
}

size_t attend_scratch_bytes(int dtype, int d, int64_t n_seq, int64_t count, int n_q, size_t max_bytes) {
    if (n_seq <= 0 || n_q <= 0) return 0;
    const AttendPlan p = attend_plan(d, dtype == BKV_BF16 ? 2 : 4, n_seq, count, 0, n_q, max_bytes);
    return p.partial_bytes + p.arrive_bytes;
}

// Rows that are read once (up to 16 queries: one query group) and are more than the 256 MB that the cache in front of the memory
// holds come back from memory the next time whatever is done, and keeping them costs.  Past the caches (4 queries, d = 128): bf16 1024 x 8321
// tokens 707 -> 649 us (on another box 711 -> 631), 1024 x 1000 (0.5 GB) 90.0 -> 81.5; fp32 256 x 8321 366 -> 340, 1024 x 1000 183 -> 175.  Below that they may still be
// there (bf16 256 x 2000 tokens, 0.26 GB: 42.4 us when they are, 46.3 past the caches), so the line lies a little above what the cache holds.
static bool attend_streams(int row_bytes, const AttendArgs& a) {
    const int64_t rows = a.n_seq * (2 * a.set[0].count + a.set[1].count);
    return rows * row_bytes > ((int64_t)320 << 20);
}

// Two sets in one workgroup per sequence: sets whose places are mostly empty, of which the caller has an estimate of how many tokens they hold
// (AttendArgs::live: a stream's), on a chip that is not full.  Splits, hand-over and merge cost about 4 us, more than such a workgroup's
// few steps (8 regions x 256 places, bf16, d = 128, over 288 tokens, append and attend: 32 streams 18.2 -> 16.6 us a token, 200 over 200
// tokens 35 -> 17.8).  The line, in halves of a group of keys, a numerator's two and a denominator's one, over eight wavefronts; one
// workgroup a compute unit.  From a quarter of the compute units on the splits have no others to go to: four groups a wavefront.  For
// fewer sequences the splits take steps at the same time that one workgroup takes one after the other.  One workgroup / splits, 4 queries, halving once,
// us (halves of a group): bf16, d = 128, 8 x 256 places, 1 stream 8.1 / 9.2 (36), 9.1 / 9.2 (46), 11.4 / 9.2 (62), 8 streams 8.8 / 9.4 (36), 9.9 / 9.4 (46),
// 6 x 128 places 7.9 / 8.4 (32), 8.7 / 8.5 (37), 128 streams 8.7 / 18.2 (36), 13.3 / 19.1 (62); d = 64 7.5 / 8.0 (36), 8.9 / 8.1 (52); fp32, d = 128, 8 x 256, 1 stream
// 9.0 / 10.5 (26), 11.5 / 10.6 (36), 13.0 / 10.6 (56), 128 streams 15.0 / 26.0 (56); d = 64 7.3 / 8.3 (26), 8.7 / 8.5 (36).
static bool attend_in_one(const AttendArgs& a, const AttendPlan& p, int keys) {
    const int64_t g0 = (a.set[0].count + keys - 1) / keys, g1 = (a.set[1].count + keys - 1) / keys;
    if (p.nqt != 1 || a.set[0].count <= 0 || a.set[1].count <= 0 || !a.set[0].V || a.live <= 0 || g0 > kOneGroups || g1 > kOneGroups) return false;
    const int64_t live0 = min(g0, a.live), n_cu = compute_units();
    const int64_t most = 4 * a.n_seq >= n_cu ? 64 : keys == 32 ? 36 : 30;
    return a.n_seq <= n_cu && 2 * live0 + g1 <= most;
}

template <typename T, int D>
static hipError_t launch_attend_t(const AttendArgs& a, const AttendPlan& p, hipStream_t st) {
    // (two dimensions: a grid may not exceed 2^32 threads in one of them)
    const unsigned int inner = (unsigned int)p.n_qg * (unsigned int)(p.ns[0] + p.ns[1]);
    const dim3 grid = a.by_xcd ? dim3(8u * inner, (unsigned)((a.n_seq + 7) / 8)) : dim3(inner, (unsigned)a.n_seq);
    const int64_t units = a.n_seq * (a.set[0].count + a.set[1].count);
    hipError_t e = hipSuccess;
    if (attend_in_one(a, p, sizeof(T) == 2 ? 32 : 16)) {
        AttendArgs one = a;
        one.n_qg = 1; one.by_xcd = 0; one.ns[0] = 1; one.ns[1] = 0;
        return launch_timed(kProfAttend, units, attend_kernel<T, D, 1, 8, false, true>, dim3(1, (unsigned)a.n_seq), dim3(512), 0, st, one);
    }
    if (p.nqt == 2) e = launch_timed(kProfAttend, units, attend_kernel<T, D, 2, 8>, grid, dim3(512), 0, st, a);
    else if (attend_streams(D * (int)sizeof(T), a)) {
        if (p.waves == 8) e = launch_timed(kProfAttend, units, attend_kernel<T, D, 1, 8, true>, grid, dim3(512), 0, st, a);
        else if constexpr (sizeof(T) == 2) e = launch_timed(kProfAttend, units, attend_kernel<T, D, 1, 4, true>, grid, dim3(256), 0, st, a);
    } else if (p.waves == 8) e = launch_timed(kProfAttend, units, attend_kernel<T, D, 1, 8>, grid, dim3(512), 0, st, a);
    else if constexpr (sizeof(T) == 2) e = launch_timed(kProfAttend, units, attend_kernel<T, D, 1, 4>, grid, dim3(256), 0, st, a);
    if (e != hipSuccess || p.ns[0] + p.ns[1] == 1 || p.fused) return e;
    return launch_timed(kProfAttendMerge, a.n_seq * a.n_q, attend_merge_kernel<T, D>, dim3(a.n_q, (unsigned)a.n_seq), dim3(kMergeThreads), 0, st,
                        a, 16 * p.nqt);
}

// Scratch of the entry point that allocates nothing: the split partials live in this array instead of a caller's
// workspace.  Every GPU holds its own copy at its own address; host code uses the address that
// hipGetSymbolAddress returns for the current device, never the array's name.
static __device__ __align__(256) unsigned char scratch[kAttendStaticScratchBytes];
namespace {
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];           // per device, filled at the first call on that device
}
hipError_t attend_static_scratch(void** ptr) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

// A number that no other launch of this process has (mix64 is one to one), and other processes' launches next to never: memory
// that another one has left must not look arrived.
static unsigned long long launch_count() {
    static const unsigned long long first = mix64((unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count()) ^
                                            mix64((unsigned long long)getpid());
    static std::atomic<unsigned long long> launches{0};
    return first + launches.fetch_add(1, std::memory_order_relaxed);
}
static unsigned long long launch_number() { return mix64(launch_count()); }
// The same in 51 bits, for launches that keep theirs in words with something else: the count itself.
unsigned long long status_label() { return launch_count() & ((1ull << 51) - 1); }

hipError_t launch_attend(int dtype, int d, AttendArgs& a, void* workspace, size_t ws_bytes, size_t max_bytes, hipStream_t st) {
    if (a.n_seq <= 0 || a.n_q <= 0) return hipSuccess;
    if (a.n_seq > 65535) return hipErrorInvalidValue;
    AttendPlan p = attend_plan(d, dtype == BKV_BF16 ? 2 : 4, a.n_seq, a.set[0].count, a.set[1].count, a.n_q, max_bytes);
    if (p.ns[0] + p.ns[1] < 1 || p.partial_bytes + p.arrive_bytes > ws_bytes) return hipErrorInvalidValue;
    a.n_qg = p.n_qg; a.rows = p.rows;
    for (int k = 0; k < 2; ++k) { a.ns[k] = p.ns[k]; a.set[k].groups_per_split = p.gps[k]; }
    if (p.fused) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &capture) != hipSuccess) {
            (void)hipGetLastError();              // (a launch says for itself what is wrong with the stream)
            p.fused = false;
        } else if (capture != hipStreamCaptureStatusNone) p.fused = false;
    }
    a.fused = p.fused;
    a.by_xcd = p.n_qg > 1 && a.n_seq >= 8;
    a.arrivals = (unsigned long long*)workspace;
    a.partial = (float*)((char*)workspace + p.arrive_bytes);
    a.label = launch_number();
    if (dtype == BKV_BF16 && d == 128) return launch_attend_t<__bf16, 128>(a, p, st);
    if (dtype == BKV_BF16 && d == 64) return launch_attend_t<__bf16, 64>(a, p, st);
    if (dtype == BKV_F32 && d == 128) return launch_attend_t<float, 128>(a, p, st);
    if (dtype == BKV_F32 && d == 64) return launch_attend_t<float, 64>(a, p, st);
    return hipErrorInvalidValue;
}

}  // namespace bkv
