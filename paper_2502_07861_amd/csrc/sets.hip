// Alg. 1 of arXiv 2502.07861 around the halving kernel: the stream of one sequence is split into buckets by the
// norm of the value rows (line 5), every bucket is a MergeAndReduce instance of its own with the value factor and
// value radius 2^i (MR-Numerator_i), negligible buckets are erased (line 8); the keys alone form one more instance
// (MR-Denominator).  Offline form: all tokens are there, so each instance is brought to the state Alg. 3 would have
// reached after its last token -- full blocks halved level by level, at most one half block left over per level, a
// tail of fewer than `block` tokens at level 0.
//
// A "segment" is the set of tokens of one (sequence, slot); slot 0 is the denominator instance, slot 256 + i is
// bucket i, slot 511 collects the rows that take no part (zero or non-finite norm, erased buckets).  Tokens are
// brought into slot order by a stable partition; the segment that starts at position `start` of that order occupies
// positions from start >> l of the level-l buffers (lengths shrink at least as fast as the starts, so segments never
// overlap).  Every round is ONE launch of the halving kernel over a table of instances (InstDesc).
#include "bkv_device.h"
#include "bkv_host.h"
#include "stream_route.h"

namespace bkv {

namespace {

// The tokens of a sequence are counted and partitioned in chunks, one workgroup each: 256 tokens, more where that would make
// more than 128 chunks (a workgroup of the partition reads the counts of all of them).
constexpr int kChunkTokens = 256, kMaxChunks = 128;
struct Chunks { int64_t tokens; int32_t n; };
inline Chunks chunks_of(int64_t n) {
    Chunks c;
    c.tokens = ((n + kMaxChunks - 1) / kMaxChunks + kChunkTokens - 1) / kChunkTokens * kChunkTokens;
    if (c.tokens < kChunkTokens) c.tokens = kChunkTokens;
    c.n = n > 0 ? (int32_t)((n + c.tokens - 1) / c.tokens) : 1;
    return c;
}

// Without the erase rule: slot of every token straight from its value row, and the chunk's counts per slot (blockIdx = chunk,
// sequence); the status words of the sequence are cleared on the way.  With it (ERASE) the slots need the largest norm of the
// sequence first: only |v|^2 (fp32 accumulation) and that maximum here, the slots in slot_kernel.
template <typename T, int D, bool ERASE>
__global__ __launch_bounds__(256) void value_slot_kernel(const char* V, int64_t n, int64_t chunk, float* norm2, unsigned int* vmax2_bits,
                                                         int32_t* slot, int32_t* chunk_cnt, int32_t* status, int32_t status_words) {
    constexpr int RB = D * (int)sizeof(T);
    constexpr int SL = RB / 16;
    constexpr int RP = 256 / SL, U = 8;           // rows per pass of the workgroup, passes in flight
    __shared__ int hist[ERASE ? 1 : kSlots];
    const int sl = threadIdx.x % SL, rg = threadIdx.x / SL;
    const int64_t seq = blockIdx.y, t0 = (int64_t)blockIdx.x * chunk, t1 = min(n, t0 + chunk);
    if (status && blockIdx.x == 0 && (int)threadIdx.x < status_words) status[seq * status_words + threadIdx.x] = 0;
    if constexpr (!ERASE) {
        for (int s = threadIdx.x; s < kSlots; s += 256) hist[s] = 0;
        __syncthreads();
    }
    float best = 0.f;
    for (int64_t r0 = t0 + rg; r0 < t1; r0 += RP * U) {
        uintx4 raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {             // (rows past the end repeat the last one)
            const int64_t row = min(r0 + u * RP, t1 - 1);
            raw[u] = *reinterpret_cast<const uintx4*>(V + (size_t)(seq * n + row) * RB + sl * 16);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t row = r0 + u * RP;
            const float x = group_sum<SL>(Elem<T>::dot(raw[u], raw[u]));
            if (row >= t1) continue;
            if constexpr (ERASE) {
                if (sl == 0) norm2[seq * n + row] = x;
                if (x < __builtin_inff()) best = fmaxf(best, x);
            } else if (sl == 0) {
                int i;
                const int s = bucket_of(x, i) ? kNumSlot0 + i : kDropSlot;
                slot[seq * n + row] = s;
                atomicAdd(&hist[s], 1);
            }
        }
    }
    if constexpr (ERASE) {
        __shared__ float wbest[4];
        best = wave_max(best);
        if ((threadIdx.x & 63) == 0) wbest[threadIdx.x >> 6] = best;
        __syncthreads();
        if (threadIdx.x == 0) {
            best = fmaxf(fmaxf(wbest[0], wbest[1]), fmaxf(wbest[2], wbest[3]));
            if (best > 0.f) atomicMax(vmax2_bits + seq, __float_as_uint(best));   // order of positive floats = order of their bits
        }
    } else {
        __syncthreads();
        for (int s = threadIdx.x; s < kSlots; s += 256) chunk_cnt[(seq * gridDim.x + blockIdx.x) * kSlots + s] = hist[s];
    }
}

// Slot of every token under the erase rule (line 8): a bucket is erased when 4^i <= erase2 * max |v|^2.
__global__ __launch_bounds__(256) void slot_kernel(const float* norm2, const unsigned int* vmax2_bits, int64_t n, int64_t chunk, float erase2,
                                                   int32_t* slot, int32_t* chunk_cnt) {
    __shared__ int hist[kSlots];
    const int64_t seq = blockIdx.y, t0 = (int64_t)blockIdx.x * chunk, t1 = min(n, t0 + chunk);
    for (int s = threadIdx.x; s < kSlots; s += 256) hist[s] = 0;
    __syncthreads();
    const float limit = erase2 * __uint_as_float(vmax2_bits[seq]);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += 256) {
        int s = kDropSlot;
        const float x = norm2[seq * n + t];
        int i;
        if (bucket_of(x, i)) s = (ldexpf(1.f, 2 * i) <= limit) ? kDropSlot : kNumSlot0 + i;
        slot[seq * n + t] = s;
        atomicAdd(&hist[s], 1);
    }
    __syncthreads();
    for (int s = threadIdx.x; s < kSlots; s += 256) chunk_cnt[(seq * gridDim.x + blockIdx.x) * kSlots + s] = hist[s];
}

// exclusive prefix sum over the 64 lanes of a wavefront
__device__ __forceinline__ int wave_exclusive_sum(int x, int lane) {
    int incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    return incl - x;
}

// The non-empty segments of a sequence (the slot that takes no part left out), ascending slot, as a list in LDS.
// Called by one wavefront; returns the length of the list.
__device__ __forceinline__ int list_segments(const int32_t* cnt, const int32_t* start, int64_t seq, int lane, int* lcnt, int* lstart) {
    int c[8], st[8], ne = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int s = lane * 8 + k;
        c[k] = s == kDropSlot ? 0 : cnt[seq * kSlots + s];
        st[k] = start[seq * kSlots + s];
        ne += c[k] > 0;
    }
    int at = wave_exclusive_sum(ne, lane);
    const int total = __shfl(at + ne, 63);
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (c[k] > 0) { lcnt[at] = c[k]; lstart[at] = st[k]; ++at; }
    __builtin_amdgcn_s_waitcnt(0xc07f);          // lgkmcnt(0): the list is in LDS before the wavefront reads it
    __builtin_amdgcn_wave_barrier();
    return total;
}

struct SegGeo {
    int64_t n;            // tokens per sequence
    int32_t b, T;
    int64_t seq_base;
    InstDesc* desc;       // instance tables, round after round: [n_seq, (n / b) >> r] each
    int64_t n_seq;
};

// One entry of the table of round r: block j of the segment of `slot` that starts at `start` (level-r buffer, survivors to
// the level-(r+1) buffer).
__device__ __forceinline__ InstDesc make_desc(const SegGeo& g, int64_t seq, int slot, int start, int r, int j) {
    InstDesc d;
    d.in_tok = seq * (g.n >> r) + (start >> r) + (int64_t)j * g.b;
    d.out_tok = seq * (g.n >> (r + 1)) + (start >> (r + 1)) + (int64_t)j * (g.b / 2);
    d.stream = 64ull * ((uint64_t)(g.seq_base + seq) * kSlots + (uint64_t)slot) + (uint64_t)r;
    d.ctr0 = (uint64_t)j * (uint64_t)g.b;
    d.seq = (int32_t)seq; d.valid = 1; d.rvalue2 = slot >= kNumSlot0 ? ldexpf(1.f, 2 * (slot - kNumSlot0)) : 0.f; d.region = 0;
    return d;
}

// Counts per chunk and slot -> those of the chunks before (in place), and the sequence's counts.  Workgroups of one wavefront, 64
// slots of a sequence each.
__global__ __launch_bounds__(64) void chunk_prefix_kernel(int32_t* chunk_cnt, int chunks, int32_t* cnt) {
    constexpr int U = 32;
    const int64_t seq = blockIdx.y;
    const int slot = (int)blockIdx.x * 64 + (int)threadIdx.x;
    int32_t* c = chunk_cnt + seq * chunks * kSlots + slot;
    int run = 0;
    for (int k0 = 0; k0 < chunks; k0 += U) {
        int x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = k0 + u < chunks ? c[(int64_t)(k0 + u) * kSlots] : 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k0 + u < chunks) { c[(int64_t)(k0 + u) * kSlots] = run; run += x[u]; }
    }
    cnt[seq * kSlots + slot] = run;
}

// The numerator's instances, from the counts per chunk and slot, in one launch.  Workgroups (seq, chunk): stable partition of the
// chunk's tokens, perm[seq][start[slot] + rank among the slot's tokens] = token; a token's place is its slot's start + the
// counts of the chunks before + the wavefronts before its own + its rank in its wavefront.  Workgroups (seq, chunks + r):
// instance table of round r, for every segment its (full blocks >> r) blocks; unused entries of the grid are marked.  Every
// workgroup sums the counts of all chunks for itself, 2 KB each from L2 (what it saves is a launch: 8 sequences x 8192 tokens, two
// rounds, starts, tables and partition 29 us in four launches, one workgroup per sequence, 7 us in one).  That is quadratic in the
// chunks: 32 MB a sequence from 32768 tokens on.  So from kPrefixFrom sums on chunk_prefix_kernel forms them once (SUMMED).
// Whole numerator call with / without it: 4 x 32768 tokens 132 / 129 us, 64 x 8192 456 / 455, 16 x 32768 453 / 459, 64 x 32768
// 1634 / 1678, 256 x 32768 6400 / 7440 (66e3, 70e3, 266e3, 1.06e6, 4.3e6 sums).
constexpr int64_t kPrefixFrom = 160 * 1024;
constexpr int kPartThreads = 512, kPartWaves = kPartThreads / 64, kPartIds = 128;   // at most 123 slots are ever in use
static_assert(kPartThreads == kSlots, "a thread per slot");
template <bool SUMMED>
__global__ __launch_bounds__(kPartThreads) void segments_kernel(const int32_t* slot, const int32_t* chunk_cnt, int chunks, int64_t chunk,
                                                                SegGeo g, int32_t* cnt, int32_t* start, int32_t* perm) {
    __shared__ int cid[kSlots];                   // slot -> dense id of the non-empty slots
    __shared__ int cbase[kPartIds];               // next free position of every dense id
    __shared__ int wcnt[kPartWaves][kPartIds];
    __shared__ int wtot[3][kPartWaves];
    __shared__ int lslot[kPartIds], lstart[kPartIds], lnb[kPartIds], lbase[kPartIds];
    const int64_t seq = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int part = (int)blockIdx.y, r = part - chunks;
    const unsigned long long lt = (1ull << lane) - 1ull;
    for (int i = tid; i < kPartWaves * kPartIds; i += kPartThreads) (&wcnt[0][0])[i] = 0;
    // thread = slot: its tokens, those of the chunks before this one, where its segment starts, its number among the occupied
    int total = 0, before = 0;
    if constexpr (SUMMED) {
        total = cnt[seq * kSlots + tid];
        if (part < chunks) before = chunk_cnt[(seq * chunks + part) * kSlots + tid];
    } else {
        const int32_t* c = chunk_cnt + seq * chunks * kSlots + tid;
#pragma unroll 8
        for (int k = 0; k < chunks; ++k) {
            const int x = c[(int64_t)k * kSlots];
            total += x;
            before += k < part ? x : 0;
        }
    }
    const unsigned long long present = __ballot(total > 0);
    const int nb = r >= 0 && tid != kDropSlot ? (total / g.b) >> r : 0;
    int at = wave_exclusive_sum(total, lane), bat = wave_exclusive_sum(nb, lane);
    if (lane == 63) { wtot[0][wave] = at + total; wtot[1][wave] = (int)__popcll(present); wtot[2][wave] = bat + nb; }
    __syncthreads();
    int id = (int)__popcll(present & lt), n_ids = 0, n_desc = 0;
    for (int w = 0; w < kPartWaves; ++w) {
        if (w < wave) { at += wtot[0][w]; id += wtot[1][w]; bat += wtot[2][w]; }
        n_ids += wtot[1][w]; n_desc += wtot[2][w];
    }
    if (n_ids > kPartIds) n_ids = kPartIds;
    if (part == 0) {
        if (!SUMMED) cnt[seq * kSlots + tid] = total;
        start[seq * kSlots + tid] = at;
    }
    if (r >= 0) {
        if (total > 0 && id < kPartIds) { lslot[id] = tid; lstart[id] = at; lnb[id] = nb; lbase[id] = bat; }
        __syncthreads();
        const int64_t max_inst = (g.n / g.b) >> r;
        InstDesc* desc = g.desc;
        for (int q = 0; q < r; ++q) desc += g.n_seq * ((g.n / g.b) >> q);
        desc += seq * max_inst;
        for (int e = 0; e < n_ids; ++e)
            for (int j = tid; j < lnb[e]; j += kPartThreads)
                if (lbase[e] + j < max_inst) desc[lbase[e] + j] = make_desc(g, seq, lslot[e], lstart[e], r, j);
        InstDesc none;
        none.in_tok = none.out_tok = 0; none.stream = none.ctr0 = 0; none.seq = 0; none.valid = 0; none.rvalue2 = 0.f; none.region = 0;
        for (int64_t j = n_desc + tid; j < max_inst; j += kPartThreads) desc[j] = none;
        return;
    }
    cid[tid] = total > 0 ? id : -1;
    if (total > 0 && id < kPartIds) cbase[id] = at + before;
    __syncthreads();
    const int64_t t0 = (int64_t)part * chunk, t1 = min(g.n, t0 + chunk);
    for (int64_t c0 = t0; c0 < t1; c0 += kPartThreads) {
        const int64_t t = c0 + tid;
        int c = -1;
        if (t < t1) c = cid[slot[seq * g.n + t]];
        const bool live = c >= 0 && c < kPartIds;
        int rank = 0;
        unsigned long long rem = __ballot(live);
        while (rem) {
            const int leader = __ffsll((long long)rem) - 1;
            const int lc = __shfl(c, leader);
            const unsigned long long same = __ballot(live && c == lc);
            if (live && c == lc) rank = (int)__popcll(same & lt);
            if (lane == leader) wcnt[wave][lc] = (int)__popcll(same);
            rem &= ~same;
        }
        __syncthreads();
        if (live) {
            int ahead = 0;
            for (int w = 0; w < wave; ++w) ahead += wcnt[w][c];
            perm[seq * g.n + cbase[c] + ahead + rank] = (int32_t)t;
        }
        if (c0 + kPartThreads >= t1) break;
        __syncthreads();
        if (tid < kPartIds) {
            int tot = 0;
            for (int w = 0; w < kPartWaves; ++w) { tot += wcnt[w][tid]; wcnt[w][tid] = 0; }
            cbase[tid] += tot;
        }
        __syncthreads();
    }
}

// The denominator's one instance per sequence (slot 0, all n tokens in their order): counts, starts, the instance tables of all
// rounds, the slots when they are asked for, and cleared status words.
__global__ __launch_bounds__(256) void single_segment_kernel(SegGeo g, int32_t* cnt, int32_t* start, int32_t* slot, int32_t* status,
                                                             int32_t status_words) {
    const int64_t seq = blockIdx.y, t0 = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
    for (int64_t s = t0; s < kSlots; s += step) {
        cnt[seq * kSlots + s] = s == kDenSlot ? (int32_t)g.n : 0;
        start[seq * kSlots + s] = s == kDenSlot ? 0 : (int32_t)g.n;
    }
    if (status && t0 < status_words) status[seq * status_words + t0] = 0;
    if (slot) for (int64_t t = t0; t < g.n; t += step) slot[seq * g.n + t] = kDenSlot;
    InstDesc* desc = g.desc;
    for (int r = 0; r < g.T; ++r) {
        const int64_t max_inst = (g.n / g.b) >> r;
        for (int64_t j = t0; j < max_inst; j += step) desc[seq * max_inst + j] = make_desc(g, seq, kDenSlot, 0, r, (int)j);
        desc += g.n_seq * max_inst;
    }
}

// dst[seq, j, :] = src[seq, idx[seq, j], :] for j < rows.
__global__ __launch_bounds__(256) void gather_rows_kernel(const char* src, const int32_t* idx, char* dst, int64_t n_seq, int64_t rows,
                                                          int row_bytes) {
    const int slices = row_bytes >> 4;
    const int64_t total = n_seq * rows * slices;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
        const int64_t row = t / slices;
        const int s = (int)(t - row * slices);
        const int64_t seq = row / rows;
        *reinterpret_cast<uintx4*>(dst + (size_t)row * row_bytes + s * 16) =
            *reinterpret_cast<const uintx4*>(src + (size_t)(seq * rows + idx[row]) * row_bytes + s * 16);
    }
}

struct LevelIdx {
    const int32_t* lvl[32];     // lvl[l]: original index of every token of the level-l buffer, [n_seq, n >> l]; lvl[0] = perm (or
};                              // null: the tokens in their order)

// The state of Alg. 3 of every segment, flattened: per slot the level-T tokens (weight 2^T), then the half block left
// at level T-1 ... 1 (weight 2^l), then the tail at level 0 (weight 1); absent places behind them (weight 0, zero rows).  A
// workgroup finds and copies kKeptRows places: every place looks up its segment and level for itself, so that nothing is serial
// over the sequence (8 x 8192 tokens, two rounds: 8 us; 26 us as one wavefront per sequence and two row gathers).
constexpr int kKeptRows = 64;
__global__ __launch_bounds__(256) void collect_kernel(const int32_t* cnt, const int32_t* start, SegGeo g, LevelIdx L, int64_t capacity,
                                                      const char* K, const char* V, int row_bytes, char* K_out, char* V_out,
                                                      int32_t* idx_out, float* w_out, int32_t* count_out) {
    __shared__ int lcnt[kSlots], lstart[kSlots];
    __shared__ int lpos[kSlots + 1];              // first place of every segment
    __shared__ int src[kKeptRows];                // token of a place, -1: none
    const int64_t seq = blockIdx.y, j0 = (int64_t)blockIdx.x * kKeptRows;
    const int tid = threadIdx.x, T = g.T, half = g.b / 2;
    if (tid < 64) {
        const int n_seg = list_segments(cnt, start, seq, tid, lcnt, lstart);
        int run = 0;
        for (int e0 = 0; e0 < n_seg; e0 += 64) {
            const int c = e0 + tid < n_seg ? lcnt[e0 + tid] : 0, full = T > 0 ? c / g.b : 0;
            int size = c - full * g.b + (T > 0 ? (full >> (T - 1)) * half : 0);
            for (int l = 1; l < T; ++l) size += ((full >> (l - 1)) & 1) * half;
            const int at = run + wave_exclusive_sum(size, tid);
            if (e0 + tid < n_seg) lpos[e0 + tid] = at;
            run = __shfl(at + size, 63);
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0)
        __builtin_amdgcn_wave_barrier();
        const int64_t j = j0 + tid;
        int tok = -1;
        float w = 0.f;
        if (j < run) {
            int lo = 0, hi = n_seg;              // the last segment that starts at or before j (all of them hold a token)
            while (hi - lo > 1) { const int m = (lo + hi) >> 1; if (lpos[m] <= j) lo = m; else hi = m; }
            const int c = lcnt[lo], st = lstart[lo], full = T > 0 ? c / g.b : 0;
            int off = (int)j - lpos[lo];
            const int top = T > 0 ? (full >> (T - 1)) * half : 0;
            if (off < top) { tok = L.lvl[T][seq * (g.n >> T) + (st >> T) + off]; w = ldexpf(1.f, T); }
            off -= top;
            for (int l = T - 1; l >= 1; --l)
                if ((full >> (l - 1)) & 1) {
                    if (off >= 0 && off < half) { tok = L.lvl[l][seq * (g.n >> l) + (st >> l) + (int64_t)(full >> l) * g.b + off]; w = ldexpf(1.f, l); }
                    off -= half;
                }
            if (off >= 0) {
                const int at = st + full * g.b + off;
                tok = L.lvl[0] ? L.lvl[0][seq * g.n + at] : at;
                w = 1.f;
            }
        }
        src[tid] = tok;
        if (j < capacity) {
            idx_out[seq * capacity + j] = tok < 0 ? 0 : tok;
            if (w_out) w_out[seq * capacity + j] = w;
        }
        if (count_out && blockIdx.x == 0 && tid == 0) count_out[seq] = run;
    }
    __syncthreads();
    const int slices = row_bytes >> 4;
    const int rows = (int)min((int64_t)kKeptRows, capacity - j0);
    for (int t = tid; t < rows * slices; t += 256) {
        const int row = t / slices, s = t - row * slices, tok = src[row];
        const size_t from = (size_t)(seq * g.n + tok) * row_bytes + s * 16, to = (size_t)(seq * capacity + j0 + row) * row_bytes + s * 16;
        uintx4 x = {0u, 0u, 0u, 0u}, y = {0u, 0u, 0u, 0u};
        if (tok >= 0) {
            if (K_out) x = *reinterpret_cast<const uintx4*>(K + from);
            if (V_out) y = *reinterpret_cast<const uintx4*>(V + from);
        }
        if (K_out) *reinterpret_cast<uintx4*>(K_out + to) = x;
        if (V_out) *reinterpret_cast<uintx4*>(V_out + to) = y;
    }
}

inline size_t up256(size_t x) { return (x + 255) / 256 * 256; }
inline unsigned grid_for(int64_t items, int per_block) {
    int64_t blocks = (items + per_block - 1) / per_block;
    if (blocks > 65536) blocks = 65536;
    if (blocks < 1) blocks = 1;
    return (unsigned)blocks;
}

}  // namespace

size_t sets_workspace_bytes(int row_bytes, int b, int64_t n_seq, int64_t n) {
    size_t s = 0;
    s += up256((size_t)n_seq * n * 4);                    // |v|^2
    s += up256((size_t)n_seq * n * 4);                    // slot of every token
    s += up256((size_t)n_seq * 4);                        // max |v|^2
    s += 2 * up256((size_t)n_seq * kSlots * 4);           // counts, starts
    s += up256((size_t)n_seq * chunks_of(n).n * kSlots * 4);   // counts per chunk
    s += 2 * up256((size_t)n_seq * n * 4);                // perm; original indices of the levels 1..T
    s += up256((size_t)n_seq * n * row_bytes);            // keys in slot order
    s += up256((size_t)n_seq * (n / 2) * row_bytes);      // level buffers, used in turn
    s += up256((size_t)n_seq * (n / 4) * row_bytes);
    s += up256((size_t)n_seq * 2 * (size_t)(n / b > 0 ? n / b : 1) * sizeof(InstDesc));   // of all rounds
    return s;
}

hipError_t run_sets(const SetsArgs& q, hipStream_t st) {
    const int64_t n_seq = q.n_seq, n = q.n;
    const int rb = q.row_bytes, b = q.b, T = q.T;
    char* ws = (char*)q.workspace;
    auto carve = [&](size_t bytes) { char* p = ws; ws += up256(bytes); return p; };
    float* norm2 = (float*)carve((size_t)n_seq * n * 4);
    int32_t* slot_ws = (int32_t*)carve((size_t)n_seq * n * 4);
    unsigned int* vmax2 = (unsigned int*)carve((size_t)n_seq * 4);
    int32_t* cnt = (int32_t*)carve((size_t)n_seq * kSlots * 4);
    int32_t* start = (int32_t*)carve((size_t)n_seq * kSlots * 4);
    const Chunks ch = chunks_of(n);
    int32_t* chunk_cnt = (int32_t*)carve((size_t)n_seq * ch.n * kSlots * 4);
    int32_t* perm = (int32_t*)carve((size_t)n_seq * n * 4);
    int32_t* lvl_idx = (int32_t*)carve((size_t)n_seq * n * 4);
    char* k_sorted = carve((size_t)n_seq * n * rb);
    char* k_a = carve((size_t)n_seq * (n / 2) * rb);
    char* k_b = carve((size_t)n_seq * (n / 4) * rb);
    InstDesc* desc = (InstDesc*)carve((size_t)n_seq * 2 * (size_t)(n / b > 0 ? n / b : 1) * sizeof(InstDesc));
    int32_t* slot = q.slot_out ? q.slot_out : slot_ws;
    hipError_t e;

    // ---- segments and the instance tables of all rounds
    const char* k0;                      // level-0 keys, slot order (or the original keys, read through perm)
    bool first_by_idx = false;
    SegGeo g;
    g.n = n; g.b = b; g.T = 0; g.seq_base = q.seq_base; g.desc = desc; g.n_seq = n_seq;
    while (g.T < T && ((n / b) >> g.T) > 0) ++g.T;                // rounds that any segment can have a block for
    const int rounds = g.T, status_words = T > 0 ? T : 1;

    if (q.numerator) {
        const bool erase = q.erase2 > 0.f;                        // only the erase rule needs the largest norm
        if (erase && (e = launch_fill_u32(vmax2, 0u, n_seq, st)) != hipSuccess) return e;
        const dim3 g1((unsigned)ch.n, (unsigned)n_seq);
#define BKV_SLOTS(TT, DD)                                                                                                              \
        do {                                                                                                                           \
            if (erase) hipLaunchKernelGGL((value_slot_kernel<TT, DD, true>), g1, dim3(256), 0, st, q.V, n, ch.tokens, norm2, vmax2,    \
                                          slot, chunk_cnt, q.status_out, status_words);                                                \
            else hipLaunchKernelGGL((value_slot_kernel<TT, DD, false>), g1, dim3(256), 0, st, q.V, n, ch.tokens, norm2, vmax2, slot,   \
                                    chunk_cnt, q.status_out, status_words);                                                            \
        } while (0)
        if (q.dtype == BKV_BF16 && q.d == 128) BKV_SLOTS(__bf16, 128);
        else if (q.dtype == BKV_BF16 && q.d == 64) BKV_SLOTS(__bf16, 64);
        else if (q.dtype == BKV_F32 && q.d == 128) BKV_SLOTS(float, 128);
        else if (q.dtype == BKV_F32 && q.d == 64) BKV_SLOTS(float, 64);
        else return hipErrorInvalidValue;
#undef BKV_SLOTS
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (erase) {
            hipLaunchKernelGGL(slot_kernel, g1, dim3(256), 0, st, norm2, vmax2, n, ch.tokens, q.erase2, slot, chunk_cnt);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        const dim3 g2((unsigned)n_seq, (unsigned)(ch.n + rounds));
        if (n_seq * ch.n * (ch.n + rounds) >= kPrefixFrom) {
            hipLaunchKernelGGL(chunk_prefix_kernel, dim3(kSlots / 64, (unsigned)n_seq), dim3(64), 0, st, chunk_cnt, (int)ch.n, cnt);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            hipLaunchKernelGGL(segments_kernel<true>, g2, dim3(kPartThreads), 0, st, slot, chunk_cnt, (int)ch.n, ch.tokens, g, cnt, start, perm);
        } else
            hipLaunchKernelGGL(segments_kernel<false>, g2, dim3(kPartThreads), 0, st, slot, chunk_cnt, (int)ch.n, ch.tokens, g, cnt, start, perm);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        // blocks resident as one chunk read their key rows through perm (no copy in slot order); larger blocks need the copy
        if (!compress_block_resident(rb, b, true)) {
            hipLaunchKernelGGL(gather_rows_kernel, dim3(grid_for(n_seq * n * (rb / 16), 256)), dim3(256), 0, st, q.K, perm, k_sorted, n_seq,
                               n, rb);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            k0 = k_sorted;
        } else {
            k0 = q.K;
            first_by_idx = true;
        }
    } else {
        hipLaunchKernelGGL(single_segment_kernel, dim3(grid_for(q.slot_out ? n : 2 * (n / b), 256), (unsigned)n_seq), dim3(256), 0, st, g, cnt,
                           start, q.slot_out, q.status_out, status_words);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        perm = nullptr;                   // already in order
        k0 = q.K;
    }
    g.T = T;

    // ---- rounds
    LevelIdx L;
    for (int l = 0; l < 32; ++l) L.lvl[l] = nullptr;
    L.lvl[0] = perm;
    {
        int32_t* p = lvl_idx;
        for (int l = 1; l <= T; ++l) { L.lvl[l] = p; p += n_seq * (n >> l); }
    }
    const char* k_in = k0;
    int64_t signs_off = 0;
    for (int r = 0; r < rounds; ++r) {
        const int64_t max_inst = (n / b) >> r;
        CompressArgs a = q.common;
        a.desc = desc;
        a.K = k_in;
        a.k_by_idx = (r == 0 && first_by_idx) ? 1 : 0;
        a.K_out = (r == T - 1) ? nullptr : ((r & 1) ? k_b : k_a);      // the last level's keys are gathered from the originals
        a.V = q.numerator ? q.V : nullptr;
        a.V_out = nullptr; a.w_out = nullptr;
        a.v_seq_stride = n;
        a.idx_in = L.lvl[r];
        a.idx_out = const_cast<int32_t*>(L.lvl[r + 1]);
        a.signs_out = q.signs_out ? q.signs_out + signs_off : nullptr;
        a.status_out = q.status_out; a.status_stride = T;
        a.tree_mode = 1; a.round = r;
        a.blocks_per_seq = 1;
        if ((e = launch_compress(q.dtype, q.d, false, a, n_seq * max_inst, st)) != hipSuccess) return e;
        k_in = a.K_out;
        signs_off += n_seq * (n >> r);
        desc += n_seq * max_inst;
    }

    // ---- the kept sets
    const int64_t tiles = q.capacity > 0 ? (q.capacity + kKeptRows - 1) / kKeptRows : 1;
    hipLaunchKernelGGL(collect_kernel, dim3((unsigned)tiles, (unsigned)n_seq), dim3(256), 0, st, cnt, start, g, L, q.capacity, q.K, q.V, rb,
                       q.K_out, q.V_out, q.idx_ws, q.w_out, q.count_out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------ Alg. 1 token by token
namespace {

template <typename T, int D>
__global__ __launch_bounds__(64) void stream_route_kernel(StreamState s, const char* k, const char* v, int32_t j) {
    (void)stream_route_token<T, D>(s, k, v, j, blockIdx.x, threadIdx.x);
}

}  // namespace

hipError_t stream_route(const StreamState& s, const void* k, const void* v, int64_t j, hipStream_t st) {
    const dim3 grid((unsigned)s.n_seq), block(64);
    const char* kp = (const char*)k;
    const char* vp = (const char*)v;
    if (s.dtype == BKV_BF16 && s.d == 128) hipLaunchKernelGGL((stream_route_kernel<__bf16, 128>), grid, block, 0, st, s, kp, vp, (int32_t)j);
    else if (s.dtype == BKV_BF16 && s.d == 64) hipLaunchKernelGGL((stream_route_kernel<__bf16, 64>), grid, block, 0, st, s, kp, vp, (int32_t)j);
    else if (s.dtype == BKV_F32 && s.d == 128) hipLaunchKernelGGL((stream_route_kernel<float, 128>), grid, block, 0, st, s, kp, vp, (int32_t)j);
    else if (s.dtype == BKV_F32 && s.d == 64) hipLaunchKernelGGL((stream_route_kernel<float, 64>), grid, block, 0, st, s, kp, vp, (int32_t)j);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace bkv
