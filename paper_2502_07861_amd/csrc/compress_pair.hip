// SoftmaxBalance for launches with more blocks than compute units: two blocks per compute unit instead of one.
//
// The same arithmetic as compress_kernel (compress.hip), operation for operation, so that both give the same decisions;
// what differs is where things live.  That kernel keeps up to 512 key rows of a block in LDS and eight wavefronts of 256
// registers on a compute unit; whatever such a block waits for (its rows, the serial walk, the gather) nothing else runs
// beside.  Here a workgroup needs half of the registers and half of LDS, so that two blocks are resident and one's waiting
// is the other's work:
//   * a column panel of 64 keys lives in the registers of the wavefront that owns it (the B operand of all its tiles);
//     LDS holds three row panels at a time (the A operands): each owner writes its panel from its registers into a slot
//     when the slot's last rows have been read by everybody;
//   * every owner walks its own panel: sigma never leaves its registers, the diagonal tile (two buffers in LDS) turns there
//     into one column per lane, and the signs go out as before;
//   * a tile is formed in two halves of 32 rows (32 accumulator registers): first half, wait for the row panel's signs,
//     signed sums, second half.  The tile whose signs come last is formed column half by column half with all its 64
//     weights held, by when the panel's own rows have left the registers;
//   * blocks of more than 512 rows: the first chunk's rows come back from memory two panels at a time, straight into LDS,
//     and all owners of the second chunk's columns use them together.
// What bounds it (bf16, d = 128): no single unit.  At b = 1024 the vector unit is busy for half and the matrix pipe for a
// quarter of the time of a block; leaving out the tiles' exponentials, half of the matrix instructions, the statistics or
// the gather shortens it by 5 to 12 % each.  At b <= 512 the traffic (3 TB/s) comes on top.
// 256 sequences x 32768 tokens, two rounds, against one block per compute unit: b = 1024 3.12 -> 2.82 ms, b = 512
// 2.50 -> 1.92, b = 256 2.91 -> 1.83; fp32, d = 64, 64 sequences: b = 256 1.27 -> 1.07.
#include <utility>

#include "bkv_device.h"
#include "bkv_host.h"
#include "compress_device.h"

namespace bkv {
namespace {

// (128 vector registers hold a panel, 32 to 64 weights and little else: every value that could be kept across the tile loops is formed
// anew where it is needed, see also args_here and local_copy.)
constexpr int kPanelBytes = 64 * 256;                       // one panel of 64 key rows
constexpr int kSlotCount = 3;                               // row panels resident in LDS
constexpr int kTileStrideA = 36, kTileStrideB = 68;         // floats per column of a diagonal tile: columns 0..31 (rows 0..31), 32..63
constexpr int kTileFloats = 32 * kTileStrideA + 32 * kTileStrideB;
constexpr int kOffTile = kSlotCount * kPanelBytes;
constexpr int kOffEta = kOffTile + 2 * kTileFloats * 4;
constexpr int kOffMask = kOffEta + 4 * 64 * 4;
constexpr int kOffScal = kOffMask + 16 * 8;
constexpr int kOffProg = kOffScal + 128;
constexpr int kOffZero = kOffProg + 128;
constexpr int kOffNa = kOffZero + 128;
constexpr int kBatchBytes = 4 * kPanelBytes;                // 256 rows on their way through LDS (slots and tiles are idle then)
constexpr int kOffPart = kBatchBytes;                       // mean partials [8][D], the mean [D]: behind the batch
static_assert(kOffPart + (8 + 1) * 128 * 4 <= kOffEta, "partials fit behind a batch");
static_assert(4 * kPanelBytes + 8 * 4 * 64 * 4 <= kOffEta, "and so do the sums that two wavefronts share");

__device__ __forceinline__ void load_lds16(const char* src, char* dst) {       // lane l: 16 bytes from src to dst + 16 l
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
// a value that the compiler forms address arithmetic from here and does not carry around in several registers
__device__ __forceinline__ int local_copy(int x) { asm volatile("" : "+v"(x)); return x; }
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// An entry of an instance table, by scalar loads.
__device__ __forceinline__ const InstDesc* table_entry(const InstDesc* table, int64_t inst) {
    return (const InstDesc*)(const __attribute__((address_space(4))) InstDesc*)(unsigned long long)(table + inst);
}

// TABLE: ragged launches, the instances' coordinates come from CompressArgs::desc.
template <typename T, int D, bool TWO, bool TABLE>
__global__ __launch_bounds__(kThreads, 4) void compress_pair_kernel(const CompressArgs a0) {
    const CompressArgs& a = *args_here();
    typedef Geo<T, D> G;
    typedef typename Elem<T>::Frag Frag;
    static_assert(G::kRowBytes == 256, "rows of 256 bytes");
    constexpr int EPL = Elem<T>::kPerFrag, SL = 16, RG = 32, KG = 8;

    extern __shared__ __align__(256) char smem[];
    const int b = a.b, nP = b >> 6;
    float* etaF = reinterpret_cast<float*>(smem + kOffEta);        // ring of 4 panels: +-1 of a panel, entry h*32 + 16*rb + r
    unsigned long long* etaMask = reinterpret_cast<unsigned long long*>(smem + kOffMask);
    float* scal = reinterpret_cast<float*>(smem + kOffScal);
    int* prog = reinterpret_cast<int*>(smem + kOffProg);
    float* narow = reinterpret_cast<float*>(smem + kOffNa);
    float* wpart = reinterpret_cast<float*>(smem + kOffPart);
    float* mu = wpart + 8 * D;
    int* keptIdx = reinterpret_cast<int*>(smem + kOffTile);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int64_t inst = blockIdx.x;
    const char* Kin;
    uint64_t key, ctr0;
    {
        const int64_t seq = inst / a.blocks_per_seq;
        const int blk = (int)(inst - seq * a.blocks_per_seq);
        uint64_t stream = a.tree_mode ? (uint64_t)(64 * (a.seq_base + seq) + a.round) : (uint64_t)inst;
        if (a.inst_ids) stream = a.inst_ids[inst];
        ctr0 = a.tree_mode ? (uint64_t)(a.blk_base + blk) * (uint64_t)b : 0ull;
        int64_t in_tok0 = seq * a.in_seq_stride + (int64_t)blk * b;
        if constexpr (TABLE) {
            const InstDesc& ds = *table_entry(a.desc, inst);
            if (!ds.valid) return;                                  // the grid is an upper bound; uniform for the workgroup, before any barrier
            in_tok0 = ds.in_tok; stream = ds.stream; ctr0 = ds.ctr0;
        }
        key = stream_key(a.seed, stream);
        Kin = a.K + in_tok0 * G::kRowBytes;
    }
    const bool center = (a.flags & BKV_CENTER_KEYS) != 0;
    const bool need_norm = !(a.rkey2 > 0.f);
    const float alpha = a.alpha;
    auto lane_here = [&]() -> int { return local_copy(threadIdx.x) & 63; };
    auto threshold = [&](int i) -> float {
        float u;
        const float* given = args_here()->uniforms;
        if (given) u = given[(size_t)inst * b + i];
        else u = (float)draw_bits_keyed(key, ctr0 + (uint64_t)i) * (1.0f / 16777216.0f);
        return 1.f - 2.f * u;
    };
    // this thread's row group and slice while rows pass through LDS linearly: place lane % 16 of row r holds slice
    // (lane % 16) ^ (r % 16), the layout that Geo describes
    const int rg = tid >> 4, pos = lane & 15, sl = pos ^ (rg & 15);
    const int own = tid * 16;                                      // this thread's 16 bytes of every 32 rows
    auto row_offset = [&]() -> int {
        const int t = local_copy(threadIdx.x), r = t >> 4;
        return r * 256 + (((t & 15) ^ (r & 15)) << 4);
    };
    // rows 32 u0 .. 32 u0 + 255 of the block -> the batch area
    auto fetch = [&](int u0) {
        const int off = row_offset();
        int rows = b, w = wave;
        const char* src = Kin;
        asm volatile("" : "+s"(rows), "+s"(w), "+s"(src));
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (32 * (u0 + u) < rows) load_lds16(src + (size_t)(u0 + u) * 8192 + off, smem + u * 8192 + w * 1024);
    };
    // this lane's fragments of a panel at `base`: row 32 rb + n, k-group g at foff ^ 32 g
    const int foff = n * 256 + ((h ^ (n & 15)) << 4);
    Frag B[KG][2];
    auto read_panel = [&](const char* base) {
        const int at = local_copy(foff) + (int)(base - smem);
#pragma unroll
        for (int g = 0; g < KG; ++g)
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) B[g][rb] = *reinterpret_cast<const Frag*>(smem + (at ^ (32 * g)) + rb * 8192);
    };

    float part[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) part[e] = 0.f;
    auto add_rows = [&](int u0) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (32 * (u0 + u) < b) {
                Elem<T>::accumulate(part, *reinterpret_cast<const uintx4*>(smem + u * 8192 + own));
                if (u & 1) __builtin_amdgcn_sched_barrier(0);     // (registers: not all eight at a time)
            }
    };
    auto load_rows = [&](uintx4 (&keep)[8], int u0) {                      // rows 32 u0 .. 32 u0 + 255 of the block -> registers
        const unsigned int off = (unsigned int)row_offset();
#pragma unroll
        for (int u = 0; u < 8; ++u)                     // (past the end: the last rows again, not counted below)
            keep[u] = *reinterpret_cast<const uintx4*>(Kin + (size_t)(unsigned)min((u0 + u) * 8192, (b - 32) * 256) + off);
    };
    auto store_rows = [&](const uintx4 (&keep)[8], int u0) {
        const int own = local_copy(threadIdx.x) * 16;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (32 * (u0 + u) < b) *reinterpret_cast<uintx4*>(smem + u * 8192 + own) = keep[u];
    };
    auto add_kept = [&](const uintx4 (&keep)[8], int u0) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (32 * (u0 + u) < b) Elem<T>::accumulate(part, keep[u]);
    };
    if (tid < 32) reinterpret_cast<float*>(smem + kOffZero)[tid] = 0.f;
    if (tid < 32) prog[tid] = 0;
    if (tid < 4) reinterpret_cast<unsigned int*>(scal + 16)[tid] = tid == 0 ? 0x7f61b1e6u : 0u;          // 3e38: no margin seen yet
    const int flip = (blockIdx.x >> 8) & 1;
    int l = flip ? 7 - wave : wave;                                 // this wavefront's column panel of the chunk
    // Blocks of two chunks fetch rows and form their statistics for a third of their time, beside a block that walks at raised priority and leaves
    // them the vector unit's gaps: 40 of 125 us, where the statistics take 2.3 by themselves.  One step up they are sooner done and the two
    // blocks' phases lie better (256 x 32768 tokens, b = 1024, one round 2.04 -> 1.97 ms, 64 x 32768, two rounds 764 -> 740 us); not in every launch
    // (launch_compress_pair).  Three steps give less, raised for the output or the second chunk's rows as well nothing; blocks of one
    // chunk lose (b = 384 340 -> 352 us, 256 488 -> 495).
    if constexpr (TWO)
        if (a.raise_fetch) __builtin_amdgcn_s_setprio(1);
    // Two batches at a time are on their way: one straight into LDS, one into registers.
    fetch(0);
    uintx4 rows1[8], keep[TWO ? 8 : 1];
    if (b > 256) load_rows(rows1, 8);
    wait_loads();
    __syncthreads();
    if (center) add_rows(0);
    if (l < 4 && l < nP) read_panel(smem + l * kPanelBytes);
    if (b > 256) {
        __syncthreads();
        store_rows(rows1, 8);
        if (center) add_kept(rows1, 8);
        __syncthreads();
        if (l >= 4 && l < nP) read_panel(smem + (l - 4) * kPanelBytes);
    }
    if constexpr (TWO) {
        __syncthreads();
        load_rows(keep, 16);                       // (these stay in registers until the statistics have used them)
        fetch(24);
        wait_loads();
        if (center) { add_kept(keep, 16); add_rows(24); }           // (a thread reads what it has fetched itself)
    }
    if (center) {
        // the four rows of 16 lanes, whose slices stand at places that differ by the row's number: row 0 collects
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
            part[e] += dpp<0xB1>(lane_pair<16>(part[e]).b);
            part[e] += dpp<0x4E>(lane_pair<32>(part[e]).b);
        }
        if (lane < SL)
#pragma unroll
            for (int q = 0; q < EPL / 4; ++q) {
                const floatx4 t = {part[4 * q], part[4 * q + 1], part[4 * q + 2], part[4 * q + 3]};
                *reinterpret_cast<floatx4*>(wpart + wave * D + sl * EPL + 4 * q) = t;
            }
    }
    __syncthreads();
    // ------------------------------------------------------------------ block statistics
    float mumu = 0.f;
    float mloc[TWO ? EPL : 1];
    if constexpr (!TWO) {
        constexpr int MH = D / 64;
        float mcol[MH];
#pragma unroll
        for (int hh = 0; hh < MH; ++hh) {
            float s0 = 0.f;
            if (center)
#pragma unroll
                for (int w = 0; w < kWaves; ++w) s0 += wpart[w * D + 64 * hh + lane];
            mcol[hh] = s0 * (1.f / (float)b);
            mumu = fmaf(mcol[hh], mcol[hh], mumu);
        }
        mumu = wave_sum(mumu);
        if (wave == 0)
#pragma unroll
            for (int hh = 0; hh < MH; ++hh) mu[64 * hh + lane] = mcol[hh];
    } else {
#pragma unroll
        for (int e = 0; e < EPL; ++e) mloc[e] = 0.f;
        if (center) {
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
#pragma unroll
                for (int e = 0; e < EPL; ++e) mloc[e] += wpart[w * D + sl * EPL + e];
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
                mloc[e] *= 1.f / (float)b;
                mumu = fmaf(mloc[e], mloc[e], mumu);
            }
            mumu = group_sum<SL>(mumu);
        }
        if (tid < SL)
#pragma unroll
            for (int e = 0; e < EPL; ++e) mu[sl * EPL + e] = mloc[e];
    }
    __syncthreads();
    if (center || need_norm) {
        float amax = -3.0e38f;
        if constexpr (TWO) {
            // rows 512..767 are still in this thread's registers, rows 768.. in LDS
            float ya[8], yn[8];
            auto terms = [&](const uintx4& raw, float& pa, float& pn) {
                float f[EPL];
                Elem<T>::unpack(raw, f);
                pa = 0.f;
#pragma unroll
                for (int e = 0; e < EPL; ++e) pa = fmaf(f[e], mloc[e], pa);
                pn = Elem<T>::dot(raw, raw);
            };
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                float pa0, pn0, pa1, pn1;
                terms(keep[k], pa0, pn0);
                terms(*reinterpret_cast<const uintx4*>(smem + k * 8192 + own), pa1, pn1);     // (rows past the end: not used below)
                ya[k] = row16_pair(pa0, pa1, pos);
                yn[k] = row16_pair(pn0, pn1, pos);
                __builtin_amdgcn_sched_barrier(0);
            }
            const float pa = row16_rest(ya, pos), pn = row16_rest(yn, pos);
            const int i = (16 + pos) * RG + rg;
            if (i < b) {
                narow[i] = -pa;
                amax = fmaxf(amax, pn - 2.f * pa + mumu);
            }
        }
        if (l < nP) {
            // one row per lane: the two halves of a wavefront trade slices, so that lane (n, h) has row 32 h + n
            float pa = 0.f, pn = 0.f;
#pragma unroll
            for (int g = 0; g < KG; ++g) {
                const uintx4 r0 = __builtin_bit_cast(uintx4, B[g][0]), r1 = __builtin_bit_cast(uintx4, B[g][1]);
                uintx4 s0, s1;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const auto sw = __builtin_amdgcn_permlane32_swap(r0[i], r1[i], false, false);
                    s0[i] = sw[0]; s1[i] = sw[1];
                }
                float f[EPL];
                Elem<T>::unpack(s0, f);
#pragma unroll
                for (int e = 0; e < EPL; ++e) pa = fmaf(f[e], mu[2 * g * EPL + e], pa);
                pn += Elem<T>::dot(s0, s0);
                Elem<T>::unpack(s1, f);
#pragma unroll
                for (int e = 0; e < EPL; ++e) pa = fmaf(f[e], mu[(2 * g + 1) * EPL + e], pa);
                pn += Elem<T>::dot(s1, s1);
            }
            narow[(l << 6) + lane] = -pa;
            amax = fmaxf(amax, pn - 2.f * pa + mumu);
        }
        amax = wave_max(amax);
        if (lane == 0) scal[2 + wave] = amax;
    } else {
        for (int i = tid; i < b; i += kThreads) narow[i] = 0.f;
    }
    __syncthreads();
    float row_const;
    {
        float A = a.rkey2;
        if (need_norm) {
            A = scal[2];
#pragma unroll
            for (int w = 1; w < kWaves; ++w) A = fmaxf(A, scal[2 + w]);
        }
        row_const = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, alpha * (mumu - A + a.cterm))));
    }

    // ------------------------------------------------------------------ the chunks
    if constexpr (TWO) __builtin_amdgcn_s_setprio(0);
    unsigned int* events = reinterpret_cast<unsigned int*>(scal + 16);   // smallest margin, largest |sigma|, near ties, FAIL
    int* eta_done = prog;
    int* diag_taken = prog + 1;
    int* sync_err = prog + 3;
    int* rowp = prog + 8;             // rowp[l]: row panels whose LDS rows the owner of column panel l needs no more
    int* ready = prog + 16;           // ready[l]: row panel l is in its slot
    float cc0, cc1;                   // rc - alpha a_j of this lane's two columns
    // kernel weights of rows 32 rb .. 32 rb + 31 of the panel at `slot` (row terms na) against this wavefront's columns
    auto half_tile = [&](const char* slot, const float* na, int rb, floatx16& w0, floatx16& w1) {
        floatx16 r;
        const int h = lane_here() >> 5;
        const int fo = local_copy(foff);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const floatx4 t = *reinterpret_cast<const floatx4*>(na + 32 * rb + 8 * q + 4 * h);
            r[4 * q] = t[0]; r[4 * q + 1] = t[1]; r[4 * q + 2] = t[2]; r[4 * q + 3] = t[3];
        }
        Frag A[KG];
        const int at = fo + (int)(slot - smem);              // (panels start at multiples of 256 bytes)
        A[0] = *reinterpret_cast<const Frag*>(smem + at + rb * 8192);
        A[1] = *reinterpret_cast<const Frag*>(smem + (at ^ 32) + rb * 8192);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < KG; ++g) {                   // fragments requested two k-groups ahead: more would not fit
            if (g + 2 < KG) A[g + 2] = *reinterpret_cast<const Frag*>(smem + (at ^ (32 * (g + 2))) + rb * 8192);
            if (g == 0) {
                w0 = Elem<T>::mma_from(A[0], B[0][0], r);
                w1 = Elem<T>::mma_from(A[0], B[0][1], r);
            } else {
                Elem<T>::mma(w0, A[g], B[g][0]);
                Elem<T>::mma(w1, A[g], B[g][1]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            w0[q] = fast_exp2(fmaf(w0[q], alpha, cc0));
            w1[q] = fast_exp2(fmaf(w1[q], alpha, cc1));
        }
    };
    auto add_signed = [&](const float* sgn /* + 32 h */, int rb, const floatx16& w0, const floatx16& w1, float& cs0, float& cs1) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const floatx4 s = *reinterpret_cast<const floatx4*>(sgn + 16 * rb + 4 * q);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                cs0 = fmaf(s[r], w0[4 * q + r], cs0);
                cs1 = fmaf(s[r], w1[4 * q + r], cs1);
            }
        }
    };

    // (a new name for the panel's registers: a spill in the statistics must not become one in the tile loops)
#pragma unroll
    for (int g = 0; g < KG; ++g)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) asm volatile("" : "+v"(B[g][rb]));
    auto chunk = [&](auto chunk_no) {
        constexpr int c = decltype(chunk_no)::value;
        const int p0 = 8 * c, nPc = min(8, nP - p0);
        if constexpr (c > 0) {
            l = 7 - l;
            __syncthreads();
            if (tid < 32 && tid != 3) prog[tid] = 0;
            fetch(16);
            uintx4 rows3[8];
            if (b > 768) load_rows(rows3, 24);
            wait_loads();
            __syncthreads();
            // (the registers of the first chunk's panel hold nothing any more: unless this says so they count as needed
            // through the first chunk's walk, on the path of a wavefront that owns no panel here)
#pragma unroll
            for (int g = 0; g < KG; ++g)
#pragma unroll
                for (int rb = 0; rb < 2; ++rb) B[g][rb] = Frag{};
            const int pl = nPc <= 4 ? l & 3 : l;                    // (four panels at most: two wavefronts hold each, see below)
            if (pl < 4 && pl < nPc) read_panel(smem + pl * kPanelBytes);
            if (b > 768) {
                __syncthreads();
                store_rows(rows3, 24);
                __syncthreads();
                if (pl >= 4 && pl < nPc) read_panel(smem + (pl - 4) * kPanelBytes);
            }
            __syncthreads();
        }
        const bool owner = l < nPc;
        const int I0 = p0 + l;
        float sig = 0.f;
        cc0 = cc1 = 0.f;
        auto column_terms = [&](int I) {
            const int n = lane_here() & 31;
            cc0 = fmaf(alpha, narow[(I << 6) + n], row_const);
            cc1 = fmaf(alpha, narow[(I << 6) + 32 + n], row_const);
        };
        if constexpr (c > 0) {
            // ---------------------------------------------------------- rows of the first chunk (all signs known)
            // Two row panels at a time, the next two on their way.  With at most four columns in this chunk two wavefronts
            // share one, a row panel of each pair for each; the owner then adds up the eight sums in order.
            const bool shared = nPc <= 4;
            const int pl = shared ? l & 3 : l, half_no = l >> 2;
            const bool mine = pl < nPc;
            float* xch = reinterpret_cast<float*>(smem + 4 * kPanelBytes);          // [8 row panels][4 columns][64]
            auto fetch_panel = [&](int I) {
                int w = wave;
                asm volatile("" : "+s"(w));
                char* dst = smem + (I & 3) * kPanelBytes + w * 1024;
                const int off = row_offset();
#pragma unroll
                for (int u = 0; u < 2; ++u) load_lds16(Kin + (size_t)(2 * I + u) * 8192 + off, dst + u * 8192);
            };
            auto expand = [&](int I) {                              // signs of panel I, accumulator order (one wavefront)
                const int lane = lane_here(), h = lane >> 5;
                const unsigned long long m = etaMask[I];
                const int k = lane & 31;
                const int row = 32 * (k >> 4) + 8 * ((k & 15) >> 2) + 4 * h + (k & 3);
                etaF[((I & 3) << 6) + lane] = ((m >> row) & 1ull) ? 1.f : -1.f;
            };
            fetch_panel(0);
            fetch_panel(1);
            if (wave < 2) expand(wave);
            if (mine) column_terms(p0 + pl);
            float tot = 0.f;
#pragma unroll 1
            for (int I = 0; I < 8; ++I) {
                if ((I & 1) == 0) {
                    wait_loads();
                    __syncthreads();
                    if (I + 2 < 8) {
                        fetch_panel(I + 2);
                        fetch_panel(I + 3);
                        if (wave < 2) expand(I + 2 + wave);
                    }
                }
                if (mine && (!shared || (I & 1) == half_no)) {
                    const char* slot = smem + (I & 3) * kPanelBytes;
                    const float* sgn = etaF + ((I & 3) << 6) + (lane_here() & 32);
                    float cs0 = 0.f, cs1 = 0.f;
                    floatx16 w0, w1;
#pragma unroll
                    for (int rb = 0; rb < 2; ++rb) {
                        half_tile(slot, narow + (I << 6), rb, w0, w1);
                        add_signed(sgn, rb, w0, w1, cs0, cs1);
                    }
                    const float cs = halves_sum(cs0, cs1);
                    if (shared) xch[(I * 4 + pl) * 64 + lane_here()] = cs;
                    else tot += cs;
                }
            }
            __syncthreads();                                        // the slots go to the panels of this chunk
            if (shared) {
                if (owner) {
                    const float* in = xch + l * 64 + lane_here();
#pragma unroll
                    for (int I = 0; I < 8; ++I) tot += in[I * 256];
                }
                __syncthreads();
            }
            sig = tot;
        } else if (owner) column_terms(I0);
        // -------------------------------------------------------------- panels of this chunk
        if (owner) {
            float* tile = reinterpret_cast<float*>(smem + kOffTile) + (l & 1) * kTileFloats;
            const float* naP = narow + (I0 << 6);
            auto diagonal = [&]() {
                const int lane = lane_here(), n = lane & 31, h = lane >> 5;
                floatx16 q0, q1;
#pragma unroll
                for (int part_ = 0; part_ < 2; ++part_) {           // rows 0..31 (both column halves), rows 32..63
                    floatx16 r;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const floatx4 t = *reinterpret_cast<const floatx4*>(naP + 32 * part_ + 8 * q + 4 * h);
                        r[4 * q] = t[0]; r[4 * q + 1] = t[1]; r[4 * q + 2] = t[2]; r[4 * q + 3] = t[3];
                    }
#pragma unroll
                    for (int g = 0; g < KG; ++g) {
                        if (g == 0) {
                            if (part_ == 0) q0 = Elem<T>::mma_from(B[0][0], B[0][0], r);
                            q1 = Elem<T>::mma_from(B[0][part_], B[0][1], r);
                        } else {
                            if (part_ == 0) Elem<T>::mma(q0, B[g][0], B[g][0]);
                            Elem<T>::mma(q1, B[g][part_], B[g][1]);
                        }
                    }
#pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        const int lrow = 8 * (q >> 2) + 4 * h + (q & 3);
                        if (part_ == 0) {
                            const float x = fast_exp2(fmaf(q0[q], alpha, cc0));
                            q0[q] = n > lrow ? x : 0.f;
                        }
                        const float y = fast_exp2(fmaf(q1[q], alpha, cc1));
                        q1[q] = (part_ == 0 || n > lrow) ? y : 0.f;
                    }
                    if (part_ == 0) await(diag_taken, l - 1, sync_err);       // the tile before the previous one is in registers
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (part_ == 0) {
                            const floatx4 t = {q0[4 * q], q0[4 * q + 1], q0[4 * q + 2], q0[4 * q + 3]};
                            *reinterpret_cast<floatx4*>(tile + n * kTileStrideA + 8 * q + 4 * h) = t;
                        }
                        const floatx4 t = {q1[4 * q], q1[4 * q + 1], q1[4 * q + 2], q1[4 * q + 3]};
                        *reinterpret_cast<floatx4*>(tile + 32 * kTileStrideA + n * kTileStrideB + 32 * part_ + 8 * q + 4 * h) = t;
                    }
                }
            };
            auto offer_rows = [&]() {
                if (l + 1 >= nPc) return;
                // this panel's rows for the columns behind it, once everybody is through with the slot's previous rows
                if (l >= kSlotCount) {
                    const int need = l - kSlotCount + 1;
                    bool ok = false;
                    const int lane = lane_here();
                    for (int it = 0; it < kSpinLimit && !ok; ++it) {
                        const int seen = __hip_atomic_load(rowp + (lane & 7), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        ok = __ballot(seen < need && (lane & 7) >= need && (lane & 7) < nPc && (lane & 7) != l) == 0ull;
                        if (!ok) __builtin_amdgcn_s_sleep(1);
                    }
                    if (!ok) __hip_atomic_store(sync_err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                }
                const int at = local_copy(foff) + (l % kSlotCount) * kPanelBytes;
#pragma unroll
                for (int g = 0; g < KG; ++g)
#pragma unroll
                    for (int rb = 0; rb < 2; ++rb) *reinterpret_cast<Frag*>(smem + (at ^ (32 * g)) + rb * 8192) = B[g][rb];
                publish_in_order(ready + l, 1);
            };
            {
                const float t = 0.f - threshold((I0 << 6) + lane_here());    // minus the decision threshold ...
                sig = c > 0 ? t + sig : t;                              // ... plus what the first chunk adds
            }
            if (l < 2) {
                __builtin_amdgcn_s_setprio(2);
                diagonal();
                offer_rows();
            }
#pragma unroll 1
            for (int i = 0; i + 1 < l; ++i) {
                if (i == l - 2) diagonal();
                await(ready + i, 1, sync_err);
                const char* slot = smem + (i % kSlotCount) * kPanelBytes;
                const float* sgn = etaF + ((i & 3) << 6) + (lane_here() & 32);
                float cs0 = 0.f, cs1 = 0.f;
                floatx16 w0, w1;
                half_tile(slot, narow + ((p0 + i) << 6), 0, w0, w1);
                asm volatile("" : "+v"(w0), "+v"(w1));
                if (i == l - 2) {
                    offer_rows();
                    __builtin_amdgcn_s_setprio(1);                // two walks from now at the latest the walk waits for this wavefront
                }
                await(eta_done, i + 1, sync_err);
                add_signed(sgn, 0, w0, w1, cs0, cs1);
                half_tile(slot, narow + ((p0 + i) << 6), 1, w0, w1);
                publish_in_order(rowp + l, i + 1);
                add_signed(sgn, 1, w0, w1, cs0, cs1);
                sig += halves_sum(cs0, cs1);
            }
            if (l > 0) {
                // the tile whose signs come last: weights first (column half by column half, after which the panel's own
                // rows leave the registers), then the signs
                const int i = l - 1;
                __builtin_amdgcn_s_setprio(2);
                await(ready + i, 1, sync_err);
                const char* slot = smem + (i % kSlotCount) * kPanelBytes;
                const float* na = narow + ((p0 + i) << 6);
                const int h = lane_here() >> 5;
                floatx16 w[2][2];                                    // [column half][row half]
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    const int at = local_copy(foff) + (int)(slot - smem);
#pragma unroll
                    for (int rb = 0; rb < 2; ++rb) {
                        floatx16 r;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const floatx4 t = *reinterpret_cast<const floatx4*>(na + 32 * rb + 8 * q + 4 * h);
                            r[4 * q] = t[0]; r[4 * q + 1] = t[1]; r[4 * q + 2] = t[2]; r[4 * q + 3] = t[3];
                        }
                        w[cb][rb] = r;
                    }
                    Frag A[KG][2];
                    auto load_a = [&](int g) {
#pragma unroll
                        for (int rb = 0; rb < 2; ++rb) A[g][rb] = *reinterpret_cast<const Frag*>(smem + (at ^ (32 * g)) + rb * 8192);
                    };
                    load_a(0);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int g = 0; g < KG; ++g) {
                        if (g + 1 < KG) load_a(g + 1);
#pragma unroll
                        for (int rb = 0; rb < 2; ++rb) Elem<T>::mma(w[cb][rb], A[g][rb], B[g][cb]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    const float cc = cb == 0 ? cc0 : cc1;
#pragma unroll
                    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                        for (int q = 0; q < 16; ++q) w[cb][rb][q] = fast_exp2(fmaf(w[cb][rb][q], alpha, cc));
                    __builtin_amdgcn_sched_barrier(0);
                }
                asm volatile("" : "+v"(w[0][0]), "+v"(w[0][1]), "+v"(w[1][0]), "+v"(w[1][1]));
                publish_in_order(rowp + l, i + 1);
                __builtin_amdgcn_s_setprio(3);
                await<true>(eta_done, i + 1, sync_err);
                const float* sgn = etaF + ((i & 3) << 6) + (lane_here() & 32);
                float cs0 = 0.f, cs1 = 0.f;
                add_signed(sgn, 0, w[0][0], w[1][0], cs0, cs1);
                add_signed(sgn, 1, w[0][1], w[1][1], cs0, cs1);
                sig += halves_sum(cs0, cs1);
            }
            // ------------------------------------------------ the walk over panel I0 (Alg. 2 lines 4-11)
            __builtin_amdgcn_s_setprio(3);
            __builtin_amdgcn_sched_barrier(0);
            const int lane = lane_here(), n = lane & 31, h = lane >> 5;
            float g[64];
            {
                const float* lo = tile + (h ? 32 * kTileStrideA + n * kTileStrideB : n * kTileStrideA);
                const float* hi = h ? lo + 32 : reinterpret_cast<const float*>(smem + kOffZero);
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const floatx4 t = *reinterpret_cast<const floatx4*>(lo + 4 * q);
                    g[4 * q] = t[0]; g[4 * q + 1] = t[1]; g[4 * q + 2] = t[2]; g[4 * q + 3] = t[3];
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const floatx4 t = *reinterpret_cast<const floatx4*>(hi + 4 * q);
                    g[32 + 4 * q] = t[0]; g[32 + 4 * q + 1] = t[1]; g[32 + 4 * q + 2] = t[2]; g[32 + 4 * q + 3] = t[3];
                }
            }
            publish(diag_taken, l + 1);
            unsigned int sign_bit = 0x80000000u;
            asm volatile("" : "+s"(sign_bit));
            float sv = sig;
            walk_panel(sv, g, sign_bit);
            const unsigned long long m = __ballot(sv < 0.f);
            if (lane == 0) etaMask[I0] = m;
            {
                const int k = lane & 31;
                const int row = 32 * (k >> 4) + 8 * ((k & 15) >> 2) + 4 * h + (k & 3);
                etaF[((l & 3) << 6) + lane] = ((m >> row) & 1ull) ? 1.f : -1.f;
            }
            publish_in_order(eta_done, l + 1);
            __builtin_amdgcn_s_setprio(0);
            if (args_here()->status_out || args_here()->stats_out) {
                // walk statistics from the decision-time values: FAIL events (Alg. 2 line 7), near-tie decisions
                const float tau = threshold((I0 << 6) + lane);
                const float sg = sv + tau;
                const bool fail = __ballot(fabsf(sg) > 1.f) != 0ull;
                const float margin = 0.5f * fabsf(fminf(fmaxf(sg, -1.f), 1.f) - tau);
                const int near = __popcll(__ballot(margin < 1e-4f));
                if (args_here()->stats_out) {               // (non-negative floats: ordered as their bits)
                    atomicMin(events, __builtin_bit_cast(unsigned int, fminf(margin, 3.0e38f)));      // (a NaN counts as nothing)
                    atomicMax(events + 1, __builtin_bit_cast(unsigned int, fmaxf(fabsf(sg), 0.f)));
                }
                if (lane == 0) {
                    if (near) atomicAdd(events + 2, (unsigned int)near);
                    if (fail) atomicOr(events + 3, 1u);
                }
            }
        }
        __syncthreads();
    };
    chunk(std::integral_constant<int, 0>{});
    if constexpr (TWO) chunk(std::integral_constant<int, 1>{});

    // ------------------------------------------------------------------ output
    const CompressArgs& o = *args_here();
    int64_t seq = inst / o.blocks_per_seq;
    const int blk = (int)(inst - seq * o.blocks_per_seq);
    int64_t in_tok0 = seq * o.in_seq_stride + (int64_t)blk * b;
    int64_t out_tok0 = seq * o.out_seq_stride + (int64_t)blk * (b / 2);
    int64_t idx_out0 = seq * o.idx_out_seq_stride + (int64_t)blk * (b / 2);
    int64_t tok_base = o.idx_base + (int64_t)blk * b;
    int64_t signs0 = inst * b;
    if constexpr (TABLE) {
        const InstDesc& ds = *table_entry(o.desc, inst);
        seq = ds.seq; in_tok0 = ds.in_tok; out_tok0 = ds.out_tok; idx_out0 = ds.out_tok; signs0 = ds.in_tok;
        tok_base = in_tok0 - seq * o.v_seq_stride;
    }
    select_survivors(etaMask, b, wave, lane, keptIdx);
    __syncthreads();
    if (wave == 0) {
        if (o.signs_out)
            for (int p = 0; p < nP; ++p) o.signs_out[(size_t)signs0 + (p << 6) + lane] = ((etaMask[p] >> lane) & 1ull) ? 1 : -1;
    } else if (wave == 2 && lane == 0 && (o.status_out || o.stats_out)) {
        const float min_margin = __builtin_bit_cast(float, events[0]), max_sigma = __builtin_bit_cast(float, events[1]);
        const int n_margin = (int)events[2], any_fail = (int)events[3];
        const int sync_failed = *sync_err;
        if (o.status_out) {
            if (o.tree_mode) add_status(o.status_out + seq * o.status_stride + o.round, any_fail, sync_failed, n_margin);
            else o.status_out[inst] = (any_fail ? BKV_STATUS_FAIL : 0) | (sync_failed ? BKV_STATUS_INTERNAL : 0) | (n_margin << 8);
        }
        if (o.stats_out) {
            o.stats_out[2 * inst] = min_margin;
            o.stats_out[2 * inst + 1] = max_sigma;
        }
    }
    if (o.sticky_err && tid == 0 && *sync_err) atomicOr(o.sticky_err, BKV_STATUS_INTERNAL);
    const int half = b >> 1;
    auto src_token = [&](int r) -> int64_t {
        const int kept = keptIdx[r];
        return o.idx_in ? (int64_t)o.idx_in[in_tok0 + kept] : tok_base + kept;
    };
    {
        char* Ko = o.K_out ? o.K_out + out_tok0 * G::kRowBytes : nullptr;
        const bool do_v = o.V_out && o.V;
        const char* Vseq = do_v ? o.V + (size_t)seq * o.v_seq_stride * G::kRowBytes : nullptr;
        char* Vo = do_v ? o.V_out + out_tok0 * G::kRowBytes : nullptr;
        const int gs = tid & 15;
        constexpr int U = 8;
        for (int r0 = rg; r0 < half; r0 += RG * U) {
            uintx4 kraw[U], vraw[U];
            if (do_v) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int r = r0 + u * RG;
                    if (r < half) vraw[u] = *reinterpret_cast<const uintx4*>(Vseq + (size_t)src_token(r) * G::kRowBytes + gs * 16);
                }
            }
            if (Ko) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int r = r0 + u * RG;
                    if (r < half) kraw[u] = *reinterpret_cast<const uintx4*>(Kin + (size_t)keptIdx[r] * G::kRowBytes + gs * 16);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int r = r0 + u * RG;
                    if (r < half) __builtin_nontemporal_store(kraw[u], reinterpret_cast<uintx4*>(Ko + (size_t)r * G::kRowBytes + gs * 16));
                }
            }
            if (do_v) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int r = r0 + u * RG;
                    if (r < half) __builtin_nontemporal_store(vraw[u], reinterpret_cast<uintx4*>(Vo + (size_t)r * G::kRowBytes + gs * 16));
                }
            }
        }
    }
    for (int r = tid; r < half; r += kThreads) {
        if (o.w_out) o.w_out[out_tok0 + r] = o.w_out_val;
        if (o.idx_out) o.idx_out[idx_out0 + r] = (int32_t)src_token(r);
    }
}

template <typename T, int D, bool TWO, bool TABLE>
hipError_t launch_pair_t(const CompressArgs& a, int64_t n_inst, hipStream_t st) {
    const size_t lds = (size_t)kOffNa + (size_t)a.b * 4;
    auto kern = compress_pair_kernel<T, D, TWO, TABLE>;
    static thread_local size_t configured = 0;
    if (lds > configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        configured = lds;
    }
    return launch_timed(kProfCompress, n_inst * a.b, kern, dim3((unsigned)n_inst), dim3(kThreads), lds, st, a);
}

}  // namespace

hipError_t launch_compress_pair(int dtype, int d, CompressArgs& a, int64_t n_inst, hipStream_t st) {
    const bool two = a.b > 512, table = a.desc != nullptr;
    const int64_t n_cu = compute_units();
    // Raised / not, us.  Up to two blocks a compute unit: b = 640, 300 blocks 71 / 75, 512 85 / 90, b = 1024 116 / 119, 139 / 142.  Between two and three the last
    // blocks are alone on theirs: b = 640, 600 blocks 135 / 126, 832 172 / 160, 1024 198 / 196, 700 blocks 214 / 209.  With more it depends on how long the
    // second chunk walks: b = 576, 1200 blocks 213 / 197, 640 217 / 207, 704 4000 blocks 676 / 654; 768 800 blocks 174 / 179, 1200 239 / 239, 4000 737 / 719;
    // 896 1200 blocks 284 / 290, 4000 875 / 919, 1024 330 / 338, 1048 / 1058.
    a.raise_fetch = n_inst <= 2 * n_cu || (a.b >= 768 && n_inst > 3 * n_cu);
#define BKV_PAIR(TT, DD, TWO) return table ? launch_pair_t<TT, DD, TWO, true>(a, n_inst, st) : launch_pair_t<TT, DD, TWO, false>(a, n_inst, st)
    if (dtype == BKV_BF16 && d == 128) { if (two) { BKV_PAIR(__bf16, 128, true); } else { BKV_PAIR(__bf16, 128, false); } }
    if (dtype == BKV_F32 && d == 64 && !two) { BKV_PAIR(float, 64, false); }
#undef BKV_PAIR
    return hipErrorInvalidValue;
}

}  // namespace bkv
