// What the two halving kernels (compress.hip, compress_pair.hip) share: the LDS layout of key rows, the walk over one
// 64-token panel, the hand-over counters.
#pragma once
#include "bkv_device.h"
#include "bkv_host.h"

namespace bkv {

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;

template <typename T, int D> struct Geo {
    static constexpr int kRowBytes = D * (int)sizeof(T);
    static constexpr int kLdsRow = kRowBytes;               // rows are packed; 16-byte slices are permuted per row instead
    static constexpr int kGroups = kRowBytes / 32;          // k-groups of 32 bytes per row
    static constexpr int kSlices = kRowBytes / 16;          // 16-byte slices per row
    // Slice s of LDS row r is stored at slice position s ^ key(r).  Sixteen consecutive rows reading the same
    // logical slice (an MFMA operand fetch) then touch sixteen different groups of four banks, and so do the
    // slices of one row (staging, gathers): no padding bytes, no bank conflicts.  key(r) = key(r + 16).
    static __device__ __forceinline__ int key(int row) { return kRowBytes >= 256 ? (row & 15) : ((row >> 1) & (kSlices - 1)); }
    static __device__ __forceinline__ int slice_off(int row, int slice) { return (slice ^ key(row)) << 4; }
};
// cs0 / cs1: per-lane partial sums for columns n / 32+n over this lane half's rows.  Returns, in lane (n, h), the
// full sum of column 32*h + n: one half-wave swap (lanes 32..63 of cs0 <-> lanes 0..31 of cs1) and one add.
__device__ __forceinline__ float halves_sum(float cs0, float cs1) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(cs0), __float_as_uint(cs1), false, false);
    return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

// One decision of the walk (Alg. 2 lines 6-9 for token j of the panel).  Every lane tests the sign of its sigma
// (which carries the threshold, see the kernel); the compare mask is then read back as data by the vector unit:
// bit j of it, sign-extended, becomes the -1/+1 that multiplies row j of the diagonal tile.  No scalar-unit hop
// on the chain: four dependent vector instructions per step.  A vector instruction that reads a scalar register
// written by the vector instruction just before it needs two wait states on this hardware, hence the s_nop.
// Lanes <= j hold g[j] = 0, so their sigma stays at its decision-time value.
// Eight consecutive steps per asm statement, so that nothing is scheduled into the chain.
template <int B>
__device__ __forceinline__ void walk_steps8(float& sv, const float (&g)[64], unsigned int sign_bit) {
    int t;
    if constexpr (B < 32)
        asm volatile("v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_lo, %11, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %3\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_lo, %12, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %4\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_lo, %13, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %5\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_lo, %14, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %6\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_lo, %15, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %7\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_lo, %16, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %8\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_lo, %17, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %9\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_lo, %18, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %10"
                     : "+&v"(sv), "=&v"(t)
                     : "s"(sign_bit), "v"(g[B]), "v"(g[B + 1]), "v"(g[B + 2]), "v"(g[B + 3]), "v"(g[B + 4]), "v"(g[B + 5]), "v"(g[B + 6]), "v"(g[B + 7]),
                       "n"(B), "n"(B + 1), "n"(B + 2), "n"(B + 3), "n"(B + 4), "n"(B + 5), "n"(B + 6), "n"(B + 7)
                     : "vcc");
    else
        asm volatile("v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_hi, %11, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %3\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_hi, %12, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %4\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_hi, %13, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %5\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_hi, %14, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %6\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_hi, %15, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %7\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_hi, %16, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %8\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_hi, %17, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %9\n\t"
                     "v_cmp_le_f32 vcc, 0, %0\n\ts_nop 1\n\tv_bfe_i32 %1, vcc_hi, %18, 1\n\tv_and_or_b32 %1, %1, %2, 1.0\n\tv_fmac_f32 %0, %1, %10"
                     : "+&v"(sv), "=&v"(t)
                     : "s"(sign_bit), "v"(g[B]), "v"(g[B + 1]), "v"(g[B + 2]), "v"(g[B + 3]), "v"(g[B + 4]), "v"(g[B + 5]), "v"(g[B + 6]), "v"(g[B + 7]),
                       "n"(B - 32), "n"(B - 31), "n"(B - 30), "n"(B - 29), "n"(B - 28), "n"(B - 27), "n"(B - 26), "n"(B - 25)
                     : "vcc");
    // per step: sigma >= 0 -> bit set, factor -1 (eta = -1); sigma < 0 -> factor +1
}
__device__ __forceinline__ void walk_panel(float& sv, const float (&g)[64], unsigned int sign_bit) {
    walk_steps8<0>(sv, g, sign_bit);  walk_steps8<8>(sv, g, sign_bit);  walk_steps8<16>(sv, g, sign_bit); walk_steps8<24>(sv, g, sign_bit);
    walk_steps8<32>(sv, g, sign_bit); walk_steps8<40>(sv, g, sign_bit); walk_steps8<48>(sv, g, sign_bit); walk_steps8<56>(sv, g, sign_bit);
}

// Progress counters in LDS (one writer each, values only grow): a wavefront publishes with a release store and
// waits with a bounded poll.  Every wait is for an event that only depends on earlier events of the same block, and
// all eight wavefronts are resident, so the polls end; the bound turns a logic error into a status bit instead of
// a hang.
constexpr int kSpinLimit = 1 << 16;
// The fences name LDS only: a wavefront with global loads or stores in flight (look-ahead touches, dumps) must
// not wait for them here.
__device__ __forceinline__ void publish(int* counter, int value) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __hip_atomic_store(counter, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// The same for a hand-over on the walk's critical path, where counter and data are both in LDS and were written by
// this wavefront just before: LDS serves a wavefront's requests in order, so the counter cannot become visible before
// the data, and the wavefront need not wait for its own stores to finish first.  (The fence only keeps the compiler
// from moving the stores.)
__device__ __forceinline__ void publish_in_order(int* counter, int value) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __hip_atomic_store(counter, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <bool EAGER = false>
__device__ __forceinline__ void await(int* counter, int value, int* err) {
    for (int it = 0; it < kSpinLimit; ++it) {
        const int seen = __builtin_amdgcn_readfirstlane(__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
        if (seen >= value) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            return;
        }
        if (!EAGER) __builtin_amdgcn_s_sleep(1);          // waits on the walk's critical path poll back to back
    }
    __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The kernel's arguments, read where they are used: an opaque pointer keeps them out of registers in between.
__device__ __forceinline__ const CompressArgs* args_here() {
    unsigned long long p = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return (const CompressArgs*)(const __attribute__((address_space(4))) CompressArgs*)p;
}

// Output step (Alg. 2 lines 12-16 + strict n/2): every wavefront handles the panels p = wave, wave + 8, ...: minority
// sign ('+' on ties), then exactly b/2 survivors = the minority class plus the lowest-index majority tokens, ascending.
__device__ __forceinline__ void select_survivors(const unsigned long long* etaMask, int b, int wave, int lane, int* keptIdx) {
    const int nP = b >> 6;
    // lane q < nP (nP <= 16) carries the counts of panel q; prefix sums run over the first row of 16 lanes
    auto row_scan = [](int x) -> int {                                // inclusive prefix sum inside a row of 16 lanes
        x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);   // row_shr:1, zero fill
        x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);   // row_shr:2
        x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);   // row_shr:4
        x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);   // row_shr:8
        return x;
    };
    int plus_q = 0;
    if (lane < nP) plus_q = __popcll(etaMask[lane]);
    const int n_plus = __builtin_amdgcn_readlane(row_scan(plus_q), 15);
    const bool plus_is_minority = n_plus <= b - n_plus;               // tie -> '+'
    const int n_min = plus_is_minority ? n_plus : b - n_plus;
    const int need = b / 2 - n_min;                                   // majority tokens to add, lowest index first
    const int min_q = (lane < nP) ? (plus_is_minority ? plus_q : 64 - plus_q) : 0;
    const int maj_q = (lane < nP) ? 64 - min_q : 0;
    const int maj_before_q = row_scan(maj_q) - maj_q;
    const int kept_q = min_q + max(0, min(maj_q, need - maj_before_q));
    const int kept_before_q = row_scan(kept_q) - kept_q;
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int p = wave; p < nP; p += kWaves) {
        const int maj_before = __builtin_amdgcn_readlane(maj_before_q, p);
        const int kept_before = __builtin_amdgcn_readlane(kept_before_q, p);
        const unsigned long long mv = etaMask[p];
        const unsigned long long m = ((unsigned long long)__builtin_amdgcn_readfirstlane((unsigned int)(mv >> 32)) << 32) |
                                     (unsigned int)__builtin_amdgcn_readfirstlane((unsigned int)mv);
        const unsigned long long minm = plus_is_minority ? m : ~m;
        const unsigned long long majm = ~minm;
        const int my_rank = maj_before + __popcll(majm & lt);
        const bool keep = ((minm >> lane) & 1ull) || (my_rank < need);
        const unsigned long long km = __ballot(keep);
        if (keep) keptIdx[kept_before + __popcll(km & lt)] = (p << 6) + lane;
    }
}

// Tree mode: the events of one block join the status word of its sequence and round.
__device__ __forceinline__ void add_status(int* dst, int any_fail, int sync_failed, int n_margin) {
    if (any_fail) atomicOr(dst, BKV_STATUS_FAIL);
    if (sync_failed) atomicOr(dst, BKV_STATUS_INTERNAL);
    if (!n_margin) return;
    // the count lives in bits 8..30 and saturates there: bit 31 is never set.  Margin decisions are rare, so the
    // compare-and-swap loop (it ends when no other block updates the word in between) is next to never entered twice.
    int seen = __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (;;) {
        const int cnt = min((seen >> 8) + n_margin, 0x7fffff);
        const int want = (seen & 0xff) | (cnt << 8);
        const int prev = atomicCAS(dst, seen, want);
        if (prev == seen) break;
        seen = prev;
    }
}

// The same without a status word that is 0 before the launch (clearing it was a launch of its own, 3.3 us in front of trees that take 20 to
// 60): every block of a sequence leaves its events in a word of its own, under the launch's label, waits until that has arrived
// and reads all words of the sequence; the one whose word arrives last finds them all and writes the sum.  (Blocks that arrive
// together may all find them: they write the same.)  Nothing that the memory held before means anything: 51 bits of a word are the
// label, which no other launch of the process has.
constexpr int kLabelShift = 13;                            // FAIL, INTERNAL, near ties of a block (at most 1024)
__device__ __forceinline__ void put_status_word(unsigned long long* word, unsigned long long label, int any_fail, int sync_failed, int n_margin) {
    const unsigned long long x = label << kLabelShift | (unsigned int)n_margin << 2 | (sync_failed ? 2u : 0u) | (any_fail ? 1u : 0u);
    __hip_atomic_store(word, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Called by the wavefront that has put its block's word.  n: at most kStatusWords.  Workgroups start in order, so nearly every block finds
// the last words missing and leaves after one load; the others follow together.  Words that lie in the
// weights (weight: their value, else 0) are replaced by them once all have been seen: a block that finds one gone knows that another has
// seen all.
__device__ __forceinline__ void sum_status_words(unsigned long long* words, int n, float weight, unsigned long long label, int lane, int32_t* status) {
    constexpr int kSteps = kStatusWords / 64;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int front = max(n - 64, 0);                       // words in front of the last 64
    bool there = true;
    unsigned int events = 0, near = 0;
    auto load = [&](int i) { return __hip_atomic_load(words + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    auto take = [&](unsigned long long x, bool counts) {
        there &= x >> kLabelShift == label;
        if (counts) { events |= (unsigned int)x & 3u; near += ((unsigned int)x & ((1u << kLabelShift) - 1u)) >> 2; }
    };
    take(load(min(front + lane, n - 1)), front + lane < n);
    if (__ballot(!there) != 0ull) return;
    if (front > 0) {
        unsigned long long x[kSteps - 1];
#pragma unroll
        for (int k = 0; k < kSteps - 1; ++k) x[k] = load(min(64 * k + lane, front - 1));
#pragma unroll
        for (int k = 0; k < kSteps - 1; ++k) take(x[k], 64 * k + lane < front);
        if (__ballot(!there) != 0ull) return;
    }
    const int any_fail = __ballot(events & 1u) != 0ull, sync_failed = __ballot(events & 2u) != 0ull;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) near += __shfl_xor(near, o);
    if (lane == 0) *status = (any_fail ? BKV_STATUS_FAIL : 0) | (sync_failed ? BKV_STATUS_INTERNAL : 0) | (int)(min(near, 0x7fffffu) << 8);
    if (weight > 0.f) {
        const unsigned long long w = __float_as_uint(weight), both = w << 32 | w;
        for (int i = lane; i < n; i += 64) __hip_atomic_store(words + i, both, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace bkv
