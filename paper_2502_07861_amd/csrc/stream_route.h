// Alg. 1 token by token: buckets, and what one token does to a sequence's state before the halvings.  Used by a launch of its own
// and in front of the halvings of round 0.
#pragma once
#include "bkv_device.h"
#include "bkv_host.h"

namespace bkv {

constexpr int kSlots = 512;
constexpr int kDenSlot = 0;
constexpr int kNumSlot0 = 256;
constexpr int kDropSlot = 511;
constexpr int kBucketMin = -60, kBucketMax = 60;      // 4^i stays a normal fp32 number

// Bucket of a value row with |v|^2 = x: the smallest i with 2^i >= |v| (Alg. 1 line 5), from the exponent of x,
// clamped to [kBucketMin, kBucketMax].  False: the row belongs to no bucket (zero or non-finite norm).
__device__ __forceinline__ bool bucket_of(float x, int& i) {
    if (!(x > 0.f && x < __builtin_inff())) return false;
    int e;
    const float m = frexpf(x, &e);                    // x = m 2^e, 1/2 <= m < 1
    const int ee = (m == 0.5f) ? e - 1 : e;           // smallest integer with 2^ee >= x
    i = ee >= 0 ? (ee + 1) / 2 : ee / 2;              // ceil(ee / 2): smallest i with 4^i >= x
    i = min(max(i, kBucketMin), kBucketMax);
    return true;
}

constexpr int kFreeRegion = INT32_MIN;

// Lines 4-12 of Alg. 1 for one token per sequence, up to the halvings themselves.  One wavefront per sequence:
//  * |v|^2, the running maximum and the erase limit (line 8): regions whose bucket has 4^i <= limit are given back;
//  * the token's bucket (line 5) -> its region (a free one on the bucket's first token) -> the row goes to the tail of
//    the region with weight 1 (line 7 feeds MR-Numerator_i); the key goes to the denominator region (line 11);
//  * the carry loop of Alg. 3 for both instances as a table: round r of this token halves the last `b` stored tokens
//    of the region as they will stand after the rounds before it (each takes b/2 away), draws from the instance's
//    stream at level r, block number = blocks that reached level r before.
// Lane l < regions looks after region l.
// Returns (in lane 0) the numerator's carry of round 0.
template <typename T, int D>
__device__ __forceinline__ InstDesc stream_route_token(const StreamState& s, const char* k, const char* v, int32_t j, int64_t seq, int lane) {
    constexpr int RB = D * (int)sizeof(T);
    constexpr int SL = RB / 16;
    const int R = s.regions, b = s.b, half = s.b / 2, Tn = s.T;
    uintx4 kraw = {0u, 0u, 0u, 0u}, vraw = {0u, 0u, 0u, 0u};
    if (lane < SL) {
        kraw = *reinterpret_cast<const uintx4*>(k + (size_t)seq * RB + lane * 16);
        vraw = *reinterpret_cast<const uintx4*>(v + (size_t)seq * RB + lane * 16);
    }
    // everything that is read of the state, in one trip to memory (behind the first store the compiler would start another)
    float vm = __uint_as_float(s.vmax2[seq]);
    int bk = lane < R ? s.bucket[seq * R + lane] : kFreeRegion;
    int my_cnt = lane < R ? s.cnt[seq * (R + 1) + lane] : 0;
    int my_jj = lane < R ? s.jj[seq * (R + 1) + lane] : 0;
    int pos_d = s.cnt[seq * (R + 1) + R];
    const int seen_d = s.jj[seq * (R + 1) + R] + 1;
    const float x = __shfl(group_sum<SL>(Elem<T>::dot(vraw, vraw)), 0);          // |v|^2, fp32
    if (x < __builtin_inff() && x > vm) {
        vm = x;
        if (lane == 0) s.vmax2[seq] = __float_as_uint(vm);
    }
    const float limit = s.erase2 > 0.f ? s.erase2 * vm : 0.f;

    // ---- line 8: erase the negligible buckets (lane l keeps region l's bucket and counters in registers; they are
    // written back once, at the end)
    const bool gone = bk != kFreeRegion && ldexpf(1.f, 2 * bk) <= limit;
    unsigned long long erased = __ballot(gone);
    while (erased) {
        const int e = __ffsll((long long)erased) - 1;
        erased &= erased - 1;
        const int c = __shfl(my_cnt, e);
        float* w = s.wn + (size_t)(seq * R + e) * s.cap_n;
        for (int t = lane; t < c; t += 64) w[t] = 0.f;
    }
    if (gone) { bk = kFreeRegion; my_cnt = 0; my_jj = 0; }

    // ---- lines 5-7: the token's bucket and region
    int i = 0;
    int reg = 0;
    bool take = bucket_of(x, i) && !(ldexpf(1.f, 2 * i) <= limit);      // a token of a negligible bucket is dropped at once
    if (take) {
        const unsigned long long hit = __ballot(bk == i);
        if (hit) reg = __ffsll((long long)hit) - 1;
        else {
            const unsigned long long vacant = __ballot(lane < R && bk == kFreeRegion);
            if (vacant) {
                reg = __ffsll((long long)vacant) - 1;
                if (lane == reg) bk = i;                         // counters of a free region are 0
            } else {
                take = false;
                if (lane == 0) atomicOr(s.err, BKV_STREAM_NO_REGION);
            }
        }
    }
    int pos_n = __shfl(my_cnt, reg);
    if (take && pos_n >= s.cap_n) {
        take = false;
        if (lane == 0) atomicOr(s.err, BKV_STREAM_NUM_FULL);
    }
    int carries_n = 0, blocks_n = 0;
    if (take) {
        const size_t at = (size_t)(seq * R + reg) * s.cap_n + pos_n;
        if (lane < SL) {
            *reinterpret_cast<uintx4*>(s.Kn + at * RB + lane * 16) = kraw;
            *reinterpret_cast<uintx4*>(s.Vn + at * RB + lane * 16) = vraw;
        }
        if (lane == 0) { s.wn[at] = 1.f; s.on[at] = j; }
        const int seen = __shfl(my_jj, reg) + 1;
        pos_n += 1;
        if (lane == reg) { my_cnt = pos_n; my_jj = seen; }
        if (Tn > 0 && seen % b == 0) {
            blocks_n = seen / b;
            carries_n = min(Tn, __ffs(blocks_n));               // rounds r < T with blocks_n divisible by 2^r
        }
    }
    if (lane < R) {
        s.bucket[seq * R + lane] = bk;
        s.cnt[seq * (R + 1) + lane] = my_cnt;
        s.jj[seq * (R + 1) + lane] = my_jj;
    }

    // ---- line 11: the key alone goes to MR-Denominator
    int carries_d = 0, blocks_d = 0;
    if (pos_d >= s.cap_d) {
        if (lane == 0) atomicOr(s.err, BKV_STREAM_DEN_FULL);
    } else {
        const size_t at = (size_t)seq * s.cap_d + pos_d;
        if (lane < SL) *reinterpret_cast<uintx4*>(s.Kd + at * RB + lane * 16) = kraw;
        if (lane == 0) {
            s.wd[at] = 1.f; s.od[at] = j;
            s.cnt[seq * (R + 1) + R] = pos_d + 1;
            s.jj[seq * (R + 1) + R] = seen_d;
        }
        pos_d += 1;
        if (Tn > 0 && seen_d % b == 0) {
            blocks_d = seen_d / b;
            carries_d = min(Tn, __ffs(blocks_d));
        }
    }

    // ---- the carries of this token, round by round (lanes 0..T-1: numerator, 32..32+T-1: denominator)
    const int r = lane & 31, kind = lane >> 5;
    InstDesc ds;
    {
        ds.in_tok = ds.out_tok = 0; ds.stream = ds.ctr0 = 0; ds.seq = (int32_t)seq; ds.valid = 0; ds.rvalue2 = 0.f; ds.region = 0;
        const int carries = r < Tn ? (kind ? carries_d : carries_n) : 0;
        if (r < carries) {
            const int64_t region0 = kind ? seq * s.cap_d : (seq * R + reg) * s.cap_n;
            const int64_t first = (kind ? pos_d : pos_n) - (int64_t)r * half - b;
            const uint64_t slot = kind ? (uint64_t)kDenSlot : (uint64_t)(kNumSlot0 + i);
            ds.in_tok = region0 + first;
            ds.out_tok = ds.in_tok;                              // in place (CompressArgs::carry_w)
            ds.stream = 64ull * ((uint64_t)(s.seq_base + seq) * kSlots + slot) + (uint64_t)r;
            ds.ctr0 = (uint64_t)(((kind ? blocks_d : blocks_n) >> r) - 1) * (uint64_t)b;
            ds.valid = 1;
            ds.rvalue2 = kind ? 0.f : ldexpf(1.f, 2 * i);
            ds.region = kind ? R : reg;
        }
        if (r < Tn) s.desc[((int64_t)r * 2 + kind) * s.n_seq + seq] = ds;
    }
    return ds;
}

}  // namespace bkv
