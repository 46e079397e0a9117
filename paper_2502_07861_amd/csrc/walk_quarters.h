// The walk over one panel of 64 tokens for the kernel with one block per compute unit: decisions travel by DPP.
#pragma once
#include "compress_device.h"

namespace bkv {

// Alg. 2 lines 6-9.  Token j's sigma (which carries the threshold, see the kernels) is
// final once the tokens before it are decided; its sign is the decision, and every later token's sigma gets +-g_jl.
//
// Four quarters of 16 tokens.  In every lane s[k] is sigma of token 16 k + lane % 16: each row of 16 lanes carries all 64
// tokens, so a decision only has to travel inside a row, which DPP does as part of the multiply-add that uses it:
//     x = +-1 with the sign of s              v_bfi_b32
//     two wait states                         (a DPP operand may not be read sooner after a vector instruction wrote it)
//     s -= x[lane j of the row] * g           v_fmac_f32 with row_newbcast:j
// four issue slots of 4 clocks a decision.  The wait states take the multiply-adds for the quarters behind: quarter 0 those of
// 1 and 2, quarter 1 those of 2 and, with the signs of quarter 0, of 3, quarter 2 the rest of 3.  259 slots a panel,
// where walk_panel's compare mask takes six a decision; one wavefront alone on its compute unit, the tile's reads from LDS included,
// 1404 clocks a panel against 1780.  It reads 40 pieces of 16 bytes a lane instead of 16: with two blocks on a compute unit, where LDS is
// the scarcer thing, that costs what the chain gains (128 x 131072 tokens, blocks of 1024: 6.34 ms, 6.40 this way), and the pair
// kernel keeps walk_panel.
// Every s[k] receives eta_j g_jl in the order of j and nothing else.  Lanes l <= j of j's own quarter hold g = 0: s[k] keeps the
// value it had at decision time.  s never is -0 (it starts as 0 - threshold, and a sum is -0 only if both terms are), so its
// sign bit says whether s < 0.  Weights that overflow make it a NaN (inf - inf), which this hardware makes with the sign bit set: it
// decides as +, as walk_panel's compare takes it, and is published as - by both kernels (it is not < 0).
// Eight decisions per asm statement, so that nothing is scheduled into the chain.  What a statement reads by DPP has been
// written two wait states before, whatever instruction precedes the statement.
#define BKV_ADD(ACC, X, G, L) "v_fmac_f32_dpp %[" ACC "], -%[" X "], %[" G "] row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t"
#define BKV_SIGN(X) "v_bfi_b32 %[" X "], %[m], 1.0, %[s]\n\t"
#define BKV_STEP(X, FILL, G, L) BKV_SIGN(X) FILL BKV_ADD("s", X, G, L)
#define BKV_WAIT1 "s_nop 0\n\t"
#define BKV_WAIT2 "s_nop 1\n\t"
#define BKV_IN8(N, P) [N##0] "v"((P)[0]), [N##1] "v"((P)[1]), [N##2] "v"((P)[2]), [N##3] "v"((P)[3]), [N##4] "v"((P)[4]), [N##5] "v"((P)[5]), \
                      [N##6] "v"((P)[6]), [N##7] "v"((P)[7])
// lanes L0..L7 decide; F0..F7 fill their wait states; LAST: the eighth one's own multiply-add (none in lane 15: nobody is behind it)
#define BKV_EIGHT(F0, F1, F2, F3, F4, F5, F6, F7, LAST, TAIL, L0, L1, L2, L3, L4, L5, L6)                                           \
    BKV_STEP("x", F0, "c0", L0) BKV_STEP("y", F1, "c1", L1) BKV_STEP("x", F2, "c2", L2) BKV_STEP("y", F3, "c3", L3)                  \
    BKV_STEP("x", F4, "c4", L4) BKV_STEP("y", F5, "c5", L5) BKV_STEP("x", F6, "c6", L6) BKV_SIGN("y") F7 LAST TAIL
// p and q += the decision before, L
#define BKV_BOTH(X, I, L) BKV_ADD("p", X, "a" #I, L) BKV_ADD("q", X, "b" #I, L)
#define BKV_EIGHT_BOTH(LAST, L0, L1, L2, L3, L4, L5, L6, L7)                                                                        \
    BKV_EIGHT(BKV_WAIT2, BKV_BOTH("x", 0, L0), BKV_BOTH("y", 1, L1), BKV_BOTH("x", 2, L2), BKV_BOTH("y", 3, L3), BKV_BOTH("x", 4, L4),     \
              BKV_BOTH("y", 5, L5), BKV_BOTH("x", 6, L6), LAST, BKV_BOTH("y", 7, L7), L0, L1, L2, L3, L4, L5, L6)
// p += the decision before, L; q += the decision of lane M of an earlier quarter (z)
#define BKV_MIX(X, I, L, J, M) BKV_ADD("p", X, "a" #I, L) BKV_ADD("q", "z", "b" #J, M)
#define BKV_EIGHT_MIX(LAST, L0, L1, L2, L3, L4, L5, L6, L7)                                                                         \
    BKV_EIGHT(BKV_WAIT1 BKV_ADD("q", "z", "b0", L0), BKV_MIX("x", 0, L0, 1, L1), BKV_MIX("y", 1, L1, 2, L2), BKV_MIX("x", 2, L2, 3, L3),  \
              BKV_MIX("y", 3, L3, 4, L4), BKV_MIX("x", 4, L4, 5, L5), BKV_MIX("y", 5, L5, 6, L6), BKV_MIX("x", 6, L6, 7, L7), LAST,        \
              BKV_ADD("p", "y", "a7", L7), L0, L1, L2, L3, L4, L5, L6)
// q += sixteen decisions of an earlier quarter (z), or those of this one (F: none in the first wait states, the last two behind)
#define BKV_TWO(X, G, L, H, M) BKV_ADD("q", X, G, L) BKV_ADD("q", X, H, M)

// x[.] of quarter K's rows: c: of the deciding quarter, a and b: of the two that are served.  Returns the sixteen signs so far.
template <int H>
__device__ __forceinline__ float walk_both(float& s, float& p, float& q, const float* c, const float* a, const float* b, unsigned int m) {
    float x, y;
    if constexpr (H == 0)
        asm volatile(BKV_EIGHT_BOTH(BKV_ADD("s", "y", "c7", 7), 0, 1, 2, 3, 4, 5, 6, 7)
                     : [s] "+&v"(s), [p] "+&v"(p), [q] "+&v"(q), [x] "=&v"(x), [y] "=&v"(y) : [m] "s"(m), BKV_IN8(c, c), BKV_IN8(a, a), BKV_IN8(b, b));
    else
        asm volatile(BKV_EIGHT_BOTH("", 8, 9, 10, 11, 12, 13, 14, 15)
                     : [s] "+&v"(s), [p] "+&v"(p), [q] "+&v"(q), [x] "=&v"(x), [y] "=&v"(y) : [m] "s"(m), BKV_IN8(c, c + 8), BKV_IN8(a, a + 8), BKV_IN8(b, b + 8));
    return y;
}
template <int H>
__device__ __forceinline__ float walk_mix(float& s, float& p, float& q, float z, const float* c, const float* a, const float* b, unsigned int m) {
    float x, y;
    if constexpr (H == 0)
        asm volatile(BKV_EIGHT_MIX(BKV_ADD("s", "y", "c7", 7), 0, 1, 2, 3, 4, 5, 6, 7)
                     : [s] "+&v"(s), [p] "+&v"(p), [q] "+&v"(q), [x] "=&v"(x), [y] "=&v"(y) : [z] "v"(z), [m] "s"(m), BKV_IN8(c, c), BKV_IN8(a, a), BKV_IN8(b, b));
    else
        asm volatile(BKV_EIGHT_MIX("", 8, 9, 10, 11, 12, 13, 14, 15)
                     : [s] "+&v"(s), [p] "+&v"(p), [q] "+&v"(q), [x] "=&v"(x), [y] "=&v"(y) : [z] "v"(z), [m] "s"(m), BKV_IN8(c, c + 8), BKV_IN8(a, a + 8), BKV_IN8(b, b + 8));
    return y;
}
// quarter 2: its first half takes the signs of quarter 1 (z) to the last quarter, its second half its own
template <int H>
__device__ __forceinline__ void walk_late(float& s, float& q, float z, const float* c, const float* a, unsigned int m) {
    float x, y;
    if constexpr (H == 0)
        asm volatile(BKV_EIGHT(BKV_WAIT1 BKV_ADD("q", "z", "a0", 0), BKV_TWO("z", "a1", 1, "a2", 2), BKV_TWO("z", "a3", 3, "a4", 4), BKV_TWO("z", "a5", 5, "a6", 6),
                               BKV_TWO("z", "a7", 7, "b0", 8), BKV_TWO("z", "b1", 9, "b2", 10), BKV_TWO("z", "b3", 11, "b4", 12), BKV_TWO("z", "b5", 13, "b6", 14),
                               BKV_ADD("s", "y", "c7", 7), BKV_ADD("q", "z", "b7", 15), 0, 1, 2, 3, 4, 5, 6)
                     : [s] "+&v"(s), [q] "+&v"(q), [x] "=&v"(x), [y] "=&v"(y) : [z] "v"(z), [m] "s"(m), BKV_IN8(c, c), BKV_IN8(a, a), BKV_IN8(b, a + 8));
    else
        asm volatile(BKV_EIGHT(BKV_WAIT2, BKV_TWO("x", "a0", 0, "a1", 1), BKV_TWO("y", "a2", 2, "a3", 3), BKV_TWO("x", "a4", 4, "a5", 5),
                               BKV_TWO("y", "a6", 6, "a7", 7), BKV_TWO("x", "b0", 8, "b1", 9), BKV_TWO("y", "b2", 10, "b3", 11), BKV_TWO("x", "b4", 12, "b5", 13),
                               "", BKV_TWO("y", "b6", 14, "b7", 15), 8, 9, 10, 11, 12, 13, 14)
                     : [s] "+&v"(s), [q] "+&v"(q), [x] "=&v"(x), [y] "=&v"(y) : [m] "s"(m), BKV_IN8(c, c + 8), BKV_IN8(a, a), BKV_IN8(b, a + 8));
}
template <int H>
__device__ __forceinline__ void walk_plain(float& s, const float* c, unsigned int m) {
    float x, y;
    if constexpr (H == 0)
        asm volatile(BKV_EIGHT(BKV_WAIT2, BKV_WAIT2, BKV_WAIT2, BKV_WAIT2, BKV_WAIT2, BKV_WAIT2, BKV_WAIT2, BKV_WAIT2, BKV_ADD("s", "y", "c7", 7), "", 0, 1, 2, 3, 4, 5, 6)
                     : [s] "+&v"(s), [x] "=&v"(x), [y] "=&v"(y) : [m] "s"(m), BKV_IN8(c, c));
    else
        asm volatile(BKV_EIGHT(BKV_WAIT2, BKV_WAIT2, BKV_WAIT2, BKV_WAIT2, BKV_WAIT2, BKV_WAIT2, BKV_WAIT2, "", "", "", 8, 9, 10, 11, 12, 13, 14)
                     : [s] "+&v"(s), [x] "=&v"(x), [y] "=&v"(y) : [m] "s"(m), BKV_IN8(c, c + 8));
}
#undef BKV_TWO
#undef BKV_EIGHT_MIX
#undef BKV_MIX
#undef BKV_EIGHT_BOTH
#undef BKV_BOTH
#undef BKV_EIGHT
#undef BKV_IN8
#undef BKV_WAIT2
#undef BKV_WAIT1
#undef BKV_STEP
#undef BKV_SIGN
#undef BKV_ADD

// The tile of a panel on its way through the walk.  load(m, k, q): g_{16 m + 4 q + r, 16 k + lane % 16}, r = 0..3 (0 unless the row
// is before the column).  walk_begin may be called while sigma is still being completed; walk_quarters calls taken() when the
// whole tile is in registers, and returns this lane's sigma: that of token `lane` at decision time (its sign is the decision).
struct WalkStart { float c[16], a[16], b[16]; };
template <typename Load>
__device__ __forceinline__ void walk_get(Load load, int m, int k, int first, int last, float (&g)[16]) {
#pragma unroll
    for (int q = first; q < last; ++q) {
        const floatx4 t = load(m, k, q);
        g[4 * q] = t[0]; g[4 * q + 1] = t[1]; g[4 * q + 2] = t[2]; g[4 * q + 3] = t[3];
    }
}
template <typename Load>
__device__ __forceinline__ void walk_begin(WalkStart& t, Load load) {
    walk_get(load, 0, 0, 0, 2, t.c); walk_get(load, 0, 1, 0, 2, t.a); walk_get(load, 0, 2, 0, 2, t.b);
    walk_get(load, 0, 0, 2, 4, t.c); walk_get(load, 0, 1, 2, 4, t.a); walk_get(load, 0, 2, 2, 4, t.b);
    __builtin_amdgcn_sched_barrier(0);
}
template <typename Load, typename Taken>
__device__ __forceinline__ float walk_quarters(float (&s)[4], int lane, const WalkStart& t, Load load, Taken taken) {
    unsigned int m = 0x7fffffffu;
    asm volatile("" : "+s"(m));                                    // stays in a scalar register
    float c1[16], a1[16], b1[16], c2[16], a2[16], b2[16], c3[16];
    __builtin_amdgcn_sched_barrier(0);
    walk_both<0>(s[0], s[1], s[2], t.c, t.a, t.b, m);
    __builtin_amdgcn_sched_barrier(0);
    walk_get(load, 1, 1, 0, 2, c1); walk_get(load, 1, 2, 0, 2, a1); walk_get(load, 0, 3, 0, 2, b1);
    walk_get(load, 1, 1, 2, 4, c1); walk_get(load, 1, 2, 2, 4, a1); walk_get(load, 0, 3, 2, 4, b1);
    __builtin_amdgcn_sched_barrier(0);
    const float z0 = walk_both<1>(s[0], s[1], s[2], t.c, t.a, t.b, m);
    walk_mix<0>(s[1], s[2], s[3], z0, c1, a1, b1, m);
    __builtin_amdgcn_sched_barrier(0);
    walk_get(load, 2, 2, 0, 2, c2); walk_get(load, 1, 3, 0, 4, a2); walk_get(load, 2, 2, 2, 4, c2); walk_get(load, 2, 3, 0, 4, b2);
    walk_get(load, 3, 3, 0, 4, c3);
    __builtin_amdgcn_sched_barrier(0);
    const float z1 = walk_mix<1>(s[1], s[2], s[3], z0, c1, a1, b1, m);
    walk_late<0>(s[2], s[3], z1, c2, a2, m);
    __builtin_amdgcn_sched_barrier(0);
    taken();
    __builtin_amdgcn_sched_barrier(0);
    walk_late<1>(s[2], s[3], z1, c2, b2, m);
    walk_plain<0>(s[3], c3, m);
    walk_plain<1>(s[3], c3, m);
    const float lo = (lane & 16) ? s[1] : s[0], hi = (lane & 16) ? s[3] : s[2];
    return (lane & 32) ? hi : lo;
}

}  // namespace bkv
