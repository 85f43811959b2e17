// fp32 decode on the fp16 matrix cores (v_mfma_f32_16x16x32_f16), shared by
// the k_mfma_f16x3*.hip translation units that instantiate it.
//
// Same computation and tiling as the fp32 family (PIC, Sec. 3.1 and App. A;
// tiles and LDS boxes in decode_common.h): fp32 weights, fp32 activations,
// binary32 accuracy.  Every product w * x that feeds a matrix core is formed
// from fp16 parts:
//
//   w = wh + wl + O(2^-23 |w|),  x = xh + xl + O(2^-23 |x|),
//   wh = fp16(w), wl = fp16(w - wh) (likewise x), all rounded to nearest,
//   w * x = wh * xh + wh * xl + wl * xh + O(2^-22 |w x|),
//
// with products of fp16 numbers exact in the fp32 accumulator.  (Relative to
// a layer's sum the split costs 7.5e-8, root mean square, whatever the width;
// a chain of binary32 multiply-adds 5.4e-8 over 8 inputs, 1.0e-7 over 33,
// 1.4e-7 over 64.  So the first layer, of few inputs, also forms wl * xl and
// takes a third part of its weights, which leaves 4.4e-8, and the output
// layer sums in two chains a lane where the fp32 family runs one.)
//
// Scaling, all by powers of two, so exact.  fp16 keeps a value's 11 bits only
// above 2^-14 and nothing below 2^-25, so every value must come near the top
// of its range whatever the spread of the weights.  Each level k, neuron n and
// tile gets a scale of its own (ReLU commutes with a positive factor):
//
//   C_k: the power of two above level k's largest weight; X: the tile's largest
//   |x_k| C_k; B_n = max(sum_i |w_ni| B_i, b_n / max_k C_k) (of a level: 1 /
//   C_k), so that neuron n's activation is at most X B_n (1 + what biases add);
//   r_n: the power of two above B_n;
//
//   level k times C_k t, neuron n times t / r_n, weight n, i times r_i / r_n,
//
// with t X in [2^14, 2^15): activations come out of the matrix cores below 2^15
// (1 + ..) as the next ones take them, and weights are about 1 at most.  Their
// lower parts are stored as wl 2^12 and meet xh 2^-12, where wl by itself would
// be too small.  A row is complete in one wavefront and needs only the B_i
// before it: one barrier a layer, once per workgroup; X alone is the tile's, and
// its staging scales the levels as it stores them.  A bias is one more input, b
// / (r_n rho) against the activation t rho (rho: their largest, or the level's
// below), or starts the accumulators, binary32, where the operands have no slot.
// A bias that a level of magnitude 1 cannot reach (a neuron of no weights but a
// bias) counts in B_n as if one could; X is at least 8 times the largest b_n /
// r_n so counted, so biases add at most 1/8 to a layer's bound.
//
// What is left.  A part loses bits where a value lies 2^13 or more below the
// bound it was scaled by: up to 2^-25 for an activation, a residue that the
// preparation measures for a weight.  Carried through the layers (each row's sum
// of |weights| times what its inputs may be off), that bounds the outputs' error
// in the last sums, E_c, in the worst case.  What is lost in fact, by roundings
// that do not all point one way, is 1/50 of it (no hidden matrix), 1/60, 1/130,
// 1/500, 1/620, 1/1250, 1/2600 (one, 16, 32, 40, 64, 96, 128 wide) or 1/145,
// 1/420, 1/560, 1/1500, 1/3300, 1/7300 (two; largest error over 8192 pixels, nets
// drawn at random, a texel that raises X so that little else is seen).  A 16-pixel
// group counts only if each of its pixels has, for each channel, an output bias or
// one of its four partial sums of at least E_c times 2^15 (no hidden matrix, or a
// layer under 40 wide), 2^13 (under 64), 2^12 (under 96), 2^11 (under 128) or
// 2^10, half of that with two: what is lost in fact is then at most 3e-7 to 6e-7
// of it, where binary32 sums are off by 3e-7 (rms) to 2e-6 of it.  Other groups
// are evaluated again by the fp32 matrix instructions.  Nets of any common
// distribution pass by a factor of 10 to 1000, whatever the scales of their
// levels, neurons and biases; tiles with a texel 2^14 times larger than the rest,
// nets whose sums cancel and pixels that no neuron is active at do not.
//
// Range.  A workgroup with a weight or bias of 2^24 or more or B_n of 2^90, a
// tile with a level of 2^24 or more (NaN and infinities included), and one whose
// levels are so large (2^13 X at its least) that negative biases cut to fp16
// would no longer be sure to win, run on the fp32 matrix instructions altogether.
//
// Matrix-core mapping (lane l, lane group g = l / 16, i = l % 16)
//   v_mfma_f32_16x16x32_f16 takes A[i][8g + j] and B[8g + j][i], j = 0..7,
//   from lane l and returns D[4g + r][i] in register r of lane l.  Row 4g + r
//   of output block ob holds neuron 16 ob + 4r + g, so lane group g holds the
//   values v_q = neuron 4q + g, q = 4 ob + r (for the first layer v_q is level
//   4q + g of the lane's pixel): every lane group holds a quarter of any width
//   and forms its own K entries.  A word (two entries) holds one part of two
//   consecutive values, a pair; the words of four pairs make one operand, and
//   their three products take three instructions over two A operands (wh, wl;
//   hs marks xh 2^-12).  One pair left over: B = (h, l, hs, s) against A = (wh,
//   wh, wl, b); two: B0 = (h, h', l, l') against A0 = (wh, wh', wh, wh') and B1
//   = (hs, hs', s, s) against A1 = (wl, wl', b, b3); three: a fourth pair of
//   zeros.  (s: the bias activation and 2^-12 of it; b: the bias's upper and
//   lower part, b3 its third, lane group 0.)  The first layer's third parts take
//   one more step: B against (0, wl 2^-12, wll, b3), or B1 against (wll, wll',
//   0, 0).
//
// What binds it (768x512 x 64, 7 -> 40 -> 40 -> 3): vector issue and, with it,
// the chip's power; past 48 wide the LDS too (3840x2160, 8 -> 64 -> 64 -> 3:
// 53 reads a pass, mostly of 16 bytes a lane; eight more, for bias rows, cost
// 25 us of 270).  A 16-pixel group takes 130 vector instructions (prologue and
// tile set-up included) and 18 matrix ones; each matrix instruction keeps
// vector ones from issuing for 8 of its 16 cycles.  768x512 x 64 470 to 485 us,
// 2047x1365 (48 wide) 74, 3840x2160 256 to 274, one 768x512 image 15.5, of which
// the preparation of the neurons' scales, about 300 vector instructions a
// wavefront and two barriers, is 0.9.  (With one scale a layer, and one per pixel
// for the levels, on the same cards: 477 to 492, 75, 258 to 268, 14.6; but values
// 2^8 below their layer's largest lost bits.)  The first version, per-layer scales from each pixel's
// activations, remainders by v_fma_mixlo/hi_f16, which issue at half rate, the
// biases and inverse scales applied per value, four chains in the output layer:
// 189 vector instructions, 664, 103, 334, 17.6 us.
// Its error against 64 bits is 0.55 to 0.85 times the fp32 family's on nets
// whose outputs lie in [0, 1]; where the last layer is drawn like the others and
// the outputs range over +-3, 0.98 to 1.03 times for 64 wide, 1.07 to 1.24 for 33
// to 48, 0.82 to 0.87 (of the vector family's) past 64.  Tried and slower: wl * xl
// in the hidden layers too (those ratios 0.04 to 0.08 less, 768x512 x 64 485 ->
// 525 us); six products of three bf16 parts (exact, nothing to scale, as many
// vector instructions, twice the matrix ones), 655 to 830 us.
#pragma once

#include "decode_common.h"

namespace pic {
namespace mfma_f16x3 {

using namespace tile;

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// The lower parts of weights are stored times 2^kLow (the activations they
// meet times 2^-kLow): far enough that a weight 2^-25 of its row keeps 11 bits,
// and no further, or the activations' would be cut.
constexpr int kLow = 12;

// A layer's input of Q values per lane group: P pairs, QUADS operands of four
// in each part, TAIL mixed ones (as many A operands as steps); BIAS: whether a
// slot is left for it.
// FIRST: the first layer (Q at most 3: no quads) has one more A operand.
template <int Q, bool FIRST = false>
struct Shape {
    static constexpr int P = (Q + 1) / 2, R = P % 4;
    static constexpr int QUADS = P / 4 + (R == 3 ? 1 : 0);
    static constexpr int TAIL = R == 3 ? 0 : R;
    static constexpr int NA = 2 * QUADS + TAIL + (FIRST ? 1 : 0);
    static constexpr bool BIAS = TAIL > 0;
    static_assert(!FIRST || (QUADS == 0 && TAIL > 0), "the first layer's pairs are left over");
};

template <int NB, int NH, int LS, int KSH, int THT>
struct Layout {
    static constexpr int N = 16 * NB;
    static constexpr int N1A = Shape<LS, true>::NA, NHA = Shape<KSH>::NA;   // A operands per output block
    static constexpr int W1A = 0;                                     // u32 [NB][N1A][64][4]
    static constexpr int WHA = W1A + NB * N1A * 256;                  // u32 [NH][NB][NHA][64][4]
    static constexpr int HB = Shape<KSH>::BIAS ? 0 : NH;              // hidden layers whose biases start the accumulators
    static constexpr int BIAS = WHA + NH * NB * NHA * 256;            // f32 [HB][N], swz order: those, scaled for the tile
    static constexpr int RAWB = BIAS + HB * N;                        // f32 [HB][N], swz: over r_n
    static constexpr int BND = RAWB + HB * N;                         // f32 [NH + 1][N], swz: B_n
    static constexpr int W3 = BND + (NH + 1) * N;                     // f32 [3][N], swz order, times r_n
    static constexpr int CMAX = W3 + 3 * N;                           // f32 [4 LS][kWaves]: largest weights of each level
    static constexpr int CSCALE = CMAX + 4 * LS * kWaves;             // f32 [4 LS]: C_k
    static constexpr int ERR = CSCALE + 4 * LS;                       // f32 [NH + 1][kWaves]: largest errors
    static constexpr int BMAX = ERR + (NH + 1) * kWaves;              // f32 [NH + 1][kWaves]: largest |b_n| / r_n
    static constexpr int XMAX = BMAX + (NH + 1) * kWaves;             // f32 [kWaves]: largest scaled levels of the tile
    static constexpr int L1C = XMAX + kWaves;                         // f32 [kWaves]: sum of |w3|, by channel
    static constexpr int BAD = L1C + kWaves;                          // u32 [2][kWaves]: out-of-range flags
    static constexpr int COL = BAD + 2 * kWaves;                      // (int, f32) [4 LS][TW]: column taps
    static constexpr int ROW = COL + 4 * LS * TW * 2;                 // (int, f32) [4 LS][THT]: row taps
    static constexpr int LAT = ROW + 4 * LS * THT * 2;                // latent boxes
    static constexpr int SIZE = LAT + box_offset<THT>(4 * LS);
};

// Each 16-neuron group of a bias vector, of the bounds and of the output
// layer's rows is stored with the two 2-bit halves of its index swapped, so that a lane
// group's four neurons of a block are one 16-byte read.
__host__ __device__ constexpr int swz(int n) { return (n & ~15) | ((n & 3) << 2) | ((n >> 2) & 3); }

// Neuron on row `row` of an output block; the map is its own inverse.
__device__ __forceinline__ int row_neuron(int row) { return 4 * (row & 3) + (row >> 2); }

// The power of two above x >= 0 (x in [p / 2, p)); 2^-126 for 0.
__device__ __forceinline__ float pow2_above(float x)
{
    return __uint_as_float((__float_as_uint(x) & 0x7f800000u) + 0x00800000u);
}

// 1 / p for a power of two (exact).
__device__ __forceinline__ float pow2_inverse(float p) { return __uint_as_float((254u << 23) - __float_as_uint(p)); }

// C_k and 1 / C_k of a level whose largest weight is m: 0 for a level without
// weights, at least 2^-60 for others.
__device__ __forceinline__ float level_scale(float m) { return m > 0.0f ? fmaxf(pow2_above(m), 0x1p-60f) : 0.0f; }
__device__ __forceinline__ float level_unscale(float c) { return c > 0.0f ? pow2_inverse(c) : 0.0f; }

// The two parts of a pair of values, as packed words (first value low).  The
// remainder x - xh is one mixed-precision fused multiply-add, exact (written
// out, because the compiler converts xh back and subtracts: two instructions).
struct Parts {
    unsigned h, l;
};

__device__ __forceinline__ Parts split2(float x0, float x1)
{
    const unsigned h = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{x0, x1}), f16x2));
    float r0, r1;
    asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r0) : "v"(h), "v"(x0));
    asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r1) : "v"(h), "v"(x1));
    const f16x2 l = __builtin_convertvector((f32x2{r0, r1}), f16x2);
    return Parts{h, __builtin_bit_cast(unsigned, l)};
}

// A pair of fp16 values times 2^-kLow.
__device__ __forceinline__ unsigned lower(unsigned h)
{
    constexpr _Float16 k = (_Float16)(1.0f / (1 << kLow));
    return __builtin_bit_cast(unsigned, __builtin_bit_cast(f16x2, h) * f16x2{k, k});
}

// The parts of a pair of weights: h, l 2^kLow, third 2^kLow; lost: what is left
// out of their products, for an activation of 1 and 2^kLow, of weights below
// 2^-14 (of those above, it is as small against the product as elsewhere): what
// the first two parts leave, and l against the activation's lower part, at most
// 2^-11.
struct WeightParts {
    unsigned h, l, third;
    float lost;
};

__device__ __forceinline__ WeightParts split_weights(float x0, float x1)
{
    constexpr float up = (float)(1 << kLow);
    auto rest = [](unsigned h, float x, bool hi) {    // x - h's low or high half
        float r;
        if (hi)
            asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h), "v"(x));
        else
            asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h), "v"(x));
        return r;
    };
    auto pack = [](float a, float b) {
        return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{a, b}), f16x2));
    };
    const unsigned h = pack(x0, x1);
    const float r0 = rest(h, x0, false) * up, r1 = rest(h, x1, true) * up;
    const unsigned l = pack(r0, r1);
    const float t0 = rest(l, r0, false), t1 = rest(l, r1, true);
    return WeightParts{h, l, pack(t0, t1),
                       (fabsf(x0) < 0x1p-14f ? __builtin_fmaf(fabsf(r0), 0x1p-11f, fabsf(t0)) : 0.0f) +
                           (fabsf(x1) < 0x1p-14f ? __builtin_fmaf(fabsf(r1), 0x1p-11f, fabsf(t1)) : 0.0f)};
}

__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
}

// A operands of one output block's row, from its scaled weights of the pairs,
// without its bias; returns what their parts lose, 2^kLow.
template <int Q, bool FIRST>
__device__ __forceinline__ float build_a(const float (&w)[2 * Shape<Q>::P], u32x4 (&a)[Shape<Q, FIRST>::NA])
{
    using S = Shape<Q, FIRST>;
    WeightParts p[4 * S::QUADS + S::TAIL];
    float lost = 0.0f;
#pragma unroll
    for (int i = 0; i < 4 * S::QUADS + S::TAIL; ++i) {
        p[i] = i < S::P ? split_weights(w[2 * i], w[2 * i + 1]) : WeightParts{0u, 0u, 0u, 0.0f};
        lost += p[i].lost;
    }
#pragma unroll
    for (int q = 0; q < S::QUADS; ++q) {
        a[2 * q] = u32x4{p[4 * q].h, p[4 * q + 1].h, p[4 * q + 2].h, p[4 * q + 3].h};
        a[2 * q + 1] = u32x4{p[4 * q].l, p[4 * q + 1].l, p[4 * q + 2].l, p[4 * q + 3].l};
    }
    if constexpr (S::TAIL == 1) {
        const WeightParts t = p[4 * S::QUADS];
        a[2 * S::QUADS] = u32x4{t.h, t.h, t.l, 0u};
        if constexpr (FIRST)
            a[1] = u32x4{0u, lower(t.l), t.third, 0u};
    } else if constexpr (S::TAIL == 2) {
        const WeightParts t = p[4 * S::QUADS], u = p[4 * S::QUADS + 1];
        a[2 * S::QUADS] = u32x4{t.h, u.h, t.h, u.h};
        a[2 * S::QUADS + 1] = u32x4{t.l, u.l, 0u, 0u};
        if constexpr (FIRST)
            a[2] = u32x4{t.third, u.third, 0u, 0u};
    }
    return lost;
}

// Put one row's scaled bias (lane group 0; zero elsewhere) into the block's
// operands at a: upper and lower part in one word, a third part in another
// where there is one left.
template <int Q, bool FIRST>
__device__ __forceinline__ void put_bias(unsigned *a, float bias)
{
    using S = Shape<Q, FIRST>;
    const WeightParts b = split_weights(bias, 0.0f);
    const unsigned w = b.h | b.l << 16, w3 = b.third << 16;
    if constexpr (S::TAIL == 1) {
        a[2 * S::QUADS * 256 + 3] = w;
        if constexpr (FIRST)
            a[256 + 3] = w3;
    } else if constexpr (S::TAIL == 2) {
        a[(2 * S::QUADS + 1) * 256 + 2] = w;
        a[(2 * S::QUADS + 1) * 256 + 3] = w3;
    }
}

// One layer for G groups of 16 pixels: d[gi][ob] = bias + W v[gi], small
// partial products first.  la: the layer's A operands (at this lane's words);
// lb: its bias rows (at this lane group's), which start the accumulators where
// the operands have no slot; sw: the bias activation's word.
template <int Q, bool FIRST, int NB, int G>
__device__ __forceinline__ void apply(const unsigned *la, const float *lb, unsigned sw, const float (&v)[G][Q],
                                      f32x4 (&d)[G][NB])
{
    using S = Shape<Q, FIRST>;
    auto op = [&](int ob, int i) { return *reinterpret_cast<const u32x4 *>(la + (ob * S::NA + i) * 256); };
    auto val = [&](int gi, int i) { return i < Q ? v[gi][i < Q ? i : 0] : 0.0f; };
    // one step of every group against output block ob; `start`: the layer's first
    auto step = [&](bool start, int ob, u32x4 w, const u32x4 (&b)[G]) {
        f32x4 bias = {0.0f, 0.0f, 0.0f, 0.0f};
        if (start && !S::BIAS)
            bias = *reinterpret_cast<const f32x4 *>(lb + 16 * ob);
#pragma unroll
        for (int gi = 0; gi < G; ++gi)
            d[gi][ob] = mfma(w, b[gi], start ? bias : d[gi][ob]);
    };
#pragma unroll
    for (int q = 0; q < S::QUADS; ++q) {
        u32x4 h[G], l[G], hs[G];
#pragma unroll
        for (int gi = 0; gi < G; ++gi)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = 4 * q + j;
                const Parts t = i < S::P ? split2(val(gi, 2 * i), val(gi, 2 * i + 1)) : Parts{0u, 0u};
                h[gi][j] = t.h;
                l[gi][j] = t.l;
                hs[gi][j] = i < S::P ? lower(t.h) : 0u;
            }
        u32x4 wh[NB], wl[NB];
#pragma unroll
        for (int ob = 0; ob < NB; ++ob) {
            wl[ob] = op(ob, 2 * q + 1);
            wh[ob] = op(ob, 2 * q);
        }
#pragma unroll
        for (int st = 0; st < 3; ++st)
#pragma unroll
            for (int ob = 0; ob < NB; ++ob)
                step(q == 0 && st == 0, ob, st == 0 ? wl[ob] : wh[ob], st == 0 ? hs : st == 1 ? l : h);
    }
    if constexpr (S::TAIL == 1) {
        constexpr int i = 4 * S::QUADS;
        u32x4 b[G];
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
            const Parts t = split2(val(gi, 2 * i), val(gi, 2 * i + 1));
            b[gi] = u32x4{t.h, t.l, lower(t.h), sw};
        }
#pragma unroll
        for (int st = FIRST ? 1 : 0; st >= 0; --st)
#pragma unroll
            for (int ob = 0; ob < NB; ++ob)
                step(S::QUADS == 0 && st == (FIRST ? 1 : 0), ob, op(ob, 2 * S::QUADS + st), b);
    } else if constexpr (S::TAIL == 2) {
        constexpr int i = 4 * S::QUADS;
        u32x4 b0[G], b1[G];
#pragma unroll
        for (int gi = 0; gi < G; ++gi) {
            const Parts t = split2(val(gi, 2 * i), val(gi, 2 * i + 1));
            const Parts u = split2(val(gi, 2 * i + 2), val(gi, 2 * i + 3));
            b0[gi] = u32x4{t.h, u.h, t.l, u.l};
            b1[gi] = u32x4{lower(t.h), lower(u.h), sw, sw};
        }
#pragma unroll
        for (int st = FIRST ? 2 : 1; st >= 0; --st)
#pragma unroll
            for (int ob = 0; ob < NB; ++ob)
                step(S::QUADS == 0 && st == (FIRST ? 2 : 1), ob, op(ob, 2 * S::QUADS + st), st == 0 ? b0 : b1);
    }
}

// Largest of x over the four lane groups of this lane's column.
__device__ __forceinline__ float column_max(float x)
{
    const unsigned xi = __float_as_uint(x);
    const u32x2 a = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
    const unsigned m = max(a[0], a[1]);
    const u32x2 c = __builtin_amdgcn_permlane32_swap(m, m, false, false);
    return __uint_as_float(max(c[0], c[1]));
}

// Reductions by data-parallel moves within the vector unit instead of exchanges
// through LDS: over each row of 16 lanes by rotations of 8, 4, 2 and 1 (every
// lane has the result), over the wavefront by broadcasts between the rows (lane
// 15 of the row before into rows 1 and 3, lane 31 into rows 2 and 3), read from
// lane 63; lanes a move does not write take part with their own value (maxima)
// or 0 (sums).  Maxima: of x >= 0, not NaN (such floats order like their bits).
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ int moved(int old, int x)
{
    return __builtin_amdgcn_update_dpp(old, x, CTRL, ROWS, 0xF, false);
}

__device__ __forceinline__ int row16_max(int v)
{
    v = max(v, moved<0x128>(v, v));    // row_ror:8
    v = max(v, moved<0x124>(v, v));
    v = max(v, moved<0x122>(v, v));
    return max(v, moved<0x121>(v, v));
}

__device__ __forceinline__ float wave_max(float x)
{
    int v = row16_max(__float_as_int(x));
    v = max(v, moved<0x142, 0xA>(v, v));   // row_bcast:15, rows 1 and 3
    v = max(v, moved<0x143, 0xC>(v, v));   // row_bcast:31, rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(v, 63));
}

__device__ __forceinline__ float wave_sum(float x)
{
    auto add = [&](int y) { x += __int_as_float(y); };
    add(moved<0x128>(0, __float_as_int(x)));
    add(moved<0x124>(0, __float_as_int(x)));
    add(moved<0x122>(0, __float_as_int(x)));
    add(moved<0x121>(0, __float_as_int(x)));
    add(moved<0x142, 0xA>(0, __float_as_int(x)));
    add(moved<0x143, 0xC>(0, __float_as_int(x)));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// t of a tile whose largest scaled level is x, and 1 / t.
__device__ __forceinline__ float tile_scale(float x, float &inv_t)
{
    const float p = pow2_above(x);
    inv_t = p * 0x1p-15f;
    return 0x1p15f * pow2_inverse(p);
}

__device__ __forceinline__ float max4(const f32x4 &m) { return fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3])); }

// Whether one of the workgroup's 2 kWaves out-of-range flags is set.
__device__ __forceinline__ unsigned any_flag(const unsigned *flags)
{
    const u32x4 a = reinterpret_cast<const u32x4 *>(flags)[0], b = reinterpret_cast<const u32x4 *>(flags)[1];
    return __builtin_amdgcn_readfirstlane(a[0] | a[1] | a[2] | a[3] | b[0] | b[1] | b[2] | b[3]);
}

__device__ __forceinline__ float uniform(float x)
{
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}

// f(register, level) for the box registers of load_boxes.
template <int KMAX, int THT, class F>
__device__ __forceinline__ void each_box_reg(F f)
{
    int idx = 0;
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
#pragma unroll
        for (int i0 = 0; i0 < box_floats<THT>(k); i0 += kThreads)
            f(idx++, k);
}

// NB: 16-neuron blocks of the hidden width; NH: hidden layers; LS: levels per
// lane group (ceil(L / 4)); KSH: values per lane group of the hidden layers'
// inputs (ceil(width / 4)); RPW: tile rows per wavefront (a tile is 4 RPW
// rows: 8, or 16 or 32 when the launch has tiles to spare).
template <int NB, int NH, int LS, int KSH, int RPW>
__global__ __launch_bounds__(kThreads) void k_mfma_f16x3(DecodeParams p, int blocks_per_image, int tiles_x,
                                                         int tiles, uint32_t tx_recip)
{
    static_assert(KSH <= 4 * NB && KSH > 4 * (NB - 1), "KSH must end in the last block");
    constexpr int THT = kWaves * RPW;   // tile rows
    constexpr int LV = 4 * LS;          // levels staged
    // 16-pixel groups per pass: they share every weight read (768x512 x 64
    // 536 -> 513 us, 4K 289 -> 274 us against one, at 4 wavefronts per SIMD
    // instead of 5 and 3 instead of 4)
    constexpr int G = NB <= 4 ? 2 : 1;
    constexpr int BPW = (NB + kWaves - 1) / kWaves;   // output blocks a wavefront forms
    constexpr int NPL = (16 * NB + 63) / 64;          // neurons a lane stages
    using LY = Layout<NB, NH, LS, KSH, THT>;
    __shared__ __attribute__((aligned(16))) float lds[LY::SIZE];
    unsigned *ldsu = reinterpret_cast<unsigned *>(lds);

    warm_kernel_args<sizeof(DecodeParams)>();
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, col = lane & 15;
    // images interleave over the grid, so that every image's workgroups are
    // spread over the dispatch order (older workgroups on a CU run ahead)
    int b = 0;
    if (p.batch > 1)
        b = blockIdx.x % p.batch;
    const TileSchedule ts = tile_schedule(p, blockIdx.x, blocks_per_image, tiles);
    const int blk = ts.first;
    const int L = p.L, H = p.H, W = p.W;
    // the output layer's bias, read now so its latency hides behind the
    // parameter loads
    const float *b3 = layer_params(p, NH + 1, b).b;
    const float b3_0 = b3[0], b3_1 = b3[1], b3_2 = b3[2];

    // In range: the sum of the magnitudes a thread checks is below 2^24 (so
    // each of them is); a NaN or an infinity makes the sum fail the compare.
    constexpr float kRange = 16777216.0f;

    // ---- this image's parameters.  Every load is issued before the first is
    // waited for (the first tile's latents first), through raw buffers whose
    // range check returns 0 past each array's end (rows past a layer's
    // outputs).  Wavefront w forms the A operands of output blocks w, w + 4:
    // lane (g, col) holds row rn(col)'s weights of the inputs 4 q + g.
    float inv_t = 0.0f;    // 1 / t of the tile
    float xfloor;          // least X
    float rho;             // scale of the biases in the operands: their activation is t rho
    bool steep;            // whether some are far above it: cut to fp16's range
    float sb = 0.0f;       // the tile's t rho
    {
        LayerParams lp[NH + 2];
        int wd[NH + 3];
#pragma unroll
        for (int l = 0; l < NH + 2; ++l)
            lp[l] = layer_params(p, l, b);
#pragma unroll
        for (int l = 0; l < NH + 3; ++l)
            wd[l] = p.widths[l];
        const int NL = wd[NH + 1];
        float boxv[box_regs<LV, THT>()];
        float w1[BPW][2 * Shape<LS>::P], wh[BPW][NH > 0 ? NH : 1][2 * Shape<KSH>::P];
        float brow[BPW][NH + 1], bv[NPL], w3v[NPL];
        const int lw = min(wave, NH), l3 = min(wave, 2);    // bias layer / output row of this wavefront
        if (blk < tiles) {
            const int by = tile_row(blk, tiles_x, tx_recip);
            load_boxes<LV, THT>(boxv, p, b, by * THT, (blk - by * tiles_x) * TW, tid);
        }
        {
            auto ld = [](__amdgpu_buffer_rsrc_t r, unsigned idx) {
                return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, idx * 4, 0, 0));
            };
            const auto w1b = raw_buffer(lp[0].w, (unsigned)(wd[1] * L) * 4);
#pragma unroll
            for (int j = 0; j < BPW; ++j) {
                const int row = 16 * (wave + kWaves * j) + row_neuron(col);
#pragma unroll
                for (int q = 0; q < LS; ++q)
                    w1[j][q] = ld(w1b, (unsigned)(row * L + g + 4 * q));
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    const auto hb = raw_buffer(lp[1 + h].w, (unsigned)(wd[2 + h] * wd[1 + h]) * 4);
#pragma unroll
                    for (int q = 0; q < KSH; ++q)
                        wh[j][h][q] = ld(hb, (unsigned)(row * wd[1 + h] + g + 4 * q));
                }
#pragma unroll
                for (int l = 0; l <= NH; ++l)
                    brow[j][l] = ld(raw_buffer(lp[l].b, (unsigned)wd[1 + l] * 4), (unsigned)row);
            }
#pragma unroll
            for (int i = 0; i < NPL; ++i) {
                bv[i] = ld(raw_buffer(layer_params(p, lw, b).b, (unsigned)p.widths[1 + lw] * 4), (unsigned)(lane + 64 * i));
                w3v[i] = ld(raw_buffer(lp[NH + 1].w, (unsigned)(3 * NL) * 4), (unsigned)(l3 * NL + lane + 64 * i));
            }
        }
        if (blk < tiles) {   // (while the loads are in flight)
            const int by = tile_row(blk, tiles_x, tx_recip);
            fill_taps<LV, THT>(ldsu, LY::COL, LY::ROW, LY::LAT, p, by * THT, (blk - by * tiles_x) * TW, wave, lane);
        }
        // entries past a layer's inputs read the next row: zeroed
        float sum = fabsf(b3_0) + fabsf(b3_1) + fabsf(b3_2), lsum = 0.0f;
#pragma unroll
        for (int j = 0; j < BPW; ++j) {
            if (LS & 1)
                w1[j][LS] = 0.0f;
            w1[j][LS - 1] = 4 * (LS - 1) + g < L ? w1[j][LS - 1] : 0.0f;
#pragma unroll
            for (int q = 0; q < LS; ++q)
                sum += fabsf(w1[j][q]);
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                if (KSH & 1)
                    wh[j][h][KSH] = 0.0f;
#pragma unroll
                for (int q = 0; q < KSH; ++q) {
                    wh[j][h][q] = 4 * q + g < wd[1 + h] ? wh[j][h][q] : 0.0f;
                    sum += fabsf(wh[j][h][q]);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < LS; ++q) {    // largest weight of levels 4 q + g
            float m = fabsf(w1[0][q]);
#pragma unroll
            for (int j = 1; j < BPW; ++j)
                m = fmaxf(m, fabsf(w1[j][q]));
            const int mb = row16_max(__float_as_int(m));
            if (col == 0)
                ldsu[LY::CMAX + (4 * q + g) * kWaves + wave] = mb;
        }
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            w3v[i] = lane + 64 * i < NL ? w3v[i] : 0.0f;
            sum += fabsf(bv[i]) + fabsf(w3v[i]);
        }
        if (blk < tiles)
            each_box_reg<LV, THT>([&](int i, int) { lsum += fabsf(boxv[i]); });
        bool pbad = !(sum < kRange);
        {
            const bool tbad = __any(!(lsum < kRange));
            if (lane == 0)
                ldsu[LY::BAD + wave] = tbad;
        }
        __syncthreads();

        // The layers in turn: each row's sum of |weights| times its inputs'
        // bounds, its bound and scale; then its operands, and what they lose.
        float ck[LV];    // C_k
        float one;       // the largest: a level of magnitude 1, scaled
#pragma unroll
        for (int l = 0; l <= NH; ++l) {
            constexpr int Q = LS > KSH ? LS : KSH;
            float cb[Q];    // B_i of the inputs 4 q + g
            if (l == 0) {
#pragma unroll
                for (int q = 0; q < LS; ++q) {
                    const float c = level_scale(max4(*reinterpret_cast<const f32x4 *>(&lds[LY::CMAX + (4 * q + g) * kWaves])));
                    if (tid == 16 * g)
                        lds[LY::CSCALE + 4 * q + g] = c;
                    cb[q] = level_unscale(c);
                    one = q == 0 ? c : fmaxf(one, c);
                }
                one = fmaxf(column_max(one), 0x1p-60f);
            } else {
#pragma unroll
                for (int q = 0; q < KSH; q += 4) {
                    const f32x4 bd = *reinterpret_cast<const f32x4 *>(&lds[LY::BND + (l - 1) * LY::N + 4 * q + 4 * g]);
#pragma unroll
                    for (int i = 0; i < 4 && q + i < KSH; ++i)
                        cb[q + i] = bd[i];
                }
            }
            if (l == (NH > 0 ? 1 : 0) && blk < tiles) {    // the first tile's largest scaled level
#pragma unroll
                for (int k = 0; k < LV; ++k)
                    ck[k] = NH > 0 ? lds[LY::CSCALE + k]
                                   : level_scale(max4(*reinterpret_cast<const f32x4 *>(&lds[LY::CMAX + k * kWaves])));
                float m = 0.0f;
                each_box_reg<LV, THT>([&](int i, int k) { m = fmaxf(m, fabsf(boxv[i]) * ck[k]); });
                m = wave_max(m);
                if (lane == 0)
                    lds[LY::XMAX + wave] = m;
            }
            // what the inputs may be off, in 2^-25 (a level: by its parts)
            const float err = l == 0 ? 1.0f
                                     : max4(*reinterpret_cast<const f32x4 *>(&lds[LY::ERR + (l > 0 ? l - 1 : 0) * kWaves])) + 1.0f;
            const float inv_one = pow2_inverse(one);
            float worst = 0.0f, bmax = 0.0f;
#pragma unroll
            for (int j = 0; j < BPW; ++j) {
                const int blk16 = wave + kWaves * j, h = l > 0 ? l - 1 : 0;
                if (blk16 >= NB)
                    break;    // wave-uniform
                float s = 0.0f, l1 = 0.0f;
                if (l == 0) {
#pragma unroll
                    for (int q = 0; q < LS; ++q)
                        s = __builtin_fmaf(fabsf(w1[j][q]), cb[q], s);
                } else {
#pragma unroll
                    for (int q = 0; q < KSH; ++q)
                        s = __builtin_fmaf(fabsf(wh[j][h][q]), cb[q], s);
                }
                s = row_sum(s);
                const float bn = fmaxf(s, brow[j][l] * inv_one);
                const float ri = bn > 0.0f ? pow2_inverse(pow2_above(bn)) : 0.0f;    // (0: never active)
                pbad = pbad || !(bn < 0x1p90f);
                if (g == 0)
                    lds[LY::BND + l * LY::N + swz(16 * blk16 + row_neuron(col))] = bn;
                brow[j][l] *= ri;
                bmax = fmaxf(bmax, fabsf(brow[j][l]));
                float lost;
                if (l == 0) {
                    u32x4 a1[LY::N1A];
#pragma unroll
                    for (int q = 0; q < LS; ++q) {
                        w1[j][q] = w1[j][q] * cb[q] * ri;
                        l1 += fabsf(w1[j][q]);
                    }
                    lost = build_a<LS, true>(w1[j], a1);
#pragma unroll
                    for (int i = 0; i < LY::N1A; ++i)
                        *reinterpret_cast<u32x4 *>(&ldsu[LY::W1A + ((blk16 * LY::N1A + i) * 64 + lane) * 4]) = a1[i];
                } else {
                    u32x4 ah[LY::NHA];
#pragma unroll
                    for (int q = 0; q < KSH; ++q) {
                        wh[j][h][q] = wh[j][h][q] * pow2_above(cb[q]) * ri;
                        l1 += fabsf(wh[j][h][q]);
                    }
                    lost = build_a<KSH, false>(wh[j][h], ah);
#pragma unroll
                    for (int i = 0; i < LY::NHA; ++i)
                        *reinterpret_cast<u32x4 *>(&ldsu[LY::WHA + (((h * NB + blk16) * LY::NHA + i) * 64 + lane) * 4]) =
                            ah[i];
                }
                // a row's inputs off by err, their upper parts times 2^-kLow by
                // 2^-25 against lower parts of 2^(kLow - 11) |w| (or 2^(kLow -
                // 25)), its weights by `lost` 2^-kLow against 2^15 (1 + l / 8)
                worst = fmaxf(worst, row_sum(__builtin_fmaf(l1, err + (float)(1 << kLow) * 0x1p-11f,
                                                            lost * (0x1p40f * (1.0f + 0.125f * l) / (1 << kLow)))));
            }
            // (a bias in the operands, at most 2, loses up to 2^-37 against its
            // activation of at most 2^12, and up to 2^-12 against one below 2^-12)
            worst = __int_as_float(row16_max(__float_as_int(worst))) + 0x1p-4f;
            bmax = __int_as_float(row16_max(__float_as_int(bmax)));
            if (l == 0 || Shape<KSH>::BIAS)
                worst += bmax > 0.0f ? 4.0f : 0.0f;
            if (lane == 0) {
                lds[LY::ERR + l * kWaves + wave] = worst;
                lds[LY::BMAX + l * kWaves + wave] = bmax;
            }
            if (l == NH) {
                const bool any = __any(pbad);
                if (lane == 0)
                    ldsu[LY::BAD + kWaves + wave] = any;
            }
            __syncthreads();
        }

        // the output layer's weights times the last r_n, the biases over r_n,
        // the first tile's scaled boxes and biases
        float bmax = 0.0f;
#pragma unroll
        for (int l = 0; l <= NH; ++l)
            bmax = fmaxf(bmax, max4(*reinterpret_cast<const f32x4 *>(&lds[LY::BMAX + l * kWaves])));
        bmax = uniform(bmax);
        const float level = fmaxf(fminf(bmax, one), 0x1p-60f);
        xfloor = 8.0f * level;
        rho = 0.5f * pow2_above(level);
        steep = __builtin_amdgcn_readfirstlane(bmax > 2.0f * rho) != 0;
        const float irho = pow2_inverse(rho);
#pragma unroll
        for (int j = 0; j < BPW; ++j) {
            const int blk16 = wave + kWaves * j;
            if (blk16 >= NB)
                break;    // wave-uniform
            auto cut = [&](int l) { return g == 0 ? fmaxf(brow[j][l] * irho, -65504.0f) : 0.0f; };
            put_bias<LS, true>(ldsu + LY::W1A + blk16 * LY::N1A * 256 + 4 * lane, cut(0));
            if constexpr (Shape<KSH>::BIAS)
#pragma unroll
                for (int h = 0; h < NH; ++h)
                    put_bias<KSH, false>(ldsu + LY::WHA + (h * NB + blk16) * LY::NHA * 256 + 4 * lane, cut(1 + h));
        }
        float l1c = 0.0f, braw[NPL];
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            const int n = lane + 64 * i, at = swz(min(n, LY::N - 1));
            const float w = w3v[i] * pow2_above(lds[LY::BND + NH * LY::N + at]);
            l1c += fabsf(w);
            if (n < LY::N && wave < 3)
                lds[LY::W3 + wave * LY::N + at] = w;
            if constexpr (LY::HB > 0) {
                braw[i] = bv[i] * pow2_inverse(pow2_above(lds[LY::BND + lw * LY::N + at]));
                if (n < LY::N && wave >= 1 && wave <= NH)
                    lds[LY::RAWB + (wave - 1) * LY::N + at] = braw[i];
            }
        }
        l1c = wave_sum(l1c);
        if (lane == 0)
            lds[LY::L1C + wave] = l1c;
        if (blk < tiles) {
            const float t = tile_scale(fmaxf(max4(*reinterpret_cast<const f32x4 *>(&lds[LY::XMAX])), xfloor), inv_t);
            sb = t * rho;
            if (any_flag(ldsu + LY::BAD) == 0)
                each_box_reg<LV, THT>([&](int i, int k) { boxv[i] *= ck[k] * t; });
            store_boxes<LV, THT>(lds + LY::LAT, boxv, tid);
            if constexpr (LY::HB > 0)
#pragma unroll
                for (int i = 0; i < NPL; ++i)
                    if (lane + 64 * i < LY::N && wave >= 1 && wave <= NH)
                        lds[LY::BIAS + (wave - 1) * LY::N + swz(lane + 64 * i)] = braw[i] * t;
        }
        __syncthreads();
    }
    // a channel's least acceptable partial sum: E_c times 2^15 to 2^9 (the
    // header says why), by the narrowest hidden layer
    float thr[3];
    {
        int n = p.widths[1];
#pragma unroll
        for (int l = 2; l <= NH + 1; ++l)
            n = min(n, p.widths[l]);
        const float above = (NH == 0 || n < 40 ? 0x1p15f : n < 64 ? 0x1p13f : n < 96 ? 0x1p12f : n < 128 ? 0x1p11f : 0x1p10f) *
                            (NH == 2 ? 0.5f : 1.0f);
        const float err = max4(*reinterpret_cast<const f32x4 *>(&lds[LY::ERR + NH * kWaves])) * (above * 0x1p-25f);
#pragma unroll
        for (int c = 0; c < 3; ++c)
            thr[c] = uniform(err * lds[LY::L1C + c]);
    }

    const int64_t plane = (int64_t)H * W;
    // Lane group g (< 3) stores channel g.
    const int64_t obase = (int64_t)(uint64_t)(uint32_t)(3 * b + min(g, 2)) * plane;
    const float ob = g == 0 ? b3_0 : g == 1 ? b3_1 : b3_2;
    unsigned pitch[LS];                // of the boxes this lane samples, bytes
#pragma unroll
    for (int s = 0; s < LS; ++s)
        pitch[s] = tap_pitch(4 * s, 1, g, L);

    // upsampled levels 4 s + g of the lane's pixel of column group cg in row
    // yr of the tile (level 0 for those past L; zero weights)
    auto sample = [&](int yr, int cg, float (&u)[LS]) {
#pragma unroll
        for (int s = 0; s < LS; ++s)
            u[s] = tap_sample(lds, *reinterpret_cast<const u32x2 *>(&ldsu[LY::ROW + ((4 * s + g) * THT + yr) * 2]),
                              *reinterpret_cast<const u32x2 *>(&ldsu[LY::COL + ((4 * s + g) * TW + 16 * cg + col) * 2]),
                              pitch[s]);
    };

    // the output layer on the vector ALU: partial sums over this lane's
    // values in two chains.  (Four chains: the same error, 10 us more of
    // 768x512 x 64's 510.)  w(c, ob): channel c's weights of block ob.
    auto output = [&](const f32x4 (&d)[NB], float (&o)[3], auto w) {
        float a[3][2];
#pragma unroll
        for (int ob16 = 0; ob16 < NB; ++ob16) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const f32x4 w3 = w(c, ob16);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (4 * ob16 + r < KSH)
                        a[c][r & 1] = ob16 == 0 && r < 2 ? w3[r] * d[ob16][r]
                                                         : __builtin_fmaf(w3[r], d[ob16][r], a[c][r & 1]);
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
            o[c] = a[c][0] + a[c][1];
    };
    // bit i (of 16): whether a lane of column i is set in m
    auto columns = [](uint64_t m) {
        const unsigned f = (unsigned)m | (unsigned)(m >> 32);
        return (f | f >> 16) & 0xffff;
    };

    // Tiles: the workgroup's first is tile blk; the others come from its
    // schedule's counter (tile ts.base + ticket, while below ts.end), so that
    // workgroups that run faster take more of them.  The grid's first
    // workgroup clears the counters of the next run.
    __shared__ int s_next;
    const bool dynamic = blocks_per_image < tiles;
    if (blockIdx.x == 0)
        for (int i = tid; i < p.tile_ctr_len; i += kThreads)
            p.tile_ctr_next[i] = 0;
    for (int t = blk;;) {
        const int tr = tile_row(t, tiles_x, tx_recip);
        const int ty0 = tr * THT, tx0 = (t - tr * tiles_x) * TW;

        if (t != blk) {       // the first tile was staged with the parameters
            __syncthreads();   // every wavefront is done with the previous tile's boxes, taps and flags
            float v[box_regs<LV, THT>()];
            int z = 0, tz = tid;     // (opaque: stage_boxes says why)
            asm volatile("" : "+s"(z), "+v"(tz));
            load_boxes<LV, THT>(v, p, b, ty0, tx0, tz, z);
            fill_taps<LV, THT>(ldsu, LY::COL, LY::ROW, LY::LAT, p, ty0, tx0, wave, lane);
            float ck[LV];
#pragma unroll
            for (int k = 0; k < LV; k += 4) {
                const f32x4 c = *reinterpret_cast<const f32x4 *>(&lds[LY::CSCALE + k]);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    ck[k + i] = c[i];
            }
            float lsum = 0.0f, m = 0.0f;
            each_box_reg<LV, THT>([&](int i, int k) {
                lsum += fabsf(v[i]);
                m = fmaxf(m, fabsf(v[i]) * ck[k]);
            });
            const bool tbad = __any(!(lsum < kRange));
            m = wave_max(m);
            if (lane == 0) {
                ldsu[LY::BAD + wave] = tbad;
                lds[LY::XMAX + wave] = m;
            }
            __syncthreads();
            const float tsc = tile_scale(fmaxf(max4(*reinterpret_cast<const f32x4 *>(&lds[LY::XMAX])), xfloor), inv_t);
            if (any_flag(ldsu + LY::BAD) == 0)
                each_box_reg<LV, THT>([&](int i, int k) { v[i] *= ck[k] * tsc; });
            store_boxes<LV, THT>(lds + LY::LAT, v, tz);
            sb = tsc * rho;
            if constexpr (LY::HB > 0)
#pragma unroll
                for (int i = 0; i < NPL; ++i)
                    if (lane + 64 * i < LY::N && wave >= 1 && wave <= NH) {
                        const int at = (wave - 1) * LY::N + swz(lane + 64 * i);
                        lds[LY::BIAS + at] = lds[LY::RAWB + at] * tsc;
                    }
            __syncthreads();
        }
        int ticket = 0;    // the tile after this one; its latency hides behind the tile
        if (dynamic && tid == 0)
            ticket = atomicAdd(ts.ctr, 1);
        // out of range: the boxes hold the levels as they are.  (Biases cut to
        // -65504 sb stay below -2^16, dead, while sb is at least 1; where some
        // are large, their lower parts count while it is at least 2^-12.)
        const unsigned raw = any_flag(ldsu + LY::BAD);
        const unsigned bad = raw | (steep && __builtin_amdgcn_readfirstlane(sb < 2.0f) != 0 ? 1u : 0u);
        const int rows = min(RPW, H - ty0 - RPW * wave);    // of this wavefront (<= 0: none)
        // groups of the wavefront's rows to evaluate in binary32, a bit each
        static_assert(RPW * TWG <= 32, "a bit per group");
        unsigned again = 0;
        if (bad == 0) {
            // the least partial sums, 0 where the output bias covers them (or
            // no output of any size could tell)
            const float th0 = uniform(fmaxf(fabsf(b3_0), 0x1p-60f) >= thr[0] * inv_t ? 0.0f : thr[0]);
            const float th1 = uniform(fmaxf(fabsf(b3_1), 0x1p-60f) >= thr[1] * inv_t ? 0.0f : thr[1]);
            const float th2 = uniform(fmaxf(fabsf(b3_2), 0x1p-60f) >= thr[2] * inv_t ? 0.0f : thr[2]);
            const bool check = !(th0 + th1 + th2 == 0.0f);
            // the bias activation's word: sb against a bias's upper part, sb
            // 2^-kLow against its lower parts
            const unsigned sw = __builtin_bit_cast(
                unsigned, __builtin_convertvector((f32x2{sb, sb * (1.0f / (1 << kLow))}), f16x2));
#pragma unroll 1
            for (int rr = 0; rr < rows; ++rr) {
                const int yr = RPW * wave + rr;
                const int64_t orow = obase + pixel_index(ty0 + yr, W, tx0 + col);
#pragma unroll
                for (int cg = 0; cg < TWG; cg += G) {
                    if (tx0 + 16 * cg >= W)
                        break;   // wave-uniform: the pass lies right of the image
                    // Re-read the LDS operands per pass rather than letting the
                    // compiler keep loop-invariant ones in VGPRs (occupancy).
                    // (A later group of a pass may lie right of the image: its
                    // taps are those of the last column, its store is skipped.)
                    asm volatile("" ::: "memory");
                    float v1[G][LS];
                    f32x4 d[G][NB];
#pragma unroll
                    for (int gi = 0; gi < G; ++gi)
                        sample(yr, cg + gi, v1[gi]);
                    apply<LS, true, NB, G>(ldsu + LY::W1A + 4 * lane, lds, sw, v1, d);

                    // hidden layers: the outputs are the next layer's inputs,
                    // scaled as they stand
#pragma unroll
                    for (int h = 0; h < NH; ++h) {
                        float v[G][KSH];
#pragma unroll
                        for (int gi = 0; gi < G; ++gi)
#pragma unroll
                            for (int q = 0; q < KSH; ++q)
                                v[gi][q] = relu(d[gi][q >> 2][q & 3]);
                        apply<KSH, false, NB, G>(ldsu + LY::WHA + h * NB * LY::NHA * 256 + 4 * lane,
                                                 lds + LY::BIAS + h * LY::N + 4 * g, sw, v, d);
                    }
                    float o[G][3];
#pragma unroll
                    for (int gi = 0; gi < G; ++gi) {
#pragma unroll
                        for (int q = 0; q < KSH; ++q)
                            d[gi][q >> 2][q & 3] = relu(d[gi][q >> 2][q & 3]);
                        output(d[gi], o[gi], [&](int c, int o16) {
                            return *reinterpret_cast<const f32x4 *>(&lds[LY::W3 + c * LY::N + 16 * o16 + 4 * g]);
                        });
                    }
                    if (check) {
                        // lanes whose partial sums reach each channel's least; a
                        // pixel with a lane that reaches all three needs no more
                        uint64_t m[G][3];
                        unsigned quick = 0xffff;
#pragma unroll
                        for (int gi = 0; gi < G; ++gi) {
                            m[gi][0] = __builtin_amdgcn_ballot_w64(fabsf(o[gi][0]) >= th0);
                            m[gi][1] = __builtin_amdgcn_ballot_w64(fabsf(o[gi][1]) >= th1);
                            m[gi][2] = __builtin_amdgcn_ballot_w64(fabsf(o[gi][2]) >= th2);
                            quick &= columns(m[gi][0] & m[gi][1] & m[gi][2]);
                        }
                        if (quick != 0xffff)
#pragma unroll
                            for (int gi = 0; gi < G; ++gi) {
                                const unsigned ok = columns(m[gi][0]) & columns(m[gi][1]) & columns(m[gi][2]);
                                again |= (ok != 0xffff ? 1u : 0u) << (rr * TWG + cg + gi);
                            }
                    }
#pragma unroll
                    for (int gi = 0; gi < G; ++gi) {
                        const float v = __builtin_fmaf(row_sum3(o[gi][0], o[gi][1], o[gi][2]), inv_t, ob);
                        if (g < 3 && tx0 + 16 * (cg + gi) + col < W)
                            store_out(p, orow + 16 * (cg + gi), v);
                    }
                }
            }
        } else if (rows > 0) {
            again = ~0u >> (32 - rows * TWG);
        }
        if (again != 0) {
            // fp32 matrix instructions (v_mfma_f32_16x16x4_f32: A[i][g],
            // B[g][i] from lane l, the same D), the products in binary32 as
            // they stand, the weights and biases from global memory through
            // raw buffers (0 past the array's end; inputs past a layer's: an
            // offset past it).  The levels' scales come off exactly.
            // (Latency of the weights binds it: with four K steps' in flight and G
            // groups per read, every tile of 3840x2160, 8 -> 64 -> 64 -> 3, takes
            // 2080 us, of which one step and one group took 3890, and the fp32
            // family 616; one tile of 768x512, 7 -> 40 -> 40 -> 3, adds 5 us to 18,
            // where it added 33.)
            int z = 0;    // (opaque, so that no layer's geometry is kept over the other tiles)
            asm volatile("" : "+s"(z));
            float back[LS];
#pragma unroll
            for (int q = 0; q < LS; ++q)
                back[q] = raw ? 1.0f : level_unscale(lds[LY::CSCALE + 4 * q + g]) * inv_t;
            auto ld = [](__amdgpu_buffer_rsrc_t r, unsigned at) {
                return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, at, 0, 0));
            };
            constexpr int kAhead = 4;    // K steps whose weights are in flight together
            auto layer = [&](int l, auto &d, auto in, int kq) {
                const LayerParams lp = layer_params(p, l + z, b);
                const unsigned fin = p.widths[l + z], fout = p.widths[l + z + 1];
                const auto wb = raw_buffer(lp.w, fin * fout * 4), bb = raw_buffer(lp.b, fout * 4);
                // (opaque, so that no operand or its address is kept over the
                // tiles that do not come here)
                unsigned n0 = row_neuron(col), k0 = g;
                asm volatile("" : "+v"(n0), "+v"(k0)::"memory");
#pragma unroll
                for (int o = 0; o < NB; ++o)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float v = ld(bb, (16 * o + 4 * r + k0) * 4);
#pragma unroll
                        for (int gi = 0; gi < G; ++gi)
                            d[gi][o][r] = v;
                    }
#pragma unroll
                for (int q0 = 0; q0 < kq; q0 += kAhead) {
                    asm volatile("" : "+v"(n0), "+v"(k0)::"memory");
                    float w[kAhead][NB];
#pragma unroll
                    for (int q = q0; q < kq && q < q0 + kAhead; ++q) {
                        const unsigned k = 4 * q + k0, at = k < fin ? (n0 * fin + k) * 4 : 0x40000000u;
#pragma unroll
                        for (int o = 0; o < NB; ++o)
                            w[q - q0][o] = ld(wb, at + 16 * o * fin * 4);
                    }
#pragma unroll
                    for (int q = q0; q < kq && q < q0 + kAhead; ++q)
#pragma unroll
                        for (int o = 0; o < NB; ++o)
#pragma unroll
                            for (int gi = 0; gi < G; ++gi)
                                d[gi][o] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[q - q0][o], in(gi, q), d[gi][o], 0, 0, 0);
                }
            };
#pragma unroll 1
            for (int i = 0; i < rows * TWG; i += G) {
                const unsigned mine = again >> i & ((1u << G) - 1);
                if (mine == 0)
                    continue;
                const int yr = RPW * wave + i / TWG, cg = i % TWG;
                float u[G][LS];
                f32x4 d[G][NB];
#pragma unroll
                for (int gi = 0; gi < G; ++gi) {
                    sample(yr, cg + gi, u[gi]);
#pragma unroll
                    for (int q = 0; q < LS; ++q)
                        u[gi][q] = 4 * q + g < L ? u[gi][q] * back[q] : 0.0f;
                }
                layer(0, d, [&](int gi, int q) { return u[gi][q]; }, LS);
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    float v[G][KSH];
#pragma unroll
                    for (int gi = 0; gi < G; ++gi)
#pragma unroll
                        for (int q = 0; q < KSH; ++q)
                            v[gi][q] = relu(d[gi][q >> 2][q & 3]);
                    layer(1 + h, d, [&](int gi, int q) { return v[gi][q]; }, KSH);
                }
                const unsigned NL = p.widths[NH + 1 + z];
                const auto w3b = raw_buffer(layer_params(p, NH + 1 + z, b).w, 3 * NL * 4);
#pragma unroll
                for (int gi = 0; gi < G; ++gi) {
#pragma unroll
                    for (int q = 0; q < KSH; ++q)
                        d[gi][q >> 2][q & 3] = relu(d[gi][q >> 2][q & 3]);
                    float o[3];
                    unsigned n0 = g;
                    output(d[gi], o, [&](int c, int o16) {
                        f32x4 w;
                        if (c == 0)    // (a block's weights in flight at a time)
                            asm volatile("" : "+v"(n0)::"memory");
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const unsigned n = 16 * o16 + 4 * r + n0;
                            w[r] = ld(w3b, n < NL ? (c * NL + n) * 4 : 0x40000000u);
                        }
                        return w;
                    });
                    const float v = row_sum3(o[0], o[1], o[2]) + ob;
                    if ((mine >> gi & 1) && g < 3 && tx0 + 16 * (cg + gi) + col < W)
                        store_out(p, obase + pixel_index(ty0 + yr, W, tx0 + 16 * (cg + gi) + col), v);
                }
            }
        }
        if (!dynamic)
            break;    // uniform: one tile per workgroup
        if (tid == 0)
            s_next = ts.base + ticket;
        __syncthreads();
        t = s_next;
        if (t >= ts.end)
            break;    // uniform
    }
}

int hidden_blocks(int nl, const int32_t *widths);

// Values per lane group of the hidden activations: ceil(width / 4) of the
// widest hidden layer (the last one feeds the output layer, so it counts too).
int hidden_values(int nl, const int32_t *widths);

template <int NB, int NH, int LS, int KSH, int RPW>
hipError_t launch_rows(const DecodeParams &p, hipStream_t s, int tiles_x, int tiles, int bpi)
{
    const int64_t nblocks = (int64_t)bpi * p.batch;
    if (nblocks > 0x7fffffff)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_mfma_f16x3<NB, NH, LS, KSH, RPW>), dim3((unsigned)nblocks), dim3(kThreads), 0, s, p,
                       bpi, tiles_x, tiles, tile_row_recip(tiles_x, tiles));
    return hipGetLastError();
}

// 32- or 16-row tiles when every workgroup of the launch averages two or
// more of them and the taller boxes keep 4 wavefronts per SIMD (or the 8-row
// instance's occupancy, if lower), else 8-row, as in the bf16 family.  (32
// rows against 16: 2048x1536 x 16 1204 -> 1173 us, 768x512 x 64 516 -> 513.)
template <int NB, int NH, int LS, int KSH>
hipError_t launch(const DecodeParams &p, hipStream_t s, int num_cus)
{
    const int tiles_x = (p.W + TW - 1) / TW;
    const int tiles8 = tiles_x * ((p.H + TH - 1) / TH);
    const int tiles16 = tiles_x * ((p.H + 4 * kWaves - 1) / (4 * kWaves));
    const int tiles32 = tiles_x * ((p.H + 8 * kWaves - 1) / (8 * kWaves));
    static int occ8 = 0, occ16 = 0, occ32 = 0;   // workgroups per CU of each instance
    const int bpi8 = blocks_per_image(k_mfma_f16x3<NB, NH, LS, KSH, 2>, p, num_cus, tiles8, occ8);
    const int bpi16 = blocks_per_image(k_mfma_f16x3<NB, NH, LS, KSH, 4>, p, num_cus, tiles16, occ16);
    const int bpi32 = blocks_per_image(k_mfma_f16x3<NB, NH, LS, KSH, 8>, p, num_cus, tiles32, occ32);
    const int occ_need = occ8 < 4 ? occ8 : 4;
    if (occ32 >= occ_need && tiles32 >= 2 * bpi32)
        return launch_rows<NB, NH, LS, KSH, 8>(p, s, tiles_x, tiles32, bpi32);
    if (occ16 >= occ_need && tiles16 >= 2 * bpi16)
        return launch_rows<NB, NH, LS, KSH, 4>(p, s, tiles_x, tiles16, bpi16);
    return launch_rows<NB, NH, LS, KSH, 2>(p, s, tiles_x, tiles8, bpi8);
}

template <int NH>
hipError_t launch_nh(const DecodeParams &p, hipStream_t s, int num_cus)
{
    const int NB = hidden_blocks(p.nl, p.widths);
    const int LS = (p.L + 3) / 4;
    // Width 33..40 (three blocks, last one half used) gets its own value
    // count; every other width runs all 4 NB values over zero padding.
    const bool k10 = NH > 0 && NB == 3 && hidden_values(p.nl, p.widths) <= 10;
#define PIC_CASE(nb, ls, ksh) \
    if (NB == nb && LS == ls && (ksh != 4 * nb) == (nb == 3 && k10)) return launch<nb, NH, ls, ksh>(p, s, num_cus);
    PIC_CASE(1, 1, 4) PIC_CASE(1, 2, 4) PIC_CASE(1, 3, 4)
    PIC_CASE(2, 1, 8) PIC_CASE(2, 2, 8) PIC_CASE(2, 3, 8)
    PIC_CASE(3, 1, 12) PIC_CASE(3, 2, 12) PIC_CASE(3, 3, 12)
    PIC_CASE(4, 1, 16) PIC_CASE(4, 2, 16) PIC_CASE(4, 3, 16)
    if constexpr (NH > 0) {
        PIC_CASE(3, 1, 10) PIC_CASE(3, 2, 10) PIC_CASE(3, 3, 10)
    }
#undef PIC_CASE
    return hipErrorInvalidValue;
}

// Nets 65 to 128 wide: six or eight blocks, one group of pixels a pass.  With a
// hidden matrix their operands leave room for one or two workgroups in a CU's
// LDS (1 or 2 wavefronts per SIMD), without one 20 to 43 KB for two or three;
// the eight-block instances of two hidden matrices take all 256 VGPRs and some
// AGPRs.  The vector family, which evaluates a pixel per lane at 13 TFLOP/s,
// against these: 768x512, 8 -> 96 -> 96 -> 3: 604 -> 39 us, 8 -> 128 -> 128 -> 128
// -> 3: 1772 -> 103, 4 -> 100 -> 3: 86 -> 16; 64x64, 12 -> 128 -> 128 -> 3: 156 -> 32.
// (wide_fits: the operands of a 128-wide net with two hidden matrices do not
// fit the LDS with more than 8 levels, nor with 16-row tiles from 5 levels on.)
constexpr int kWideLds = 160 * 1024;
template <int NB, int NH, int LS, int RPW>
constexpr bool wide_fits = Layout<NB, NH, LS, 4 * NB, RPW * kWaves>::SIZE * 4 + 64 <= kWideLds;

template <int NB, int NH, int LS>
hipError_t launch_wide_one(const DecodeParams &p, hipStream_t s, int num_cus)
{
    if constexpr (wide_fits<NB, NH, LS, 2>) {
        const int tiles_x = (p.W + TW - 1) / TW;
        const int tiles8 = tiles_x * ((p.H + TH - 1) / TH);
        static int occ8 = 0;
        const int bpi8 = blocks_per_image(k_mfma_f16x3<NB, NH, LS, 4 * NB, 2>, p, num_cus, tiles8, occ8);
        if constexpr (wide_fits<NB, NH, LS, 4>) {
            const int tiles16 = tiles_x * ((p.H + 4 * kWaves - 1) / (4 * kWaves));
            static int occ16 = 0;
            const int bpi16 = blocks_per_image(k_mfma_f16x3<NB, NH, LS, 4 * NB, 4>, p, num_cus, tiles16, occ16);
            if (occ16 >= occ8 && tiles16 >= 2 * bpi16)
                return launch_rows<NB, NH, LS, 4 * NB, 4>(p, s, tiles_x, tiles16, bpi16);
        }
        return launch_rows<NB, NH, LS, 4 * NB, 2>(p, s, tiles_x, tiles8, bpi8);
    } else {
        return hipErrorInvalidValue;
    }
}

template <int NH>
hipError_t launch_wide_nh(const DecodeParams &p, hipStream_t s, int num_cus)
{
    const bool six = hidden_blocks(p.nl, p.widths) <= 6;
    switch ((p.L + 3) / 4) {
    case 1: return six ? launch_wide_one<6, NH, 1>(p, s, num_cus) : launch_wide_one<8, NH, 1>(p, s, num_cus);
    case 2: return six ? launch_wide_one<6, NH, 2>(p, s, num_cus) : launch_wide_one<8, NH, 2>(p, s, num_cus);
    case 3: return six ? launch_wide_one<6, NH, 3>(p, s, num_cus) : launch_wide_one<8, NH, 3>(p, s, num_cus);
    }
    return hipErrorInvalidValue;
}

}  // namespace mfma_f16x3
}  // namespace pic
