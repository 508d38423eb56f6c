// The paper-size autoencoder (Sec. IV-C, Table I: 1-64-128-256-64-4; Table II: 4-4-32-64-128-32-1), each stack as
// one launch on the bf16 matrix cores, in fp32 precision (gfx950, wave64, v_mfma_f32_32x32x16_bf16).
//
// A block takes a short run of latent positions through all layers.  The layers' windows overlap by one position
// per layer only (31 positions of conv3, 63 of conv2, 127 of conv1 for 15 latent ones), so recomputing the edges
// costs 3-6 % of the arithmetic, and no intermediate tensor leaves the LDS: what a block moves is its input, its
// output and the weights, which it streams from the L2.
//
// fp32 precision from bf16 products: every fp32 operand is the exact sum of three bf16 numbers
// (x = h + m + l: h = bf16(x), m = bf16(x - h), l = x - h - m has at most 8 bits left), and
//   x w = h h' + (h m' + m h') + (m m' + h l' + l h') + terms below 2^-26 |x w|
// so six bf16 products, exact in the fp32 accumulators' input, take the place of one fp32 product.  The matrix
// cores run bf16 at 16 times the fp32 rate: 2.7 times fewer matrix-core cycles for the same precision (the sums are
// rounded once per 16 products instead of once per 2).  The last layer of each stack adds its few products per output in
// 64 bits: the cost cannot be told from none (4 x 25 600: 26.0 us either way), and in 32 bits those sums were over half
// of the latent's error.
// Measured against one fp32-MFMA launch per deep layer (ae_mfma.hip, which other stacks still use): 4 nodes x 25 600
// values, encoder 79.4 -> 26.7 us (165 TFLOP/s of fp32 products), decoder 58.0 -> 19.0 us (141); 8 x 67 000, both
// together 468 -> 212 us (175); 1 x 1 023 (latency) 79 -> 20.0 us (one card, two directions; other cards take up to 5 % less).
// Relative error against 64 bits, six sizes from 1 x 500 to 8 x 67 000 x six seeds, mean (least to largest): latent
// 1.32e-7 (0.93 to 2.48) -> 0.46e-7 (0.32 to 0.83), decoder 8.8e-8 (2.2 to 31.6) -> 5.3e-8 (1.9 to 16.8): lower at every
// size with every seed.  What bounds it: while a compute unit has blocks its matrix cores are busy 56-59 % of the cycles
// (encoder) and 43-51 % (decoder).  A wavefront's products, once begun, hold them until it waits; what else its block has
// to do goes on beside another wavefront's products only where no barrier stands between.
//
// The split is exact only for finite values; an Inf would meet products of both signs.  Such a value (or one that rounds
// to Inf) leaves a NaN among its parts, which makes every output it reaches a NaN.  And it is exact only while the parts
// are normal numbers: these matrix instructions take smaller ones for zero, so parts below 2^-126 are lost.  What that can
// do to an output has a bound that the weights give (fused_limits).  A block with an output that is not finite, or is
// small enough for the bound to matter, redoes its outputs in plain fp32 on the fp32 matrix cores, which keep small numbers
// (inputs of about 1e-33, no biases: the reconstruction is 5.7e-7 off; 9.4e-4 without the redo, 7.3e-7 with fp32
// launches).  Every block doing so: 4 nodes x 25 600 values, encoder 25 -> 92 us, decoder 18 -> 50 us; 8 x 67 000: 114 -> 424
// and 74 -> 213 us; 1 x 1 023: 12 -> 55 and 8 -> 23 us (one fp32-MFMA launch per layer: 83, 59, 270 and 194 us for the
// first four; one position after the other on the vector units: 3.3, 1.6, 16 and 8 ms).
//
// Operand layout of v_mfma_f32_32x32x16_bf16: lane l supplies A[i = l % 32][k = 8 (l / 32) + 0..7] and
// B[k = 8 (l / 32) + 0..7][j = l % 32]; result r of 16 is C[i = 8 (r / 4) + 4 (l / 32) + r % 4][j = l % 32].  Here
// i is the output channel, j the position, k runs over 16 input channels of one tap.  Weights are laid out in this
// order when the handle is created (fragments of 1 KB, a step's three parts one after the other), activations are
// kept in the LDS position by position, [h | m | l][channels], so that every operand is one 16-byte read per lane.  Rows are
// padded by 16 bytes: eight neighbouring positions then start in eight different groups of banks.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "lgc_internal.h"

namespace lgc {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef float acc16 __attribute__((ext_vector_type(16)));
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

namespace {

__device__ __forceinline__ float leaky_f(float x, float slope) { return x > 0.f ? x : slope * x; }

// The non-linearity at a position: the factors of positive and other values, both 0 where the position does not exist.  A sum that is
// not finite leaves a NaN there, where a 0 belongs: right for the split's pass alone, whose NaNs make the block redo its outputs.
struct Act {
    float pos, neg;
    __device__ __forceinline__ Act(const float slope, const bool valid) : pos(valid ? 1.f : 0.f), neg(valid ? slope : 0.f) {}
    __device__ __forceinline__ float operator()(const float x) const { return x * (x > 0.f ? pos : neg); }
};

// Two values split into three bf16 pairs.  What a part leaves is taken by one instruction a value, a - h.lo * 1 + h.hi * 0 and
// the like, exact as there is nothing to round (by shift or mask and subtraction two; with the choice of factors above,
// 8 x 67 000 values, encoder 132.9 -> 130.7 us, decoder 82.8 -> 80.4).  A value that is not finite, or rounds to Inf, leaves
// NaNs among the parts of both.
// The factors come in scalar registers: as constants within the instruction they would go to the wrong halves.
__device__ __forceinline__ void split2(const float a, const float b, uint32_t &h, uint32_t &m, uint32_t &l) {
    uint32_t minus_lo = 0x0000bf80u, minus_hi = 0xbf800000u;
    asm("" : "+s"(minus_lo), "+s"(minus_hi));
    const bf2 lo = __builtin_bit_cast(bf2, minus_lo), hi = __builtin_bit_cast(bf2, minus_hi);
    const bf2 x = __builtin_convertvector((f2v){a, b}, bf2);
    const float ra = __builtin_amdgcn_fdot2_f32_bf16(x, lo, a, false), rb = __builtin_amdgcn_fdot2_f32_bf16(x, hi, b, false);
    const bf2 y = __builtin_convertvector((f2v){ra, rb}, bf2);
    const float sa = __builtin_amdgcn_fdot2_f32_bf16(y, lo, ra, false), sb = __builtin_amdgcn_fdot2_f32_bf16(y, hi, rb, false);
    h = __builtin_bit_cast(uint32_t, x);
    m = __builtin_bit_cast(uint32_t, y);
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2v){sa, sb}, bf2));
}

// acc[i][j] + cross[i][j] += A[i] B[j] for one step of 16 input channels, both operands in three parts.  The five
// products that hold an m or an l have sums of their own: rounded at their own, 2^8 times smaller size, they leave
// the large sum one rounding per step instead of six.  The tiles are taken in turn, so that consecutive
// instructions do not wait for each other's sums.
template <int MT, int NT>
__device__ __forceinline__ void mma6(acc16 (&acc)[MT][NT], acc16 (&cross)[MT][NT], const u4v (&a)[MT][3], const u4v (&b)[NT][3]) {
    constexpr int kA[6] = {2, 0, 1, 1, 0, 0}, kB[6] = {0, 2, 1, 0, 1, 0};   // parts h, m, l = 0, 1, 2
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                acc16 &c = q < 5 ? cross[i][j] : acc[i][j];
                c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a[i][kA[q]]), __builtin_bit_cast(bf8, b[j][kB[q]]), c, 0, 0, 0);
            }
}

// sum[i] + cross[i] += a[i] x for one step, as in mma6 (the five products that hold an m or an l have sums of their own)
template <int N>
__device__ __forceinline__ void mma6_by(acc16 (&sum)[2], acc16 (&cross)[2], const u4v (&a)[N][3], const u4v (&x)[3]) {
    constexpr int kA[6] = {2, 0, 1, 1, 0, 0}, kB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            acc16 &c = q < 5 ? cross[i] : sum[i];
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, a[i][kA[q]]), __builtin_bit_cast(bf8, x[kB[q]]), c, 0, 0, 0);
        }
}

// The four outputs of two transposed layers in a row: e, o = the first one's outputs 2i and 2i + 1, n = its 2i + 2;
// a = taps 2, 1, 0
__device__ __forceinline__ void mma6_up4(acc16 (&y)[4], const u4v (&a)[3][3], const u4v (&e)[3], const u4v (&o)[3], const u4v (&n)[3]) {
    constexpr int kA[6] = {2, 0, 1, 1, 0, 0}, kB[6] = {0, 2, 1, 0, 1, 0};
    auto mul = [](const u4v &p, const u4v &q, const acc16 &c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8, p), __builtin_bit_cast(bf8, q), c, 0, 0, 0);
    };
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        y[1] = mul(a[0][kA[q]], e[kB[q]], y[1]);
        y[3] = mul(a[0][kA[q]], o[kB[q]], y[3]);
        y[0] = mul(a[1][kA[q]], e[kB[q]], y[0]);
        y[2] = mul(a[1][kA[q]], o[kB[q]], y[2]);
        y[1] = mul(a[2][kA[q]], o[kB[q]], y[1]);
        y[3] = mul(a[2][kA[q]], n[kB[q]], y[3]);
    }
}

// A result tile that starts from the bias of its channels co0 + 8 (r / 4) + 4 half + r % 4
__device__ __forceinline__ acc16 bias16(const float *__restrict__ bias, const int co0, const int half) {
    acc16 z;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const f4v b = *(const f4v *)(bias + co0 + 8 * g + 4 * half);
#pragma unroll
        for (int c = 0; c < 4; ++c) z[4 * g + c] = b[c];
    }
    return z;
}

__device__ __forceinline__ acc16 zero16() {
    acc16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}

// Bytes of one position with C channels in the LDS: three parts, 16 bytes of padding.
constexpr int row_bytes(int c) { return 6 * c + 16; }

// Four consecutive channels of one position, co on, split and stored.  AS_RESULTS: to where weights laid out `as_results` meet them.
template <int C, bool AS_RESULTS>
__device__ __forceinline__ void store_split(unsigned char *row, const int co, const float (&y)[4]) {
    const int at = AS_RESULTS ? (co & ~15) + 2 * (co & 4) + ((co & 8) >> 1) : co;
    u2v h, m, l;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        uint32_t x, z, w;
        split2(y[2 * c], y[2 * c + 1], x, z, w);
        h[c] = x; m[c] = z; l[c] = w;
    }
    *(u2v *)(row + 2 * at) = h;
    *(u2v *)(row + 2 * C + 2 * at) = m;
    *(u2v *)(row + 4 * C + 2 * at) = l;
}

// One 32 x 32 result tile with the non-linearity into the LDS: `row` is the lane's position, channels
// co0 + 8 (r / 4) + 4 half + r % 4.  Positions that do not exist (valid false) hold zeros.
template <int C, bool AS_RESULTS = false>
__device__ __forceinline__ void store_tile(unsigned char *row, const int co0, const int half, const acc16 &acc,
                                           const float slope, const bool valid) {
    const Act act(slope, valid);
#pragma unroll
    for (int g = 0; g < 4; ++g)
        store_split<C, AS_RESULTS>(row, co0 + 8 * g + 4 * half, {act(acc[4 * g]), act(acc[4 * g + 1]), act(acc[4 * g + 2]), act(acc[4 * g + 3])});
}

// One result tile with the non-linearity as operands of the next layer, 16 channels a step: r[step][part] (weights `as_results`)
__device__ __forceinline__ void as_operands(const acc16 &acc, const float slope, const bool valid, u4v (&r)[2][3]) {
    const Act act(slope, valid);
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
        uint32_t h, m, l;
        split2(act(acc[i]), act(acc[i + 1]), h, m, l);
        r[i >> 3][0][(i & 7) >> 1] = h; r[i >> 3][1][(i & 7) >> 1] = m; r[i >> 3][2][(i & 7) >> 1] = l;
    }
}

// The same of the next lane's position (of the last lane of each half: whatever)
__device__ __forceinline__ void next_position(const u4v (&r)[2][3], u4v (&n)[2][3]) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < 4; ++i) n[q][p][i] = __builtin_amdgcn_update_dpp(0u, r[q][p][i], 0x130 /* wave_shl:1 */, 0xf, 0xf, true);
}

// ---- weights as bf16 fragments --------------------------------------------------------------------
// out[((mt * steps + s) * 3 + part) * 512 + lane * 8 + e], s = tap * (c_in / 16) + ci / 16: part `part` of
// w[co = 32 mt + lane % 32][ci = 16 (s % (c_in / 16)) + 8 (lane / 32) + e][tap].  One thread per (mt, s, lane).
// as_results: element e of half h is input channel 4 h + e (e < 4) or 8 + 4 h + e - 4 of the 16 instead, which is where a lane of
// the layer before holds them among its results: those then are operands without leaving their registers.
// *bad counts the weights that are not finite (the handle then keeps to the fp32 kernels).
__global__ __launch_bounds__(256) void k_weights_split(const float *__restrict__ w, uint16_t *__restrict__ out, int c_in, int c_out,
                                                       int transposed, int as_results, uint32_t *bad) {
    const int steps = 3 * (c_in / 16), total = (c_out / 32) * steps * 64;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int lane = i & 63, s = (i >> 6) % steps, mt = (i >> 6) / steps;
    const int tap = s / (c_in / 16), co = 32 * mt + (lane & 31), ci0 = 16 * (s % (c_in / 16));
    const int half = lane >> 5;
    uint16_t *o = out + (size_t)((i >> 6) * 3) * 512 + lane * 8;
    float chk = 0.f;
    for (int e = 0; e < 8; e += 2) {
        float x[2];
        for (int c = 0; c < 2; ++c) {
            const int i = e + c, ci = ci0 + (as_results ? 8 * (i >> 2) + 4 * half + (i & 3) : 8 * half + i);
            x[c] = transposed ? w[((size_t)ci * c_out + co) * 3 + tap] : w[((size_t)co * c_in + ci) * 3 + tap];
        }
        uint32_t h, m, l;
        split2(x[0], x[1], h, m, l);
        chk = fmaf(__uint_as_float(m << 16), 0.f, fmaf(__uint_as_float(m & 0xffff0000u), 0.f, chk));   // a NaN if a part is one
        *(uint32_t *)(o + e) = h;
        *(uint32_t *)(o + 512 + e) = m;
        *(uint32_t *)(o + 1024 + e) = l;
    }
    if (chk != chk) atomicAdd(bad, 1u);
}

// *most = the largest magnitude (bits) of w, from zero on
__global__ __launch_bounds__(256) void k_most(const float *__restrict__ w, int count, uint32_t *most) {
    uint32_t m = 0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < count; i += gridDim.x * 256) { const uint32_t x = __float_as_uint(w[i]) & 0x7fffffffu; m = x > m ? x : m; }
    atomicMax(most, m);
}

}  // namespace

void launch_weights_split(const float *w, uint16_t *out, int c_in, int c_out, bool transposed, bool as_results, uint32_t *bad, hipStream_t st) {
    const int total = (c_out / 32) * 3 * (c_in / 16) * 64;
    hipLaunchKernelGGL(k_weights_split, dim3((total + 255) / 256), dim3(256), 0, st, w, out, c_in, c_out, (int)transposed, (int)as_results, bad);
}

void launch_most(const float *w, int count, uint32_t *most, hipStream_t st) {
    hipLaunchKernelGGL(k_most, dim3((count + 2047) / 2048), dim3(256), 0, st, w, count, most);
}

// How far an output can be off because numbers below 2^-126 count as zero in the split's products: a stored value loses up to
// two parts, a product of up to 6 terms per input is off by as many such numbers, and a layer passes on what comes in times
// its largest weight times its inputs per output (and the slope, if that enlarges).  An output 2^24 times as large does not
// feel it.  Weights lose parts too: a layer whose largest one is 2^25 times 2^-126 loses no more than
// rounding would.
bool fused_limits(const LayerDev *l, int split, const float *most, bool transposed, float slope, bool no_bias, FusedLimits &out) {
    const double tiny = ldexp(1.0, -126), steep = fmax(1.0, fabs((double)slope));
    double off = 0.0;
    for (int i = 0; i < split; ++i) {
        if (most[i] != 0.f && most[i] < ldexpf(1.f, -101)) return false;
        const double inputs = (transposed ? 2.0 : 3.0) * l[i].c_in;
        off = steep * inputs * (most[i] * (off + 2 * tiny) + 6 * tiny);
    }
    off *= (double)most[split] * l[split].c_in;
    out.least = (float)ldexp(off, 24);
    out.no_bias = no_bias;
    return out.least <= ldexpf(1.f, -40);   // (also no NaN: weights so large that usual outputs would all be redone)
}

// ---- encoder ---------------------------------------------------------------------------------------
// Four kernel-3 / stride-2 layers 1 -> C1 -> C2 -> C3 -> C4 and a kernel-1 layer C4 -> C5.

struct EncoderDev {
    const float *w1, *b1;                       // [C1][1][3]
    const float *w2, *w3, *w4, *b2, *b3, *b4;   // [c_out][c_in][3]
    const uint16_t *s2, *s3, *s4;               // the same as bf16 fragments
    const float *w5, *b5;                       // [C5][C4][1]
    FusedLimits limits;
};

namespace {

// Fragments of one step of 16 input channels: the three parts of one tap
__device__ __forceinline__ void load_a(u4v (&r)[3], const u4v *__restrict__ a, const int step) {
#pragma unroll
    for (int p = 0; p < 3; ++p) r[p] = a[(step * 3 + p) * 64];
}

// The order of one step's instructions: a read from the LDS, then a load, behind each product in turn, which they then cost no
// time beside (ahead of the products they are issued while the matrix cores wait; a block of 31 positions 57.4 -> 54.5 K
// cycles, 8 x 67 000 values 129.4 -> 127.9 us, as the clock falls with the denser products; the decoder's steps, 8 x 67 000
// 82.4 -> 80.8, 1 x 1 023 8.5 -> 8.2).
template <int MMAS, int READS, int LOADS>
__device__ __forceinline__ void interleave() {
#pragma unroll
    for (int i = 0; i < MMAS; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (i < READS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        else if (i < READS + LOADS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
}

// The K loop of one convolution for MT x NT tiles: STEPS steps of 16 input channels.  where(j, s): the LDS address of this
// lane's position of tile j for step s.  frag(i, s): this lane's fragments of tile i.  They come from the L2: AHEAD steps of
// them are kept in flight, the first ones from before the barrier that the loop waits at, and the LDS reads run one step ahead.
// interleave() keeps it that way (left to itself the compiler moves the loads down to their uses: conv4 then waits out the L2's
// latency in every step).
template <int MT, int AHEAD>
struct Fragments { u4v r[AHEAD + 1][MT][3]; };

template <int MT, int AHEAD, typename Frag>
__device__ __forceinline__ void fragments_start(Fragments<MT, AHEAD> &f, Frag frag) {
#pragma unroll
    for (int d = 0; d < AHEAD; ++d)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int p = 0; p < 3; ++p) f.r[d][i][p] = frag(i, d)[p * 64];
    __builtin_amdgcn_sched_barrier(0);
}

template <int C, int MT, int NT, int STEPS, int AHEAD, typename Frag, typename Where>
__device__ __forceinline__ void conv_mma(acc16 (&acc)[MT][NT], Fragments<MT, AHEAD> &f, Frag frag, Where where) {
    u4v rb[2][NT][3];
    auto read_b = [&](u4v (&r)[NT][3], const int s) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const unsigned char *b = where(j, s);
#pragma unroll
            for (int p = 0; p < 3; ++p) r[j][p] = *(const u4v *)(b + p * 2 * C);
        }
    };
    acc16 cross[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) cross[i][j] = zero16();
    read_b(rb[0], 0);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        if (s + AHEAD < STEPS) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int p = 0; p < 3; ++p) f.r[(s + AHEAD) % (AHEAD + 1)][i][p] = frag(i, s + AHEAD)[p * 64];
        }
        if (s + 1 < STEPS) read_b(rb[(s + 1) & 1], s + 1);
        if (NT == 1) __builtin_amdgcn_sched_barrier(0);   // (too few products to put them behind: 4 x 15 000 values 20.7 us so, 19.8 ahead of them)
        mma6<MT, NT>(acc, cross, f.r[s % (AHEAD + 1)], rb[s & 1]);
        if (NT > 1) interleave<6 * MT * NT, 3 * NT, 3 * MT>();
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] += cross[i][j];
}

// The redo in plain fp32, for blocks with a value that the split cannot carry: the same tiles and windows on the fp32 matrix
// cores (v_mfma_f32_32x32x2_f32: lane l supplies A[i = l % 32][k = l / 32] and B[k = l / 32][j = l % 32], results as above),
// activations as rows of fp32 in the same LDS.  A lane's half takes four of eight channels in turn, so that its operands are 16-byte reads.
__device__ __forceinline__ acc16 mma_fp32(const float a, const float b, const acc16 &c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

constexpr int row_floats(int c) { return c + 4; }

// acc += one tile: w = the lane's output channel [CI][3], b = its row for tap 0, `odd` floats before the odd positions',
// both from the half's first channel on.  Sums of 96 products are added up: one running sum of 768 is off twice as far.
template <int CI>
__device__ __forceinline__ void conv_fp32(acc16 &acc, const float *__restrict__ w, const float *b, const int odd) {
#pragma unroll 1
    for (int c0 = 0; c0 < CI; c0 += 32) {
        acc16 sum = zero16();
#pragma unroll 2
        for (int c = c0; c < c0 + 32; c += 8) {
            const f4v x[3] = {*(const f4v *)(b + c), *(const f4v *)(b + odd + c), *(const f4v *)(b + row_floats(CI) + c)};
            f4v y[3];
#pragma unroll
            for (int t = 0; t < 3; ++t) y[t] = *(const f4v *)(w + 3 * c + 4 * t);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int t = 0; t < 3; ++t) sum = mma_fp32(y[(3 * e + t) / 4][(3 * e + t) % 4], x[t][e], sum);
        }
        acc += sum;
    }
}

// One kernel-3 / stride-2 layer for N positions from q0 on, in place in buf; W wavefronts share the tiles out.  The outputs:
// even positions, then (after N / 2 + 1 rows) odd ones.
template <int CI, int CO, int N, int W>
__device__ __forceinline__ void layer_fp32(float *buf, const float *__restrict__ wt, const float *__restrict__ bias, const int wave,
                                           const long long q0, const long long len, const float slope) {
    constexpr int kTiles = (CO / 32) * ((N + 31) / 32), kMine = (kTiles + W - 1) / W, R = row_floats(CI), S = row_floats(CO);
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    acc16 acc[kMine];
#pragma unroll
    for (int m = 0; m < kMine; ++m) {
        const int tile = wave + m * W, co0 = tile % (CO / 32) * 32, i = tile / (CO / 32) * 32 + col;
        if (tile < kTiles) {                       // wave-uniform
            acc[m] = bias16(bias, co0, half);
            conv_fp32<CI>(acc[m], wt + (size_t)(co0 + col) * CI * 3 + 12 * half, buf + (i < N ? i : N - 1) * R + 4 * half, (N + 1) * R);
        }
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < kMine; ++m) {
        const int tile = wave + m * W, co0 = tile % (CO / 32) * 32, i = tile / (CO / 32) * 32 + col;
        if (tile < kTiles && i < N) {
            float *row = buf + ((i & 1) ? (N / 2 + 1) * S : 0) + (i >> 1) * S + co0 + 4 * half;
            const bool valid = q0 + i >= 0 && q0 + i < len;
#pragma unroll
            for (int r = 0; r < 16; ++r) row[8 * (r >> 2) + (r & 3)] = valid ? leaky_f(acc[m][r], slope) : 0.f;
        }
    }
    __syncthreads();
}

}  // namespace

namespace {

// P latent positions per block of W wavefronts.  Local numbering: conv3's position i is 2 p0 - 1 + i, conv2's 4 p0 - 3 + i,
// conv1's 8 p0 - 7 + i, the input's 16 p0 - 15 + i, so that position i of one layer takes 2i, 2i + 1, 2i + 2 of
// the layer before; 2P + 1, 4P + 3, 8P + 7 and 16P + 15 of them are needed, and the tiles hold one more.
//
// S blocks share a run of 15 positions: each makes conv1 and conv2 for itself, 1 / S of conv3's channels (whose steps several
// wavefronts share) and what those give of conv4's sums; the last one to come adds them up, in order whichever it is, and goes
// on.  Short vectors would leave most compute units idle, and draw 1 MB of weights through each one that works: 1 x 1 023
// values (5 runs) 15.9 us with a block each, 11.7 with four; 2 x 2 000 (18 runs) 16.0 / 12.1, 4 x 5 000 (84 runs, two blocks)
// 16.2 / 14.6.
template <int P, int S, int C1, int C2, int C3, int C4, int C5, int W>
struct EncoderRun {
    static constexpr int N4 = P + 1, N3 = 2 * N4, N2 = 4 * N4;   // tile widths (positions) of conv4, conv3, conv2
    static constexpr int CS = C3 / S, R1 = row_bytes(C1), R2 = row_bytes(C2), R3 = row_bytes(CS);
    static constexpr int kSplit = W / (C4 / 32);                 // conv4: wavefronts that share a tile, each a run of its steps
    static constexpr int kPart3 = S > 1 ? W * 32 * 33 * 4 : 0;   // conv3's partial sums, ahead of its rows
    static constexpr int max(int a, int b) { return a > b ? a : b; }
    static constexpr int kRedo = max(max((2 * N2 + 1) * row_floats(C1), (2 * N3 + 1) * row_floats(C2)), max((2 * N4 + 1) * row_floats(C3), 2 * (N4 / 2 + 1) * row_floats(C4))) * 4;
    static constexpr int kBytes = max(max(max((2 * N2 + 1) * R1, (2 * N3 + 1) * R2), kPart3 + (2 * N4 + 1) * R3), max(kRedo, kSplit * C4 * 33 * 4 + W * 2 * C5 * 32 * 8));
    static constexpr int kXs = 4 * N2 + 4, kSmall = 4 * C1 + C5 * C4 + C4 + C5;
    static_assert(C1 == 8 * W && C2 % 32 == 0 && CS % 32 == 0 && C4 == 64 && C3 == 32 * W && N3 % 32 == 0 && N4 <= 32 && C5 <= 4, "tiles");
    static_assert(S == 1 || P == 15 && (S == 2 || S == 4), "shares");
};

// sums: [S][C4][16] per run of positions, taken: the counts of the blocks that have come (zero between calls)
template <int P, int S, int C1, int C2, int C3, int C4, int C5, int W>
__device__ __forceinline__ void encode_run(const float *__restrict__ x, float *__restrict__ out, const EncoderDev &w, const uint32_t l0, const uint32_t l1,
                                           const uint32_t l2, const uint32_t l3, const uint32_t l4, const float slope, const long long p0, const int share,
                                           float *sums, uint32_t *taken, unsigned char *buf, float *xs, float *small) {
    using K = EncoderRun<P, S, C1, C2, C3, C4, C5, W>;
    constexpr int N4 = K::N4, N3 = K::N3, N2 = K::N2, CS = K::CS, R1 = K::R1, R2 = K::R2, R3 = K::R3, kSplit = K::kSplit;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    // the small layers' weights and biases
    constexpr int kB1 = 3 * C1, kW5 = kB1 + C1, kB4 = kW5 + C5 * C4, kB5 = kB4 + C4;
    static_assert(kB4 == W * 64 && K::kSmall == kB5 + C5 && C4 + C5 <= W * 64, "a word per thread, and one more for some");

    // conv1: a wavefront takes 8 channels at 64 positions at a time; put(position, values)
    auto conv1 = [&](auto put) {
        f4v wt[6], bias[2];
#pragma unroll
        for (int i = 0; i < 6; ++i) wt[i] = *(const f4v *)(small + wave * 24 + 4 * i);
#pragma unroll
        for (int i = 0; i < 2; ++i) bias[i] = *(const f4v *)(small + kB1 + wave * 8 + 4 * i);
#pragma unroll 1
        for (int i = lane; i < 2 * N2; i += 64) {
            const long long q = 8 * p0 - 7 + i;
            const Act act(slope, q >= 0 && q < (long long)l1);
            const float x0 = xs[2 * i], x1 = xs[2 * i + 1], x2 = xs[2 * i + 2];
            float y[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                auto tap = [&](const int t) { return wt[(3 * c + t) / 4][(3 * c + t) % 4]; };
                y[c] = act(fmaf(tap(2), x2, fmaf(tap(1), x1, fmaf(tap(0), x0, bias[c / 4][c % 4]))));
            }
            put(i, y);
        }
    };
    const float s0 = *(tid < kB1 ? w.w1 + tid : tid < kW5 ? w.b1 + tid - kB1 : w.w5 + tid - kW5);
    const float s1 = *(tid < C4 ? w.b4 + tid : w.b5 + (tid < C4 + C5 ? tid - C4 : 0));
    for (int i = tid; i < 4 * N2 + 3; i += W * 64) {
        const long long e = 16 * p0 - 15 + i;
        xs[i] = e >= 0 && e < (long long)l0 ? x[e] : 0.f;
    }
    small[tid] = s0;
    if (tid < C4 + C5) small[kB4 + tid] = s1;
    __syncthreads();
    conv1([&](const int i, const float (&y)[8]) {
        u4v h, m, l;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            uint32_t a, b, d;
            split2(y[2 * c], y[2 * c + 1], a, b, d);
            h[c] = a; m[c] = b; l[c] = d;
        }
        unsigned char *row = buf + ((i & 1) ? (N2 + 1) * R1 : 0) + (i >> 1) * R1 + wave * 16;
        *(u4v *)row = h;
        *(u4v *)(row + 2 * C1) = m;
        *(u4v *)(row + 4 * C1) = l;
    });

    {   // conv2: C2 / 32 channel tiles x N2 / 32 position tiles
        constexpr int kM = C2 / 32, kNW = W / kM, NT = N2 / 32 / kNW, kPer = C1 / 16, kSteps = 3 * kPer, kAhead = 2;
        static_assert(W % kM == 0 && (N2 / 32) % kNW == 0, "conv2 tiles");
        const int mt = wave / kNW, n0 = (wave % kNW) * NT;
        const u4v *a = (const u4v *)w.s2 + (size_t)mt * kSteps * 192 + lane;
        auto frag = [&](int, const int s) { return a + s * 192; };
        Fragments<1, kAhead> f;
        fragments_start(f, frag);
        acc16 acc[1][NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[0][j] = bias16(w.b2, mt * 32, half);
        const unsigned char *b[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) b[j] = buf + ((n0 + j) * 32 + col) * R1 + half * 16;
        __syncthreads();
        conv_mma<C1, 1, NT, kSteps, kAhead>(acc, f, frag, [&](const int j, const int s) {
            const int tap = s / kPer;
            return b[j] + (tap == 1 ? (N2 + 1) * R1 : (tap >> 1) * R1) + 32 * (s % kPer);
        });
        __syncthreads();   // conv1's outputs have been read
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int i = (n0 + j) * 32 + col;
            const long long q = 4 * p0 - 3 + i;
            unsigned char *row = buf + ((i & 1) ? (N3 + 1) * R2 : 0) + (i >> 1) * R2;
            store_tile<C2>(row, mt * 32, half, acc[0][j], slope, q >= 0 && q < (long long)l2 && i < N2 - 1);
        }
    }

    float *part = (float *)buf;                               // conv4's partial sums [kSplit][C4][33]
    double *red = (double *)(part + kSplit * C4 * 33);         // conv5's [W * 2][C5][32]
    static_assert(kSplit * C4 * 33 % 2 == 0, "partial sums");
    constexpr int kPer2 = C2 / 16, kPer3 = C3 / 16;
    {
        unsigned char *rows3 = buf + K::kPart3;
        {   // conv3: a channel tile is shared by S wavefronts, each a run of its steps
            constexpr int NT = N3 / 32, kSteps = 3 * kPer2 / S, kAhead = 1;
            static_assert(S == 1 || NT == 1, "one tile to share");
            const int mt = wave / S, s0 = (wave % S) * kSteps;
            const u4v *a = (const u4v *)w.s3 + (size_t)((share * (CS / 32) + mt) * 3 * kPer2 + s0) * 192 + lane;
            auto frag = [&](int, const int s) { return a + s * 192; };
            Fragments<1, kAhead> f;
            fragments_start(f, frag);
            acc16 acc[1][NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                if (S == 1) acc[0][j] = bias16(w.b3, mt * 32, half);
                else acc[0][j] = zero16();
            }
            const unsigned char *b[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) b[j] = buf + (j * 32 + col) * R2 + half * 16;
            __syncthreads();
            conv_mma<C2, 1, NT, kSteps, kAhead>(acc, f, frag, [&](const int j, const int s) {
                const int tap = (s0 + s) / kPer2;
                return b[j] + (tap == 1 ? (N3 + 1) * R2 : (tap >> 1) * R2) + 32 * ((s0 + s) % kPer2);
            });
            __syncthreads();
            const long long q = 2 * p0 - 1;
            auto row = [&](const int i) { return rows3 + ((i & 1) ? (N4 + 1) * R3 : 0) + (i >> 1) * R3; };
            if constexpr (S == 1) {
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const int i = 32 * j + col;
                    store_tile<CS, true>(row(i), mt * 32, half, acc[0][j], slope, q + i >= 0 && q + i < (long long)l3 && i < N3 - 1);
                }
            } else {   // [S][CS][33], then a position and four channels a thread
                float *part3 = (float *)buf;
#pragma unroll
                for (int r = 0; r < 16; ++r) part3[((wave % S) * CS + mt * 32 + (r >> 2) * 8 + half * 4 + (r & 3)) * 33 + col] = acc[0][0][r];
                __syncthreads();
                const int i = tid & 31;
                const Act act(slope, q + i >= 0 && q + i < (long long)l3 && i < N3 - 1);
#pragma unroll
                for (int g = tid >> 5; g < CS / 4; g += W * 2) {
                    const f4v bias = *(const f4v *)(w.b3 + share * CS + 4 * g);
                    float y[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        float sum = bias[c];
#pragma unroll
                        for (int k = 0; k < S; ++k) sum += part3[(k * CS + 4 * g + c) * 33 + i];
                        y[c] = act(sum);
                    }
                    store_split<CS, true>(row(i), 4 * g, y);
                }
            }
        }
        {   // conv4: one position tile (of which N4 columns are used); the steps are shared out over kSplit wavefronts
            constexpr int kPer = CS / 16, kSteps = 3 * kPer / kSplit, kAhead = kSteps < 4 ? kSteps : 4;
            static_assert(3 * kPer % kSplit == 0, "conv4 steps");
            static_assert(kSplit == 4, "runs of steps");
            const int mt = wave / kSplit, ks = wave % kSplit;
            const u4v *a = (const u4v *)w.s4 + (size_t)(mt * 3 * kPer3 + share * kPer) * 192 + lane;
            auto frag = [&](int, const int s) { return a + ((ks * kSteps + s) / kPer * kPer3 + (ks * kSteps + s) % kPer) * 192; };
            Fragments<1, kAhead> f;
            fragments_start(f, frag);
            acc16 acc[1][1];
            acc[0][0] = zero16();
            const unsigned char *b = rows3 + (col < N4 ? col : N4 - 1) * R3 + half * 16;
            // a constant for each wavefront: the addresses of its steps are then parts of the instructions (4 x 10 000 values
            // 16.5 us without, 16.1 with)
            auto run = [&](auto k) {
                constexpr int s0 = decltype(k)::value * kSteps;
                conv_mma<CS, 1, 1, kSteps, kAhead>(acc, f, [&](int, const int s) { return a + ((s0 + s) / kPer * kPer3 + (s0 + s) % kPer) * 192; }, [&](int, const int s) {
                    const int tap = (s0 + s) / kPer;
                    return b + (tap == 1 ? (N4 + 1) * R3 : (tap >> 1) * R3) + 32 * ((s0 + s) % kPer);
                });
            };
            __syncthreads();
            if (ks == 0) run(std::integral_constant<int, 0>());    // wave-uniform
            else if (ks == 1) run(std::integral_constant<int, 1>());
            else if (ks == 2) run(std::integral_constant<int, 2>());
            else run(std::integral_constant<int, 3>());
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 16; ++r)
                part[(ks * C4 + mt * 32 + (r >> 2) * 8 + half * 4 + (r & 3)) * 33 + col] = acc[0][0][r];
        }
    }
    __syncthreads();
    constexpr int kGroups = W * 2, kCh = C4 / kGroups;
    {   // conv4's sums, bias and non-linearity; conv5's sums over this thread's channels
        const int p = tid & 31, cg = tid >> 5;
        float y[kCh];
#pragma unroll
        for (int i = 0; i < kCh; ++i) {
            y[i] = part[(cg * kCh + i) * 33 + p];
#pragma unroll
            for (int s = 1; s < kSplit; ++s) y[i] += part[(s * C4 + cg * kCh + i) * 33 + p];
        }
        if constexpr (S > 1) {
            // Through the device's memory, past the L2s: what a wavefront has stored is there once it has been acknowledged,
            // the barrier collects the wavefronts, and one thread counts the block.
            __shared__ uint32_t before;
            if (p < N4) {
#pragma unroll
                for (int i = 0; i < kCh; ++i) __hip_atomic_store(sums + (share * C4 + cg * kCh + i) * 16 + p, y[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
            __syncthreads();
            if (tid == 0) before = __hip_atomic_fetch_add(taken, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(before) != S - 1) return;
            if (tid == 0) __hip_atomic_store(taken, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // as the next call expects it
            float in[S][kCh];
            if (p < N4) {
#pragma unroll
                for (int k = 0; k < S; ++k)
#pragma unroll
                    for (int i = 0; i < kCh; ++i) in[k][i] = __hip_atomic_load(sums + (k * C4 + cg * kCh + i) * 16 + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int i = 0; i < kCh; ++i) {
                    y[i] = in[0][i];
#pragma unroll
                    for (int k = 1; k < S; ++k) y[i] += in[k][i];
                }
            }
        }
        double t[C5];
#pragma unroll
        for (int c = 0; c < C5; ++c) t[c] = 0.;
#pragma unroll
        for (int i = 0; i < kCh; ++i) {
            const int co = cg * kCh + i;
            const float v = leaky_f(y[i] + small[kB4 + co], slope);
#pragma unroll
            for (int c = 0; c < C5; ++c) t[c] = fma((double)small[kW5 + c * C4 + co], (double)v, t[c]);
        }
#pragma unroll
        for (int c = 0; c < C5; ++c) red[(cg * C5 + c) * 32 + p] = t[c];
    }
    __syncthreads();
    const int c = tid >> 5, p = tid & 31;
    const bool mine = c < C5 && p < P && p0 + p < (long long)l4;
    float z = 0.f;
    if (mine) {
        double sum = small[kB5 + c];
#pragma unroll
        for (int g = 0; g < W * 2; ++g) sum += red[(g * C5 + c) * 32 + p];
        z = (float)sum;
    }
    bool redo = __syncthreads_or(mine && !(fabsf(z) >= w.limits.least && fabsf(z) < INFINITY));
    if (redo && w.limits.no_bias) {   // nothing but zeros gives zeros
        bool any = false;
        for (int i = tid; i < 4 * N2 + 3; i += W * 64) any = any || xs[i] != 0.f;
        redo = __syncthreads_or(any);
    }
    if (!redo) {
        if (mine) out[(size_t)c * l4 + p0 + p] = z;
        return;
    }
    float *f = (float *)buf;
    conv1([&](const int i, const float (&y)[8]) {
        float *row = f + ((i & 1) ? (N2 + 1) * row_floats(C1) : 0) + (i >> 1) * row_floats(C1) + wave * 8;
        const long long q = 8 * p0 - 7 + i;
        const bool valid = q >= 0 && q < (long long)l1;   // (chosen, not multiplied: see Act)
        *(f4v *)row = valid ? (f4v){y[0], y[1], y[2], y[3]} : (f4v){0.f, 0.f, 0.f, 0.f};
        *(f4v *)(row + 4) = valid ? (f4v){y[4], y[5], y[6], y[7]} : (f4v){0.f, 0.f, 0.f, 0.f};
    });
    __syncthreads();
    layer_fp32<C1, C2, N2, W>(f, w.w2, w.b2, wave, 4 * p0 - 3, l2, slope);
    layer_fp32<C2, C3, N3, W>(f, w.w3, w.b3, wave, 2 * p0 - 1, l3, slope);
    layer_fp32<C3, C4, N4, W>(f, w.w4, w.b4, wave, p0, l4, slope);
    if (mine) {
        const float *row = f + ((p & 1) ? (N4 / 2 + 1) * row_floats(C4) : 0) + (p >> 1) * row_floats(C4);
        double sum = w.b5[c];
        for (int ci = 0; ci < C4; ++ci) sum = fma((double)w.w5[c * C4 + ci], (double)row[ci], sum);
        out[(size_t)c * l4 + p0 + p] = (float)sum;
    }
}

}  // namespace

struct EncoderCall {
    const float *x;
    float *out, *sums;
    uint32_t *taken;
    uint32_t l[5];          // lengths: the input, conv1 .. conv4
    uint32_t longs, shorts; // per node: runs of 31 positions, then of 15
    int batch;
    float slope;
};

// S = 0: runs of 31 positions, those of all nodes first, and then of 15: what is left over from whole rounds of the long ones
// takes a round of short ones instead of a long one that few compute units have a part in (6 x 25 600 values, 312 runs of 31:
// 51.3 -> 42.3 us; 8 x 67 000, 1088: 133.8 -> 124.2, both with loads behind the products).
// S > 0: runs of 15 positions, S blocks each, grid (runs, nodes, S).
template <int C1, int C2, int C3, int C4, int C5, int W, int S>
__global__ __launch_bounds__(W * 64) void k_encoder_fused(EncoderCall c, EncoderDev w) {
    using L = EncoderRun<S == 0 ? 31 : 15, S == 0 ? 1 : S, C1, C2, C3, C4, C5, W>;
    using T = EncoderRun<15, S == 0 ? 1 : S, C1, C2, C3, C4, C5, W>;
    __shared__ __align__(16) unsigned char buf[L::kBytes > T::kBytes ? L::kBytes : T::kBytes];
    __shared__ __align__(16) float xs[L::kXs], small[L::kSmall];
    const uint32_t longs = S == 0 ? c.longs * c.batch : 0;
    if (S == 0 && blockIdx.x < longs) {   // block-uniform
        const uint32_t node = blockIdx.x / c.longs, run = blockIdx.x % c.longs;
        encode_run<31, 1, C1, C2, C3, C4, C5, W>(c.x + (size_t)node * c.l[0], c.out + (size_t)node * C5 * c.l[4], w, c.l[0], c.l[1], c.l[2], c.l[3], c.l[4], c.slope,
                                                 31ll * run, 0, nullptr, nullptr, buf, xs, small);
        return;
    }
    const uint32_t node = S == 0 ? (blockIdx.x - longs) / c.shorts : blockIdx.y, run = S == 0 ? (blockIdx.x - longs) % c.shorts : blockIdx.x;
    const uint32_t at = S == 0 ? 0 : node * gridDim.x + run;
    encode_run<15, S == 0 ? 1 : S, C1, C2, C3, C4, C5, W>(c.x + (size_t)node * c.l[0], c.out + (size_t)node * C5 * c.l[4], w, c.l[0], c.l[1], c.l[2], c.l[3], c.l[4],
                                                          c.slope, 31ll * c.longs + 15ll * run, blockIdx.z, c.sums + (size_t)at * S * C4 * 16, c.taken + at, buf, xs, small);
}

// ---- decoder ---------------------------------------------------------------------------------------
// A kernel-3 / stride-1 transposed layer D0 -> D1, four kernel-3 / stride-2 ones D1 -> D2 -> D3 -> D4 -> D5 and a
// kernel-1 layer D5 -> 1.  A stride-2 transposed layer is two products: output 2m from input m (tap 1), output
// 2m + 1 from inputs m (tap 2) and m + 1 (tap 0).

struct DecoderDev {
    const float *w1, *w2, *w3, *w4, *w5, *w6;   // [c_in][c_out][3]; w6 [D5]
    const float *b1, *b2, *b3, *b4, *b5, *b6;
    const uint16_t *s3, *s4, *s5;               // the deep layers as bf16 fragments
    FusedLimits limits;
};

namespace {

template <int C>
__device__ __forceinline__ void load_b(u4v (&r)[3], const unsigned char *b, const int at) {
#pragma unroll
    for (int p = 0; p < 3; ++p) r[p] = *(const u4v *)(b + p * 2 * C + at);
}

// The even and the odd outputs of a transposed layer in plain fp32, CI input channels from row b (the lane's input m; m + 1
// lies R floats on): w = the lane's output channel of [CI][CO][3], both from the half's first channel on
template <int CI, int CO, int R>
__device__ __forceinline__ void up_fp32(acc16 &even, acc16 &odd, const float *__restrict__ w, const float *b) {
#pragma unroll 1
    for (int c = 0; c < CI; c += 8) {
        const f4v x0 = *(const f4v *)(b + c), x1 = *(const f4v *)(b + R + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float *wc = w + (size_t)(c + e) * CO * 3;
            odd = mma_fp32(wc[2], x0[e], odd);
            even = mma_fp32(wc[1], x0[e], even);
            odd = mma_fp32(wc[0], x1[e], odd);
        }
    }
}

// One result tile with the non-linearity as fp32: `row` is the lane's position
__device__ __forceinline__ void store_fp32(float *row, const int co0, const int half, const acc16 &acc, const float slope, const bool valid) {
#pragma unroll
    for (int r = 0; r < 16; ++r) row[co0 + 8 * (r >> 2) + 4 * half + (r & 3)] = valid ? leaky_f(acc[r], slope) : 0.f;
}

}  // namespace

// T latent positions per block of four wavefronts.  Local numbering from 1, 2, 4, 8 and 16 p0 on: T + 1 outputs of deconv1,
// 2T + 1 of deconv2, 4T + 1 of deconv3, 8T + 1 of deconv4 and 16T of deconv5.  A wavefront takes 32 of deconv3's positions through
// deconv4 and deconv5, 32 channels of deconv4 at a time: lane i holds its outputs 2i and 2i + 1, splits them in registers and
// multiplies on, so that no barrier and no exchange through the LDS stands between the two layers that make up the work, and
// one wavefront converts while another one multiplies.  deconv5's output 4i + 3 needs deconv4's 2i + 2, which is the next
// lane's: 31 of the 32 positions come out.  4 / NP wavefronts share a position tile's channels of deconv4 and add their sums up
// at the end.  The bound of two wavefronts per SIMD leaves room for the weights' fragments that are under way (one step ahead).
// Through the LDS, in two runs of 64 channels with four barriers each, 4 x 25 600 values took 21.2 us where this and the loads
// behind the products take 19.0, 8 x 67 000 86.5 / 78.2, 1 x 1 023 12.4 / 8.1 (with 7 positions per block).  What bounds it:
// two blocks on a compute unit have 18.4 K cycles of products in 39 K; the rest is each block's way to the first product (9 K:
// a read from memory, three small layers, three barriers) and its end (5 K).
template <int D0, int D1, int D2, int D3, int D4, int D5, int T, bool RING>
__global__ __launch_bounds__(256, 2) void k_decoder_fused(const float *__restrict__ z, float *__restrict__ out, DecoderDev w,
                                                       uint32_t lz, uint32_t l2, uint32_t l3, uint32_t l4, uint32_t l5,
                                                       float slope) {
    constexpr int NP = (4 * T + 30) / 31, KG = 4 / NP, CT = D4 / 32 / KG;   // position tiles; wavefronts per tile; their tiles of 32 channels
    constexpr int M3 = 2 * (T + 1), M4 = 4 * (T + 1), M5 = 8 * (T + 1);     // outputs of deconv2, 3, 4 that are kept (of which one or three too many)
    constexpr int R2 = row_bytes(D2), R3 = row_bytes(D3);
    constexpr int CH = 64, RH = row_floats(CH);                             // the redo: 64 of deconv4's outputs x CH channels in each half of the ring
    constexpr int kStep = KG * 9 * 1024;                                    // a step's fragments: three parts of three taps per group of channels
    constexpr int kHandOver = 2 * (KG == 4 ? 3 : 2) * 4096;                 // sums that change wavefronts: half of them
    constexpr int kRedo = 65 * RH * 4, kMost = kRedo > kHandOver ? kRedo : kHandOver;
    constexpr int kBytesA = RING && kStep > kMost ? kStep : kMost;
    static_assert(!RING || KG == 2, "two wavefronts read a step");
    static_assert((M5 == 128 || M5 == 64) && D4 == 2 * CH, "two wavefronts per half of the ring");
    static_assert(NP * KG == 4 && CT * KG * 32 == D4 && M3 <= 32 && D2 % 16 == 0 && D3 == 64 && D4 == 128 && D5 == 32, "tiles");
    static_assert(row_floats(D2) * 4 <= R2 && row_floats(D3) * 4 <= R3 && M4 <= 64 && 31 * NP + 2 <= 65, "rows");
    // steps of weights on their way to the wavefronts; sums handed over; in the redo: deconv4's outputs
    __shared__ __align__(16) unsigned char ring0[kBytesA], ring1[kBytesA];
    __shared__ __align__(16) unsigned char bufA[33 * R2], bufB[65 * R3];   // deconv2's outputs, deconv3's
    __shared__ float zs[D0 * (T + 3)], h1[D1 * (T + 1)];
    // the small layers' weights and all biases
    constexpr int kW2 = 0, kB3 = kW2 + D1 * D2 * 3, kB5 = kB3 + D3, kW6 = kB5 + D5, kB4 = kW6 + D5, kW1 = kB4 + D4, kB1 = kW1 + 3 * D0 * D1, kB2 = 736;
    __shared__ __align__(16) float small[768];
    static_assert(kB3 == 384 && kB4 == 512 && kW1 == 640 && kB1 == 688 && kB1 + D1 <= kB2 && kB2 + D2 <= 768, "three words per thread");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    const long long p0 = (long long)blockIdx.x * T;
    z += (size_t)blockIdx.y * D0 * lz;
    out += (size_t)blockIdx.y * l5;

    // everything that the first three layers read from memory, at once: one wait instead of four in a row
    constexpr int kCh = D2 / 8, kPer3 = D2 / 16;
    static_assert(D0 == 4 && D1 == 4 && kCh == 4 && D0 * (T + 3) <= 256 && D1 * (T + 1) <= 256, "one value per thread");
    const int zc = tid / (T + 3);
    const long long ze = p0 - 1 + tid % (T + 3);
    const float zv = zc < D0 && ze >= 0 && ze < (long long)lz ? z[(size_t)zc * lz + ze] : 0.f;
    float sv[3];
    sv[0] = w.w2[tid];
    sv[1] = *(tid < 128 ? w.w2 + 256 + tid : tid < 192 ? w.b3 + tid - 128 : tid < 224 ? w.b5 + tid - 192 : w.w6 + tid - 224);
    sv[2] = *(tid < 128 ? w.b4 + tid : tid < 176 ? w.w1 + tid - 128 : tid < 180 ? w.b1 + tid - 176 : w.b2 + (tid < 224 ? 0 : tid - 224));
    const int mt3 = wave & 1, par3 = wave >> 1;   // deconv3: wavefront = channel tile x (even or odd outputs)
    u4v a3[2 * kPer3][1][3];
    {
        const u4v *a = (const u4v *)w.s3 + (size_t)mt3 * 3 * kPer3 * 192 + lane;
#pragma unroll
        for (int s = 0; s < kPer3; ++s) {
            load_a(a3[s][0], a, (par3 ? 2 : 1) * kPer3 + s);
            load_a(a3[kPer3 + s][0], a, s);   // of the odd outputs only
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // deconv4 and deconv5: this wavefront's position tile and channels, the latter's weights step by step (four steps of deconv4, two of
    // deconv5 for each 32 channels)
    const int pt = wave % NP, kg = wave / NP;
    constexpr int kPer = D3 / 16, kPer5 = D4 / 16, kSteps = kPer + 2;
    const u4v *a4 = (const u4v *)w.s4 + (size_t)(kg * CT) * 3 * kPer * 192, *a5 = (const u4v *)w.s5 + kg * CT * 2 * 192;
    const uint32_t lane16 = 16u * (uint32_t)lane;
    auto fragments = [&](const int ct, const int s, const int t) {   // of tap 2 - t
        return s < kPer ? a4 + (ct * 3 * kPer + (2 - t) * kPer + s) * 192 : a5 + (ct * 2 + (2 - t) * kPer5 + s - kPer) * 192;
    };
    auto scalar = [](const u4v *p) {   // left alone the compiler keeps a pair of vector registers for each of these addresses
        uint64_t at = (uint64_t)p;
        asm("" : "+s"(at));
        return at;
    };
    // RING: the two wavefronts of a group of channels fetch a step's fragments for both, into the LDS without registers on the way
    auto fetch = [&](unsigned char *ring, const int ct, const int s) {
#pragma unroll
        for (int i = 0; i < 5; ++i) {   // nine between two: both fetch the middle one, so that each knows how many it waits for
            const int f = pt * 4 + i;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(scalar(fragments(ct, s, f / 3) + (f % 3) * 64) + lane16),
                                             (__attribute__((address_space(3))) void *)(ring + (kg * 9 + f) * 1024), 16, 0, 0);
        }
    };
    if (zc < D0) zs[tid] = zv;
#pragma unroll
    for (int i = 0; i < 3; ++i) small[256 * i + tid] = sv[i];
    __builtin_amdgcn_sched_barrier(0);
    if (RING) { fetch(ring0, 0, 0); fetch(ring1, 0, 1); }   // (ahead of those stores the compiler waits for it before them)
    __syncthreads();
    if (tid < D1 * (T + 1)) {   // deconv1: thread = channel x position
        const int c = tid / (T + 1), j = tid % (T + 1);
        float a = small[kB1 + c];
#pragma unroll
        for (int ci = 0; ci < D0; ++ci) {
            const float *zi = zs + ci * (T + 3) + j, *wc = small + kW1 + (ci * D1 + c) * 3;
            a = fmaf(wc[0], zi[2], a);
            a = fmaf(wc[1], zi[1], a);
            a = fmaf(wc[2], zi[0], a);
        }
        h1[tid] = p0 + j < (long long)lz ? leaky_f(a, slope) : 0.f;
    }
    __syncthreads();
    auto deconv2 = [&](float (&y)[kCh], const int thread) {   // thread = position x group of D2 / 8 channels
        const int j = thread & 31, m = j >> 1;
        const bool odd = j & 1, valid = 2 * p0 + j < (long long)l2 && j < 2 * T + 1;
#pragma unroll
        for (int c = 0; c < kCh; ++c) y[c] = small[kB2 + (thread >> 5) * kCh + c];
#pragma unroll
        for (int ci = 0; ci < D1; ++ci) {
            const float x0 = m <= T ? h1[ci * (T + 1) + m] : 0.f, x1 = m < T ? h1[ci * (T + 1) + m + 1] : 0.f;
#pragma unroll
            for (int c = 0; c < kCh; ++c) {
                const float *wc = small + kW2 + (ci * D2 + (thread >> 5) * kCh + c) * 3;
                const float e = fmaf(wc[1], x0, y[c]), o = fmaf(wc[2], x0, fmaf(wc[0], x1, y[c]));
                y[c] = odd ? o : e;
            }
        }
#pragma unroll
        for (int c = 0; c < kCh; ++c) y[c] = valid ? leaky_f(y[c], slope) : 0.f;
    };
    {
        float y[kCh];
        deconv2(y, tid);
        unsigned char *row = bufA + (tid & 31) * R2 + (tid >> 5) * kCh * 2;
#pragma unroll
        for (int c = 0; c < kCh; c += 2) {
            uint32_t h, m_, l;
            split2(y[c], y[c + 1], h, m_, l);
            *(uint32_t *)(row + 2 * c) = h;
            *(uint32_t *)(row + 2 * D2 + 2 * c) = m_;
            *(uint32_t *)(row + 4 * D2 + 2 * c) = l;
        }
    }
    __syncthreads();
    {   // deconv3
        const unsigned char *b = bufA + col * R2 + half * 16;
        acc16 acc[1][1], cross[1][1];
        acc[0][0] = bias16(small + kB3, mt3 * 32, half);
        cross[0][0] = zero16();
        u4v rb[1][3];
#pragma unroll
        for (int s = 0; s < kPer3; ++s) {
            load_b<D2>(rb[0], b, 32 * s);
            mma6<1, 1>(acc, cross, a3[s], rb);
            if (par3) {
                load_b<D2>(rb[0], b + R2, 32 * s);
                mma6<1, 1>(acc, cross, a3[kPer3 + s], rb);
            }
        }
        acc[0][0] += cross[0][0];
        const int i = 2 * col + par3;
        store_tile<D3>(bufB + i * R3, mt3 * 32, half, acc[0][0], slope, 4 * p0 + i < (long long)l3 && i < 4 * T + 1);
    }

    const int i0 = 31 * pt + col;   // this lane's position of deconv3
    acc16 y[4];   // deconv5's outputs 4 i0 .. 4 i0 + 3
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = zero16();
    {
        const unsigned char *b = bufB + i0 * R3 + half * 16;
        u4v ra[2][3][3], x0[3], x1[3];   // taps 2, 1, 0; inputs i0 and i0 + 1
        auto take = [&](const int ct, const int s) {   // step s into registers
#pragma unroll
            for (int t = 0; t < 3; ++t)
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    if (RING) ra[s & 1][t][p] = *(const u4v *)(((s & 1) ? ring1 : ring0) + (kg * 9 + t * 3 + p) * 1024 + lane16);
                    else ra[s & 1][t][p] = *(const __attribute__((address_space(1))) u4v *)(scalar(fragments(ct, s, t) + p * 64) + lane16);
        };
        // Before step s: the next one into registers, and the one after it under way.  What is in the ring is there for all
        // once each wavefront has waited for its own share; what was in its other half has been read.  The fences keep the LDS
        // reads of either step on their side of the barrier.
        auto advance = [&](const int ct, const int s) {
            if (RING) {
                if (s + 1 < kSteps || ct + 1 < CT) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0)
                    __builtin_amdgcn_s_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (s + 2 < kSteps) fetch((s & 1) ? ring1 : ring0, ct, s + 2);
                else if (ct + 1 < CT) fetch((s & 1) ? ring1 : ring0, ct + 1, s + 2 - kSteps);
            }
            if (s + 1 < kSteps) take(ct, s + 1);
            else if (ct + 1 < CT) take(ct + 1, 0);
        };
        if (!RING) take(0, 0);
        if (RING) __builtin_amdgcn_s_waitcnt(0x0070);
        __syncthreads();   // deconv3's outputs are there, and the first two steps
        if (RING) take(0, 0);
#pragma unroll 1
        for (int ct = 0; ct < CT; ++ct) {
            acc16 up[2], cross[2];   // the odd and the even outputs
            up[0] = bias16(small + kB4 + (kg * CT + ct) * 32, 0, half);
            up[1] = up[0];
            cross[0] = zero16(); cross[1] = zero16();
            load_b<D3>(x0, b, 0);
#pragma unroll
            for (int s = 0; s < kPer; ++s) {
                load_b<D3>(x1, b + R3, 32 * s);
                __builtin_amdgcn_sched_barrier(0);
                advance(ct, s);
                mma6_by<2>(up, cross, (const u4v (&)[2][3])ra[s & 1], x0);
                interleave<12, RING ? 9 : 0, RING ? 5 : 9>();
                __builtin_amdgcn_sched_barrier(0);
                if (s + 1 < kPer) load_b<D3>(x0, b, 32 * (s + 1));
                mma6_by<1>(up, cross, (const u4v (&)[1][3])ra[s & 1][2], x1);
                interleave<6, 3, 0>();
                __builtin_amdgcn_sched_barrier(0);
            }
            up[0] += cross[0]; up[1] += cross[1];
            u4v e[2][3], o[2][3], n[2][3];
            as_operands(up[1], slope, 8 * p0 + 2 * i0 < (long long)l4 && 2 * i0 < 8 * T + 1, e);
            as_operands(up[0], slope, 8 * p0 + 2 * i0 + 1 < (long long)l4 && 2 * i0 + 1 < 8 * T + 1, o);
            next_position(e, n);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                advance(ct, kPer + q);
                mma6_up4(y, ra[q & 1], e[q], o[q], n[q]);
                interleave<36, RING ? 9 : 0, RING ? 5 : 9>();
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    if (RING) __syncthreads();   // the last step has been read
    // The numbers of this thread anew, from its lane: kept over the loop they would be the registers too many.  (Unknown to the compiler as
    // well, so that the values loaded above are not kept for the redo.)
    uint32_t every = ~0u;
    asm volatile("" : "+s"(every));
    const int ln = (int)__builtin_amdgcn_mbcnt_hi(every, __builtin_amdgcn_mbcnt_lo(every, 0u)), id = wave * 64 + ln, hf = ln >> 5, cl = ln & 31, at = 31 * pt + cl;
    // the sums of a tile's wavefronts meet: wavefront kg finishes outputs kOwn kg .. of every four and hands the others over
    constexpr int kOwn = 4 / KG;   // 2 or 1
    // [tile][output][from: the other wavefronts in order][16][64], the first two outputs of a tile in one half of the ring
    auto swap = [&](const int j) { return (float *)(j < 2 ? ring0 : ring1) + (pt * 2 + (j & 1)) * (KG - 1) * 1024 + ln; };
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (j / kOwn != kg) {      // wave-uniform
            const int from = kg < j / kOwn ? kg : kg - 1;
            float *to = swap(j) + from * 1024;
#pragma unroll
            for (int r = 0; r < 16; ++r) to[r * 64] = y[j][r];
        }
    }
    __syncthreads();
    double sum[kOwn];
    acc16 own[kOwn];
#pragma unroll
    for (int k = 0; k < KG; ++k)
        if (kg == k) {             // wave-uniform
#pragma unroll
            for (int j = 0; j < kOwn; ++j) own[j] = y[k * kOwn + j];
        }
#pragma unroll
    for (int j = 0; j < kOwn; ++j) {
        const float *from = swap(kg * kOwn + j);
        sum[j] = 0.;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f4v bv = *(const f4v *)(small + kB5 + 8 * g + 4 * hf), wv = *(const f4v *)(small + kW6 + 8 * g + 4 * hf);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int r = 4 * g + c;
                float x = own[j][r];
#pragma unroll
                for (int k = 0; k < KG - 1; ++k) x += from[k * 1024 + r * 64];
                sum[j] = fma((double)wv[c], (double)leaky_f(x + bv[c], slope), sum[j]);
            }
        }
        sum[j] += __shfl_xor(sum[j], 32, 64);
    }
    // the halves of a wavefront have the same sums: two outputs are stored by a half each, one by the first half
    const int o = kg * kOwn + (kOwn == 2 ? hf : 0), i = 4 * at + o;
    const bool mine = cl < 31 && (kOwn == 2 || hf == 0) && i < 16 * T && 16 * p0 + i < (long long)l5;
    const float result = (float)(w.b6[0] + (kOwn == 2 && hf ? sum[kOwn - 1] : sum[0]));
    bool redo = __syncthreads_or(mine && !(fabsf(result) >= w.limits.least && fabsf(result) < INFINITY));
    if (redo && w.limits.no_bias) {   // nothing but zeros gives zeros
        redo = __syncthreads_or(id < D0 * (T + 3) && zs[id] != 0.f);
    }
    if (!redo) {
        if (mine) out[16 * p0 + i] = result;
        return;
    }
    float *fd = (float *)bufA, *fb = (float *)bufB;
    {
        float y2[kCh];
        deconv2(y2, id);
#pragma unroll
        for (int c = 0; c < kCh; ++c) fd[(id & 31) * row_floats(D2) + (id >> 5) * kCh + c] = y2[c];
    }
    __syncthreads();
    if (wave < D3 / 32) {   // deconv3: wavefront = channel tile
        acc16 even = bias16(w.b3, wave * 32, hf), odd = even;
        up_fp32<D2, D3, row_floats(D2)>(even, odd, w.w3 + (4 * hf * D3 + wave * 32 + cl) * 3, fd + cl * row_floats(D2) + 4 * hf);
        const int j = 2 * cl;
        store_fp32(fb + j * row_floats(D3), wave * 32, hf, even, slope, 4 * p0 + j < (long long)l3 && j < 4 * T + 1);
        store_fp32(fb + (j + 1) * row_floats(D3), wave * 32, hf, odd, slope, 4 * p0 + j + 1 < (long long)l3 && j + 1 < 4 * T + 1);
    }
    // deconv4, every wavefront a tile of 32 channels x 32 of deconv3's positions: two of each, run by run, for 128 outputs, and
    // the halves of the ring hold 64 outputs each, the first one also the next after them; all four channel tiles at once for
    // 64, and they hold 64 channels each.  (Every block redoing: 22.8 us for 1 x 1 023 values, 213 for 8 x 67 000; runs of 32
    // channels in one half, which half of the wavefronts or a quarter of them made, took 35.5 and 268.)
    __syncthreads();
    constexpr bool kRuns = M5 == 128;
    float *const mine4 = (float *)(wave >= 2 ? ring1 : ring0);
    acc16 e = bias16(w.b5, 0, hf), od = e;   // deconv5: wavefront = position tile
#pragma unroll 1
    for (int run = 0; run < (kRuns ? 2 : 1); ++run) {
        const int co0 = (kRuns ? run * CH : (wave >> 1) * CH) + (wave & 1) * 32, m0 = (kRuns ? (wave >> 1) * 32 : 0) + cl, j = 2 * m0;
        acc16 even = bias16(w.b4, co0, hf), odd = even;
        up_fp32<D3, D4, row_floats(D3)>(even, odd, w.w4 + (4 * hf * D4 + co0 + cl) * 3, fb + m0 * row_floats(D3) + 4 * hf);
        __syncthreads();   // the run before has been read
        const bool valid = 8 * p0 + j < (long long)l4 && j < 8 * T + 1;
        store_fp32(mine4 + 2 * cl * RH, (wave & 1) * 32, hf, even, slope, valid);
        store_fp32(mine4 + (2 * cl + 1) * RH, (wave & 1) * 32, hf, odd, slope, 8 * p0 + j + 1 < (long long)l4 && j + 1 < 8 * T + 1);
        if (kRuns && wave >= 2 && cl == 0) store_fp32((float *)ring0 + 64 * RH, (wave & 1) * 32, hf, even, slope, valid);
        __syncthreads();
        auto multiply = [&](const float *x, const int ci0) { up_fp32<CH, D5, RH>(e, od, w.w5 + ((ci0 + 4 * hf) * D5 + cl) * 3, x + ((wave & 1) * 32 + cl) * RH + 4 * hf); };
        if (kRuns) multiply(mine4, run * CH);
        else if (wave < 2) { multiply((const float *)ring0, 0); multiply((const float *)ring1, CH); }
    }
    double se = 0., so = 0.;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float wv = w.w6[(r >> 2) * 8 + hf * 4 + (r & 3)];
        se = fma((double)wv, (double)leaky_f(e[r], slope), se);
        so = fma((double)wv, (double)leaky_f(od[r], slope), so);
    }
    se += __shfl_xor(se, 32, 64);
    so += __shfl_xor(so, 32, 64);
    const int m1 = wave * 32 + cl, i1 = 2 * m1 + hf;
    if (m1 < 8 * T && 16 * p0 + i1 < (long long)l5) out[16 * p0 + i1] = (float)(w.b6[0] + (hf ? so : se));
}

// ---- launchers ---------------------------------------------------------------------------------------

static bool is_layer(const LayerDev &l, int ci, int co, int ks, int st) {
    return l.c_in == ci && l.c_out == co && l.ksize == ks && l.stride == st;
}

bool encoder_fused_covers(const LayerDev *l, int count) {
    return count == 5 && is_layer(l[0], 1, 64, 3, 2) && is_layer(l[1], 64, 128, 3, 2) && is_layer(l[2], 128, 256, 3, 2) &&
           is_layer(l[3], 256, 64, 3, 2) && is_layer(l[4], 64, 4, 1, 1);
}

bool decoder_fused_covers(const LayerDev *l, int count) {
    return count == 6 && is_layer(l[0], 4, 4, 3, 1) && is_layer(l[1], 4, 32, 3, 2) && is_layer(l[2], 32, 64, 3, 2) &&
           is_layer(l[3], 64, 128, 3, 2) && is_layer(l[4], 128, 32, 3, 2) && is_layer(l[5], 32, 1, 1, 1);
}

// Runs of 15 positions, each of which 16 values make, are shared while there are no more blocks than compute units: two or four of them a
// run, with 64 channels x 16 positions each
EncoderScratch encoder_scratch(uint64_t max_k, int max_batch, int cus) {
    const uint64_t runs = (max_k + 239) / 240 * max_batch;
    EncoderScratch s;
    s.sum_floats = (size_t)std::min<uint64_t>(4 * runs, cus) * 64 * 16;
    s.taken_words = (uint32_t)std::min<uint64_t>(runs, cus / 2);
    return s;
}

bool launch_encoder_fused(const float *x, float *out, const LayerDev *l, int count, const uint64_t *len, int batch, float slope,
                          const FusedLimits &limits, int cus, const EncoderScratch &scratch, hipStream_t st) {
    if (!encoder_fused_covers(l, count) || !l[1].ws || !l[2].ws || !l[3].ws) return false;
    EncoderCall c;
    c.x = x; c.out = out; c.sums = scratch.sums; c.taken = scratch.taken;
    for (int i = 0; i < 5; ++i) c.l[i] = (uint32_t)len[i];
    c.batch = batch; c.slope = slope; c.longs = c.shorts = 0;
    const uint32_t l4 = c.l[4];
    if (l4 == 0) return true;
    EncoderDev w;
    w.w1 = l[0].w; w.b1 = l[0].b;
    w.w2 = l[1].w; w.b2 = l[1].b; w.s2 = l[1].ws;
    w.w3 = l[2].w; w.b3 = l[2].b; w.s3 = l[2].ws;
    w.w4 = l[3].w; w.b4 = l[3].b; w.s4 = l[3].ws;
    w.w5 = l[4].w; w.b5 = l[4].b;
    w.limits = limits;
    const uint32_t runs = (l4 + 14) / 15;
    const uint64_t all = (uint64_t)runs * batch;
    auto fits = [&](uint64_t shares) { return all * shares <= (uint64_t)cus && (shares == 1 || (all <= scratch.taken_words && all * shares * 64 * 16 <= scratch.sum_floats)); };
#define LGC_ENC(S) hipLaunchKernelGGL((k_encoder_fused<64, 128, 256, 64, 4, 8, S>), dim3(runs, batch, S), dim3(512), 0, st, c, w)
    // as many blocks as there are compute units for the runs of 15
    if (fits(4)) { LGC_ENC(4); return true; }
    if (fits(2)) { LGC_ENC(2); return true; }
    if (fits(1)) { LGC_ENC(1); return true; }
#undef LGC_ENC
    // 31 positions per block stream the 1 MB of weights half as often as 15 do, and waste no half tile in conv4
    // (4 nodes x 25 600 values: 25.8 against 32.7 us)
    const uint32_t longs = (l4 + 30) / 31, rounds = (uint32_t)((uint64_t)longs * batch / cus);   // rounds in which every compute unit has a run of 31
    c.longs = longs; c.shorts = 0;
    if (rounds > 0) {
        const uint32_t most = (uint32_t)((uint64_t)rounds * cus / batch);
        if (most < longs) {
            const uint32_t rest = (l4 - 31 * most + 14) / 15;
            if ((uint64_t)rest * batch <= (uint64_t)cus) { c.longs = most; c.shorts = rest; }
        }
    }
    hipLaunchKernelGGL((k_encoder_fused<64, 128, 256, 64, 4, 8, 0>), dim3((c.longs + c.shorts) * batch), dim3(512), 0, st, c, w);
    return true;
}

bool launch_decoder_fused(const float *z, float *out, const LayerDev *l, int count, uint64_t l_z, const uint64_t *len, int batch,
                          float slope, const FusedLimits &limits, int cus, hipStream_t st) {
    if (!decoder_fused_covers(l, count) || !l[2].ws || !l[3].ws || !l[4].ws) return false;
    if (len[4] == 0) return true;
    DecoderDev w;
    w.w1 = l[0].w; w.b1 = l[0].b;
    w.w2 = l[1].w; w.b2 = l[1].b;
    w.w3 = l[2].w; w.b3 = l[2].b; w.s3 = l[2].ws;
    w.w4 = l[3].w; w.b4 = l[3].b; w.s4 = l[3].ws;
    w.w5 = l[4].w; w.b5 = l[4].b; w.s5 = l[4].ws;
    w.w6 = l[5].w; w.b6 = l[5].b;
    w.limits = limits;
#define LGC_DEC(T, RING) hipLaunchKernelGGL((k_decoder_fused<4, 4, 32, 64, 128, 32, T, RING>), dim3(((uint32_t)l_z + T - 1) / T, batch), dim3(256), 0, st, z, out, w, \
                                            (uint32_t)l_z, (uint32_t)len[1], (uint32_t)len[2], (uint32_t)len[3], (uint32_t)len[4], slope)
    // 7 positions per block while that gives every compute unit at most one: the shorter chain counts (1 x 1 023 values: 8.3 us
    // against 11.6 with 15, 4 x 5 000: 8.9 against 11.6); from two such blocks per compute unit on 15 are better (2 x 15 000:
    // 14.3 against 12.4).  Where those come to two per compute unit as well, their wavefronts fetch the weights once for two,
    // through the LDS (4 x 25 600: 21.9 against 20.4 us, 8 x 67 000: 85.1 against 82.6); a block that has its compute unit to
    // itself loses more by the barriers than it gains (4 x 15 000: 12.5 against 13.4; both before their loads went behind the
    // products).
    if ((uint64_t)((l_z + 6) / 7) * batch <= (uint64_t)cus) LGC_DEC(7, false);
    else if ((uint64_t)((l_z + 14) / 15) * batch <= (uint64_t)cus) LGC_DEC(15, false);
    else LGC_DEC(15, true);
#undef LGC_DEC
    return true;
}

}  // namespace lgc
