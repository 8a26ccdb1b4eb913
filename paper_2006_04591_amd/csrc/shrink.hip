// gfx950 kernels of the learned shrinkage network (inference and training).
//
// Three 3x3 circular cross-correlations (K -> 32 -> 32 -> K channels) map the
// noise-normalised coefficients z_k = c_k / (sigma RMS_k) of a noisy image to
// per-coefficient thresholds tau = softplus(o); coefficients with |z| < tau are
// set to zero (the low-pass plane is kept). Every layer is an implicit GEMM on
// the matrix cores: pixels x (9 taps x input channels) times (9 taps x input
// channels) x output channels, bfloat16 operands, FP32 accumulation
// (v_mfma_f32_16x16x32_bf16).
//
// Lane layout of v_mfma_f32_16x16x32_bf16 (checked on the device): lane l
// holds A row l%16 and B column l%16 with k = 8(l/16) .. 8(l/16)+7, and D
// column l%16 with rows 4(l/16) .. 4(l/16)+3.
//
// A block of k_conv3x3 computes a tile of TH x TW = 8 x 32 output pixels of one
// image for all output channels; the persistent kernels walk tiles of 8 x 64 or
// 4 x 128. An input tile with a one-pixel halo (wrapped around the plane) is
// staged in LDS channel-last, one padded run of channels per pixel, so that a
// lane's 8 consecutive k of one tap are one 16-byte read.
// Hidden activations are stored channel-last in bfloat16: [b][y][x][32].
#include "shrink.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

namespace shear {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int TH = 8, TW = 32;                     // output tile (rows x cols)
constexpr int HH = TH + 2, HW = TW + 2;            // with halo
constexpr int THREADS = 256;                       // 4 wavefronts, 2 tile rows each

// round to nearest bfloat16, ties to even (finite inputs)
__device__ __forceinline__ unsigned short f2bf(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

// softplus(x) = max(x, 0) + log1p(u), u = e^{-|x|} in (0, 1], from the hardware exponential and
// logarithm (relative error ~1e-6, far inside the threshold tolerance). log1p(u) is taken as
// log(w) u / (w - 1) with w = 1 + u rounded, which cancels the rounding of w (Goldberg, 1991,
// "What every computer scientist should know about floating-point arithmetic", Theorem 4);
// when w rounds to 1, log1p(u) = u to working precision.
__device__ __forceinline__ float softplusf(float x) {
    const float u = __expf(-fabsf(x));
    const float w = 1.0f + u;
    const float l = (w == 1.0f) ? u : __logf(w) * (u * __builtin_amdgcn_rcpf(w - 1.0f));
    return fmaxf(x, 0.0f) + l;
}

// bf16 per staged pixel: an odd multiple of 32 bytes, which puts the 16-byte pieces that a fragment read takes
// together (4 consecutive pixels of one piece beside 4 others of the next piece) on distinct banks. With 16
// bytes of padding instead of 32, an LDS instruction lost 4 cycles to conflicts: the hidden layer 115 -> 108 us,
// the backward data 254 -> 249 and 148 -> 144, the first layer 397 -> 395 (16 x 512^2 x 49).
template <int CINP>
struct Pix {
    static constexpr int value = CINP + 16;
};

// LDS of a conv block: the staged input tile; the padded gradient planes of the last layer's training
// epilogue reuse it once the products are done. The shrink epilogue (MODE 5) works from registers.
template <int CINP, int OUTC, int MODE>
constexpr size_t conv_lds_bytes() {
    constexpr size_t in = (size_t)HH * HW * Pix<CINP>::value * 2, out = (size_t)TH * TW * OUTC * 2;
    return (MODE == 2 || MODE == 5 || in >= out) ? in : out;
}

// 2^(x c) for c given as the float chi and the rest clo, to about an ulp: the rounding error of x chi and the
// product x clo enter as a factor 1 + ln 2 times their sum (a rounded product alone would cost |x c| / 2 ulp
// of the result, the rounding of c as much again). RANGE: any x; beyond 2^126 it stays there, so that
// 1 + 2^(x c) has a normal reciprocal, and NaN stays NaN. Else -126 <= x <= 0.
template <bool RANGE>
__device__ __forceinline__ float exp2_product(float x, float chi, float clo) {
    constexpr float LN2 = 0.693147180559945309f;
    const float t = x * chi;
    const float e = __builtin_amdgcn_exp2f(RANGE && t > 126.0f ? 126.0f : t);
    const float lo = !RANGE || fabsf(t) < 126.0f ? fmaf(x, clo, fmaf(x, chi, -t)) : 0.0f;
    return fmaf(e, lo * LN2, e);
}
// 1 / w, 1 <= w <= 2^126 + 1: the hardware's reciprocal and one Newton step
__device__ __forceinline__ float rcp_newton(float w) {
    const float r = __builtin_amdgcn_rcpf(w);
    return fmaf(fmaf(-w, r, 1.0f), r, r);
}

// The training loss of one coefficient, with o the network's output and z, zc the noisy and clean
// coefficients in noise units: tau = softplus(o), g = sigmoid((|z| - tau) / T), r = z g - zc; adds r^2 to
// lsum and gives v = d(loss_scale r^2) / d o = -2 loss_scale / T r z g (1 - g) sigmoid(o). With
// u = e^-|o| and w = 1 + u, softplus(o) = max(o, 0) + log1p(u) and sigmoid(o) is 1 / w or u / w, so the three
// functions of o share one exponential and one reciprocal; the division by T is part of the gate's
// exponent. log1p(u) is log w plus what the rounding of w left out, (u - (w - 1)) / w: tau keeps its relative
// precision for small thresholds (log w alone loses it: below o = -17 it is 0, and a small temperature
// magnifies the loss before that). The exponentials are within about an ulp and the reciprocals within one:
// against 64 bits, tau, g and the gradient are no further off than with the library's expf and IEEE
// divisions, at 42 VALU instructions instead of 105, which bound the epilogue (205 M values at 16 x 512^2 x
// 49). The bare hardware functions (20 instructions; a training step 1.96 ms instead of 1.98) put r and the
// gradient about a fifth to a third further off.
struct GateLoss {
    float ehi, elo;  // log2(e) / T
    float c;         // -2 loss_scale / T
};
__device__ __forceinline__ void gate_loss(float o, float z, float zc, const GateLoss& gl, float& lsum, float& v) {
    constexpr float L2E = 1.44269504088896341f, L2E_LO = (float)(1.44269504088896340736 - (double)L2E);
    constexpr float LN2 = 0.693147180559945309f;
    const float u = exp2_product<false>(fmaxf(-fabsf(o), -126.0f), L2E, L2E_LO);  // (o = NaN reaches tau)
    const float w = 1.0f + u, rw = rcp_newton(w);
    const float tau = (o < 0.0f ? 0.0f : o) + fmaf(__builtin_amdgcn_logf(w), LN2, (u - (w - 1.0f)) * rw);
    const float so = (o < 0.0f ? u : 1.0f) * rw;
    const float g = rcp_newton(1.0f + exp2_product<true>(tau - fabsf(z), gl.ehi, gl.elo));
    const float r = fmaf(z, g, -zc);
    lsum = fmaf(r, r, lsum);
    v = gl.c * r * (z * g) * (1.0f - g) * so;
}

// Stages the halo tile of one image from bfloat16 channel-last activations with C channels per pixel.
template <int C>
__device__ __forceinline__ void stage(const ConvArgs& a, unsigned short* s, int b, int y0, int x0) {
    constexpr int PIX = Pix<C>::value;
    const int N = a.N, M = a.M;
    const uint4* in = reinterpret_cast<const uint4*>(a.in);
    constexpr int CH = C / 8;  // 16-byte chunks per pixel
    constexpr int TOTAL = HH * HW * CH, NIT = (TOTAL + THREADS - 1) / THREADS;
    // all of a thread's loads are issued before its first LDS store, so that they are in flight
    // together (one load, wait and store at a time left each wavefront waiting on memory latency)
    uint4 v[NIT];
#pragma unroll
    for (int j = 0; j < NIT; ++j) {
        const int i = (int)threadIdx.x + j * THREADS;
        v[j] = make_uint4(0u, 0u, 0u, 0u);
        if (i < TOTAL) {
            const int ch = i % CH, p = i / CH, xx = p % HW, yy = p / HW;
            const int y = (y0 + yy - 1 + N) & (N - 1), x = (x0 + xx - 1 + M) & (M - 1);
            v[j] = in[(((size_t)b * N + y) * M + x) * CH + ch];
        }
    }
#pragma unroll
    for (int j = 0; j < NIT; ++j) {
        const int i = (int)threadIdx.x + j * THREADS;
        if (i < TOTAL) {
            const int ch = i % CH, p = i / CH, xx = p % HW, yy = p / HW;
            *reinterpret_cast<uint4*>(s + (yy * HW + xx) * PIX + ch * 8) = v[j];
        }
    }
}

// Four bfloat16 of 4 floats, rounded to nearest even (v_cvt_pk_bf16_f32), as one 8-byte word.
__device__ __forceinline__ uint2 pack_bf16x4(float a, float b, float c, float d) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const bf16x2 lo = __builtin_convertvector((f32x2){a, b}, bf16x2);
    const bf16x2 hi = __builtin_convertvector((f32x2){c, d}, bf16x2);
    return make_uint2(__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi));
}

template <int NT>
__device__ __forceinline__ void zero_acc(f32x4 (&acc)[4][NT]) {
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
}

// out[pixel][co] accumulators of a wavefront: 4 m-tiles (16 pixels of one row) x NT n-tiles, added
// to acc: output channels co0 .. co0 + COUTP - 1 of the packed weights, CINP input channels staged in s.
template <int CINP, int COUTP, int PD = 2>
__device__ __forceinline__ void mma(const ConvArgs& a, const unsigned short* s, f32x4 (&acc)[4][COUTP / 16], int co0) {
    constexpr int PIX = Pix<CINP>::value, NT = COUTP / 16;
    const int w = threadIdx.x / 64, l = threadIdx.x % 64;
    const int lr = l % 16, lk = 8 * (l / 16);
    const unsigned short* W = a.W;
    // steps (tap, 32-channel chunk kc) in order
    constexpr int KCN = CINP / 32, STEPS = 9 * KCN;
    auto wfrag = [&](int it, int nt) {
        const int tap = it / KCN, kc = it % KCN;
        return *reinterpret_cast<const bf16x8*>(W + ((size_t)(co0 + nt * 16 + lr) * 9 + tap) * CINP + kc * 32 + lk);
    };
    auto step = [&](int it, const bf16x8(&bf)[NT]) {
        const int tap = it / KCN, kc = it % KCN, dy = tap / 3, dx = tap % 3;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const int row = 2 * w + mt / 2, xs = (mt % 2) * 16;
            const bf16x8 afr =
                *reinterpret_cast<const bf16x8*>(s + ((row + dy) * HW + xs + lr + dx) * PIX + kc * 32 + lk);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afr, bf[nt], acc[mt][nt], 0, 0, 0);
        }
    };
    if constexpr (PD > 0) {
        // fully unrolled; the weight fragments are loaded PD steps ahead of their products, so that
        // their latency (an L2 hit, several times one step's products) overlaps PD steps of products
        // ((PD + 1) x NT x 4 VGPRs). A scheduling barrier after each step's loads keeps them there:
        // with a distance of one step and no barrier, the scheduler moved each load down to its use
        // and every step waited for L2.
        bf16x8 bq[STEPS][NT];
#pragma unroll
        for (int it = 0; it < PD && it < STEPS; ++it)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) bq[it][nt] = wfrag(it, nt);
#pragma unroll
        for (int it = 0; it < STEPS; ++it) {
            if (it + PD < STEPS) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) bq[it + PD][nt] = wfrag(it + PD, nt);
            }
            __builtin_amdgcn_sched_barrier(0);
            step(it, bq[it]);
        }
    } else {
        // one step at a time (the shrink layer: one step ahead measured no faster, 0.565 against
        // 0.572 ms, as its registers then hold it to 3 waves per SIMD instead of 4)
#pragma unroll 1
        for (int it = 0; it < STEPS; ++it) {
            bf16x8 bf[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) bf[nt] = wfrag(it, nt);
            step(it, bf);
        }
    }
}

// Tile of a conv block. Hardware blocks go to the 8 XCDs in turn (block w on XCD w mod 8), each XCD
// with its own L2. Each XCD takes a contiguous range of the tile order (x fastest, then rows, then
// images), so that horizontally and vertically adjacent tiles, whose halos are each other's
// interiors, run on one XCD close in time and the halo re-reads hit its L2 (a tile's two halo
// columns of the channel-first coefficient planes are 4 bytes of a 128-byte line each: fetched
// from memory per tile, they tripled the first layer's traffic). A tail of fewer than 8 blocks
// keeps its order.
__device__ __forceinline__ int conv_tile() {
    const int w = (int)blockIdx.x, per = (int)gridDim.x / 8;
    if (w >= per * 8) return w;
    return (w % 8) * per + w / 8;
}

// The decision |c scale| >= tau = softplus(o) is taken without forming tau: with a = |c scale| >= 0,
// m = max(o, 0), u = e^-|o| in (0, 1] and d = a - m, softplus(o) = m + log1p(u), so a >= softplus(o)
// <=> expm1(d) >= u. d is clamped to [0, 0.75] (below 0, expm1 < 0 < u; above, expm1 > 1 >= u), where
// expm1 is its Taylor polynomial of degree 9 (remainder < 2e-8 relative), and for o > 0, u is kept
// above 1e-30 (beyond o = 87 it underflows: then softplus(o) = o in FP32 and the test is d > 0). The
// low-pass plane takes o = -inf: u = 0, every coefficient kept. One hardware exponential replaces
// softplus's exponential, logarithm and reciprocal, with no branch, and the decision keeps softplus's
// relative precision for small and large thresholds alike.
__device__ __forceinline__ float shrink_keep(float v, float sc, float o) {
    constexpr float L2E = 1.44269504088896341f;
    const float d = fminf(fmaxf(fabsf(v * sc) - fmaxf(o, 0.0f), 0.0f), 0.75f);
    const float u = fmaxf(__builtin_amdgcn_exp2f(-fabsf(o) * L2E), o > 0.0f ? 1e-30f : 0.0f);
    float e = 1.0f / 362880.0f;
    e = fmaf(e, d, 1.0f / 40320.0f);
    e = fmaf(e, d, 1.0f / 5040.0f);
    e = fmaf(e, d, 1.0f / 720.0f);
    e = fmaf(e, d, 1.0f / 120.0f);
    e = fmaf(e, d, 1.0f / 24.0f);
    e = fmaf(e, d, 1.0f / 6.0f);
    e = fmaf(e, d, 0.5f);
    e = fmaf(e, d, 1.0f);
    return (e * d >= u) ? v : 0.0f;
}

// MODE 2: activations -> o + b -> shrink of the coefficients where |c scale| >= tau = softplus(o); 5: and tau;
// MODE 3 (training, last layer): o -> smooth-gate loss (each tile's sum to loss[tile]) and its gradient d o,
//   stored as bf16 channel-last planes [b][y][x][OUTC] (zero beyond COUTP and on the low-pass plane).
template <int CINP, int COUTP, int MODE, int OUTC = 32>
__global__ __launch_bounds__(THREADS) void k_conv3x3(ConvArgs a) {
    constexpr int NT = COUTP / 16;
    extern __shared__ unsigned short smem[];
    unsigned short* s_in = smem;
    const int tx = a.M / TW, ty = a.N / TH, tile = conv_tile();
    const int bx = tile % tx, by = (tile / tx) % ty, b = tile / (tx * ty);
    const int x0 = bx * TW, y0 = by * TH;
    constexpr bool SHRINK = MODE == 5 || MODE == 2;
    stage<CINP>(a, s_in, b, y0, x0);
    __syncthreads();
    const int w = threadIdx.x / 64, l = threadIdx.x % 64;
    const int lr = l % 16, lm = 4 * (l / 16);
    if constexpr (SHRINK) {
        // o = acc + bias, tau = softplus(o) (0 on the low-pass plane), keep |c scale| >= tau. A lane
        // holds 4 consecutive pixels of one channel, so it reads and writes the channel-first
        // coefficient planes directly as 16-byte vectors. At most 32 output channels per pass over
        // the staged tile, so that fewer accumulators leave room for more waves per SIMD.
        // (48 padded channels go in three passes of 16: a pass never reads weight rows past COUTP)
        constexpr int CG = COUTP <= 32 ? COUTP : (COUTP % 32 == 0 ? 32 : 16), NG = CG / 16;
        static_assert(COUTP % CG == 0, "the passes cover the padded output channels exactly");
        // offset of the lane's first vector in a plane: row y0 + 2 w, column x0 + lm; vector mt is
        // (mt / 2) rows and (mt % 2) 16 columns further
        const size_t pix0 = (size_t)(y0 + 2 * w) * a.M + x0 + lm;
#pragma unroll 1
        for (int c0 = 0; c0 < COUTP; c0 += CG) {
        // the pass's coefficient vectors, bias and scale are loaded before its products, so that
        // their latency overlaps the matrix work (loaded after the stores of the previous vector,
        // each load would also wait for those stores: one memory counter covers both)
        float4 cvs[NG][4];
        float biass[NG], scs[NG];
        size_t offs[NG];
#pragma unroll
        for (int nt = 0; nt < NG; ++nt) {
            const int k = c0 + nt * 16 + lr;
            biass[nt] = scs[nt] = 0.0f;
            offs[nt] = ((size_t)b * a.cout + k) * a.N * a.M + pix0;
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) cvs[nt][mt] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (k < a.cout) {
                biass[nt] = a.bias[k];
                scs[nt] = a.scale[b * a.cout + k];
                const float* cp = a.coef + offs[nt];
#pragma unroll
                for (int mt = 0; mt < 4; ++mt)
                    cvs[nt][mt] = *reinterpret_cast<const float4*>(cp + (mt / 2) * a.M + (mt % 2) * 16);
            }
        }
        f32x4 acc[4][NG];
        zero_acc(acc);
        mma<CINP, CG, 0>(a, s_in, acc, c0);
#pragma unroll
        for (int nt = 0; nt < NG; ++nt) {
            const int k = c0 + nt * 16 + lr;
            if (k >= a.cout) continue;
            const bool lowpass = (k == a.lowpass);
            const float bias = biass[nt];
            const float sc = scs[nt];
            float* op = a.out_f + offs[nt];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const int vo = (mt / 2) * a.M + (mt % 2) * 16;
                const float4 cv = cvs[nt][mt];
                const float v[4] = {cv.x, cv.y, cv.z, cv.w};
                float t[4], r[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (MODE == 5) {
                        t[i] = lowpass ? 0.0f : softplusf(acc[mt][nt][i] + bias);
                        r[i] = (fabsf(v[i] * sc) >= t[i]) ? v[i] : 0.0f;
                    } else {
                        r[i] = shrink_keep(v[i], sc, lowpass ? -INFINITY : acc[mt][nt][i] + bias);
                    }
                }
                *reinterpret_cast<float4*>(op + vo) = make_float4(r[0], r[1], r[2], r[3]);
                if constexpr (MODE == 5)
                    *reinterpret_cast<float4*>(a.tau + offs[nt] + vo) = make_float4(t[0], t[1], t[2], t[3]);
            }
        }
        }
    } else {
        f32x4 acc[4][NT];
        zero_acc(acc);
        mma<CINP, COUTP>(a, s_in, acc, 0);
        // bf16 results through LDS, then 16-byte channel-last stores of OUTC channels per pixel;
        // the output tile overwrites the staged input once every wave is done reading it
        unsigned short* s_out = smem;
        __syncthreads();
        __shared__ float s_loss[THREADS / 64];
        float lsum = 0.0f;
        const GateLoss gl = {a.gate_ehi, a.gate_elo, a.gate_c};
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const int prow = (2 * w + mt / 2) * TW + (mt % 2) * 16 + lm;
            const int y = y0 + 2 * w + mt / 2, x = x0 + (mt % 2) * 16 + lm;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int co = nt * 16 + lr;
                float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                if (co < a.cout && co != a.lowpass) {
                    const size_t off = (((size_t)b * a.cout + co) * a.N + y) * a.M + x;
                    const float4 cn = *reinterpret_cast<const float4*>(a.coef + off);
                    const float4 cc = *reinterpret_cast<const float4*>(a.coef2 + off);
                    const float sc = a.scale[b * a.cout + co], bias = a.bias[co];
                    const float n4[4] = {cn.x, cn.y, cn.z, cn.w}, c4[4] = {cc.x, cc.y, cc.z, cc.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) gate_loss(acc[mt][nt][i] + bias, n4[i] * sc, c4[i] * sc, gl, lsum, v[i]);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) s_out[(prow + i) * OUTC + co] = f2bf(v[i]);
            }
        }
        if constexpr (OUTC > COUTP) {
            for (int i = threadIdx.x; i < TH * TW * (OUTC - COUTP); i += THREADS)
                s_out[(i / (OUTC - COUTP)) * OUTC + COUTP + i % (OUTC - COUTP)] = 0;
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) lsum += __shfl_xor(lsum, off, 64);
        if (l == 0) s_loss[w] = lsum;
        __syncthreads();
        // the tile's squared residuals, summed over tiles by k_loss_sum
        if (threadIdx.x == 0) a.loss[tile] = (s_loss[0] + s_loss[1]) + (s_loss[2] + s_loss[3]);
        constexpr int CH = OUTC / 8;
        uint4* out = reinterpret_cast<uint4*>(a.out_bf);
        for (int i = threadIdx.x; i < TH * TW * CH; i += THREADS) {
            const int ch = i % CH, p = i / CH, px = p % TW, py = p / TW;
            out[(((size_t)b * a.N + y0 + py) * a.M + x0 + px) * CH + ch] =
                *reinterpret_cast<const uint4*>(s_out + p * OUTC + ch * 8);
        }
    }
}

// ---------------------------------------------------------------- persistent first layer
// The first layer (coefficients -> 32 hidden channels) as a persistent kernel: one 512-thread block
// per CU keeps the layer's weights in LDS and walks a list of 4 x 128-pixel tiles, software
// pipelined: while the matrix cores work on tile t out of LDS, the FP32 loads of tile t + 1 are
// in flight in registers; then tile t's bf16 outputs leave and tile t + 1 is converted into the staging
// buffer. Only these loads and stores use the vector-memory
// counter, so waiting for the prefetched tile never waits for weight loads, and the stores of
// tile t (issued after the prefetch) are not waited for. A tile reads 512-byte runs of each
// coefficient plane. The tiles
// of the batch are cut into 8 contiguous ranges, one per XCD (block w runs on XCD w mod 8), so
// that the halo re-reads of neighbouring tiles hit that XCD's L2. The hidden layer (32 bf16
// channels in, 32 out) runs in the same kernel with its own staging and 8 x 64-pixel tiles.
constexpr int PTH = 8, PHH = PTH + 2;     // tile rows, with halo
constexpr int PTW = 64, PHW = PTW + 2;    // tile columns, with halo
constexpr int PTHREADS = 512;             // 8 wavefronts, 64 pixels of a tile row each
// the first layer's tiles: its input is FP32 planes, and a tile's halo columns touch two more lines of every
// row of a plane, beside 4 lines of 128 pixels or 2 of 64, so its tiles are half as high and twice as wide:
// inference 878 -> 837 us at 16 x 512^2 x 49, 731 -> 706 at 33 planes; two tiles per block and less
// (4 x 256^2 x 33), where a strip's first two rows weigh more, 55.3 -> 56.2 us
constexpr int CTH = 4, CHH = CTH + 2, CTW = 128, CHW = CTW + 2;

template <int CS, bool COEF>
struct PLds {
    static constexpr int TH = COEF ? CTH : PTH, TW = COEF ? CTW : PTW, HH = TH + 2, HW = TW + 2;
    static constexpr int PIX = Pix<CS>::value;
    // bf16 per output channel of the staged weights: padded like a pixel, or, at 32 channels, where two blocks
    // have to share a CU's LDS, without padding and with the 16-byte pieces of every other group of 4
    // output channels exchanged in pairs (WSW), which avoids the same conflicts
    static constexpr int WP = CS == 32 ? 9 * CS : 9 * CS + 16, WSW = CS == 32 ? 16 : 0;
    static constexpr size_t in = (size_t)HH * HW * PIX * 2, w = (size_t)32 * WP * 2;
    static constexpr size_t bytes = in + w;
};

// Staged rows R0 .. R0 + NR - 1 of a tile's FP32 inputs (staged row yy is image row y0 + yy - 1),
// held in registers between their loads and their conversion to LDS.
template <int CS, int NR>
struct CoefRegs {
    static constexpr int G = CS / 8, QW = CTW / 4;
    static constexpr int TOTAL = G * QW * NR, NIT = (TOTAL + PTHREADS - 1) / PTHREADS;
    static constexpr int HTOTAL = G * NR * 2, HNIT = (HTOTAL + PTHREADS - 1) / PTHREADS;
    float4 v[NIT][8];
    float h[HNIT][8];
};

// Loads staged rows R0 .. R0 + NR - 1 of tile (b, y0, x0) in units of 8 consecutive channels (one
// 16-byte run of a staged pixel) of 4 consecutive interior pixels of one row: 8 aligned 16-byte
// loads, one per channel plane. Lanes take the channel groups fastest: in each load instruction the
// lanes of one group read consecutive 16-byte pieces of a row of a plane. A lane's channel group is
// fixed (512 is a multiple of G), and so are its 8 scales within an image. The two halo columns come
// one value per channel. J: only unit J of the interior, or, with J = NIT, only the halo.
template <int CS, int NR, int J = -1>
__device__ __forceinline__ void coef_load(const ConvArgs& a, CoefRegs<CS, NR>& r, int b, int y0, int x0, int R0) {
    using R = CoefRegs<CS, NR>;
    const int N = a.N, M = a.M, K = a.cin;
    const int g = (int)threadIdx.x % R::G, k0 = 8 * g;
    const size_t plane = (size_t)N * M;
    const float* base = a.coef + ((size_t)b * K + k0) * plane;
#pragma unroll
    for (int j = 0; j < R::HNIT; ++j) {
        if (J >= 0 && J != R::NIT) break;
        const int i = (int)threadIdx.x + j * PTHREADS;
        const int side = (i / R::G) % 2, yy = R0 + i / (2 * R::G);
        const int y = (y0 + yy - 1 + N) & (N - 1), x = side ? (x0 + CTW) & (M - 1) : (x0 - 1 + M) & (M - 1);
#pragma unroll
        for (int c = 0; c < 8; ++c)
            r.h[j][c] = (i < R::HTOTAL && k0 + c < K) ? base[c * plane + (size_t)y * M + x] : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < R::NIT; ++j) {
        if (J >= 0 && J != j) continue;
        const int i = (int)threadIdx.x + j * PTHREADS;
        const int q = (i / R::G) % R::QW, yy = R0 + i / (R::G * R::QW);
        const int y = (y0 + yy - 1 + N) & (N - 1);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            r.v[j][c] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (i < R::TOTAL && k0 + c < K)
                r.v[j][c] = *reinterpret_cast<const float4*>(base + c * plane + (size_t)y * M + x0 + 4 * q);
        }
    }
}

// z = bf16(c scale) of the loaded rows -> the channel-last staging buffer (16-byte runs), a ring of CHH
// rows whose row 0 is at slot rb
template <int CS, int NR, int J = -1>
__device__ __forceinline__ void coef_store(const CoefRegs<CS, NR>& r, const float* sc, unsigned short* s, int R0, int rb) {
    auto slot = [rb](int yy) { return yy + rb < CHH ? yy + rb : yy + rb - CHH; };
    using R = CoefRegs<CS, NR>;
    constexpr int PIX = Pix<CS>::value;
    const int g = (int)threadIdx.x % R::G;
#pragma unroll
    for (int j = 0; j < R::NIT; ++j) {
        if (J >= 0 && J != j) continue;
        const int i = (int)threadIdx.x + j * PTHREADS;
        if (i < R::TOTAL) {
            const int q = (i / R::G) % R::QW, yy = R0 + i / (R::G * R::QW);
            unsigned short* d = s + (slot(yy) * CHW + 1 + 4 * q) * PIX + 8 * g;
            const float4* w = r.v[j];
            const uint2 p0a = pack_bf16x4(w[0].x * sc[0], w[1].x * sc[1], w[2].x * sc[2], w[3].x * sc[3]);
            const uint2 p0b = pack_bf16x4(w[4].x * sc[4], w[5].x * sc[5], w[6].x * sc[6], w[7].x * sc[7]);
            const uint2 p1a = pack_bf16x4(w[0].y * sc[0], w[1].y * sc[1], w[2].y * sc[2], w[3].y * sc[3]);
            const uint2 p1b = pack_bf16x4(w[4].y * sc[4], w[5].y * sc[5], w[6].y * sc[6], w[7].y * sc[7]);
            const uint2 p2a = pack_bf16x4(w[0].z * sc[0], w[1].z * sc[1], w[2].z * sc[2], w[3].z * sc[3]);
            const uint2 p2b = pack_bf16x4(w[4].z * sc[4], w[5].z * sc[5], w[6].z * sc[6], w[7].z * sc[7]);
            const uint2 p3a = pack_bf16x4(w[0].w * sc[0], w[1].w * sc[1], w[2].w * sc[2], w[3].w * sc[3]);
            const uint2 p3b = pack_bf16x4(w[4].w * sc[4], w[5].w * sc[5], w[6].w * sc[6], w[7].w * sc[7]);
            *reinterpret_cast<uint4*>(d) = make_uint4(p0a.x, p0a.y, p0b.x, p0b.y);
            *reinterpret_cast<uint4*>(d + PIX) = make_uint4(p1a.x, p1a.y, p1b.x, p1b.y);
            *reinterpret_cast<uint4*>(d + 2 * PIX) = make_uint4(p2a.x, p2a.y, p2b.x, p2b.y);
            *reinterpret_cast<uint4*>(d + 3 * PIX) = make_uint4(p3a.x, p3a.y, p3b.x, p3b.y);
        }
    }
#pragma unroll
    for (int j = 0; j < R::HNIT; ++j) {
        if (J >= 0 && J != R::NIT) break;
        const int i = (int)threadIdx.x + j * PTHREADS;
        if (i < R::HTOTAL) {
            const int side = (i / R::G) % 2, yy = R0 + i / (2 * R::G);
            const float* w = r.h[j];
            const uint2 pa = pack_bf16x4(w[0] * sc[0], w[1] * sc[1], w[2] * sc[2], w[3] * sc[3]);
            const uint2 pb = pack_bf16x4(w[4] * sc[4], w[5] * sc[5], w[6] * sc[6], w[7] * sc[7]);
            *reinterpret_cast<uint4*>(s + (slot(yy) * CHW + (side ? CHW - 1 : 0)) * PIX + 8 * g) =
                make_uint4(pa.x, pa.y, pb.x, pb.y);
        }
    }
}

// Staged rows R0 .. R0 + NR - 1 of a tile's channel-last bf16 input (hidden activations or gradients, C
// channels) with the halo columns, in 16-byte units.
template <int NR, int C = 32, int THR = PTHREADS>
struct HidRegs {
    static constexpr int U = C / 8, TOTAL = NR * PHW * U, NIT = (TOTAL + THR - 1) / THR;
    uint4 v[NIT];
};

template <int NR, int C = 32, int THR = PTHREADS>
__device__ __forceinline__ void hid_load(const ConvArgs& a, HidRegs<NR, C, THR>& r, int b, int y0, int x0, int R0) {
    using R = HidRegs<NR, C, THR>;
    const int N = a.N, M = a.M;
    const uint4* in = reinterpret_cast<const uint4*>(a.in);
#pragma unroll
    for (int j = 0; j < R::NIT; ++j) {
        const int i = (int)threadIdx.x + j * THR;
        r.v[j] = make_uint4(0u, 0u, 0u, 0u);
        if (i < R::TOTAL) {
            const int ch = i % R::U, p = i / R::U, xx = p % PHW, yy = R0 + p / PHW;
            const int y = (y0 + yy - 1 + N) & (N - 1), x = (x0 + xx - 1 + M) & (M - 1);
            r.v[j] = in[(((size_t)b * N + y) * M + x) * R::U + ch];
        }
    }
}

template <int NR, int C = 32, int THR = PTHREADS, int PIX = Pix<C>::value>
__device__ __forceinline__ void hid_store(const HidRegs<NR, C, THR>& r, unsigned short* s, int R0) {
    using R = HidRegs<NR, C, THR>;
#pragma unroll
    for (int j = 0; j < R::NIT; ++j) {
        const int i = (int)threadIdx.x + j * THR;
        if (i < R::TOTAL) {
            const int ch = i % R::U, p = i / R::U;
            *reinterpret_cast<uint4*>(s + (R0 * PHW + p) * PIX + ch * 8) = r.v[j];
        }
    }
}

// The tiles of block w: t0 + j, t0 + j + per, ... < t1, where [t0, t1) is the (w mod 8)-th of 8
// contiguous ranges of the ntiles tiles, j = w / 8 and per = gridDim.x / 8 (the blocks on one XCD).
__device__ __forceinline__ void xcd_range(int ntiles, int& first, int& end, int& stride) {
    const int w = (int)blockIdx.x, per = (int)gridDim.x / 8, x = w % 8, j = w / 8;
    first = (int)(((long long)x * ntiles) / 8) + j;
    end = (int)(((long long)(x + 1) * ntiles) / 8);
    stride = per;
}

// The contiguous chunk [first, end) of tiles of block w: the j-th of per equal parts of the (w mod 8)-th
// of 8 contiguous ranges of the ntiles tiles (j = w / 8, per = gridDim.x / 8, the blocks on one XCD).
__device__ __forceinline__ void xcd_chunk(int ntiles, int& first, int& end) {
    const int w = (int)blockIdx.x, per = (int)gridDim.x / 8, x = w % 8, j = w / 8;
    const long long lo = ((long long)x * ntiles) / 8, hi = ((long long)(x + 1) * ntiles) / 8;
    first = (int)(lo + ((hi - lo) * j) / per);
    end = (int)(lo + ((hi - lo) * (j + 1)) / per);
}

// the bf16 of v where the bf16 of m (a saved activation, never NaN) is > 0, else 0
__device__ __forceinline__ uint2 positive_only(uint2 v, uint2 m) {
    auto f = [](unsigned x, unsigned y) {
        return x & (((int)(y << 16) > 0 ? 0xFFFFu : 0u) | ((int)y > 0xFFFF ? 0xFFFF0000u : 0u));
    };
    return make_uint2(f(v.x, m.x), f(v.y, m.y));
}

// COEF_RELU: the first layer (input: the FP32 coefficient planes, normalised and rounded on staging);
// COEF_RELU_Z: the first layer in training, which also writes the staged input z (bf16, channel-last, CINP
// channels) for the weight gradient; HID_RELU: the hidden layer (input: the bf16 activations of the
// first, CINP = 32); GRAD_MASK: backward data (input: gradient planes; flipped, transposed weights; the
// output is masked by relu's derivative, mask_act > 0, as it leaves).
// The first layer walks its block's chunk of tiles down vertical strips (tile index: rows of tiles
// fastest, then strips of 128 columns, then images), as a sliding window over a ring of staged rows: the
// staged tile's last two rows (its bottom halo and last row) are the next tile's first two and stay where
// they are, and only 4 new rows are loaded per tile (6 at the top of a strip); neighbouring chunks of an
// XCD run down neighbouring strips together, so the halo columns hit that XCD's L2 (0.449 -> 0.406 ms).
// The other layers, whose tiles are a quarter or half of the bytes, take their tiles interleaved over
// the XCD's blocks and load all 10 rows.
// The products are taken with the weights as the first operand, so that a lane ends with 4 consecutive
// channels of one pixel: 8 bytes that go straight to memory (a wavefront's store covers 16 pixels' 32-byte
// halves, the next one the other halves). Through LDS, from 2-byte stores, the outputs cost two more
// barriers and most of a tile's LDS stores, and the two rows of the sliding window were moved between two
// more: the network's inference 894 -> 881 us at 16 x 512^2 x 49, the first layer in training 0.52 -> 0.44 ms.
// In a training step at 16 x 512^2 x 49, z and the first layer took 0.33 + 0.40 ms as a packing pass and
// a layer of one-tile blocks, and the backward data of the last and the hidden layer 0.41 and 0.18 ms as
// one-tile blocks; here 0.44, 0.26 and 0.15 ms.
enum ConvKind { COEF_RELU, COEF_RELU_Z, HID_RELU, GRAD_MASK };
template <int CINP, ConvKind KIND>
__global__ __launch_bounds__(PTHREADS, CINP == 32 && KIND >= HID_RELU ? 4 : 2) void k_conv_relu(ConvArgs a, int ntiles) {
    constexpr bool FROM_COEF = KIND == COEF_RELU || KIND == COEF_RELU_Z;
    constexpr int CS = CINP, PIX = Pix<CS>::value, WP = PLds<CS, FROM_COEF>::WP, KCN = CS / 32, STEPS = 9 * KCN;
    constexpr bool SLIDE = FROM_COEF;
    using L = PLds<CS, FROM_COEF>;
    constexpr int TH = L::TH, TW = L::TW, HH = L::HH, HW = L::HW;
    constexpr int R0 = SLIDE ? 2 : 0, NR = HH - R0;  // staged rows loaded per tile (the prefetch)
    using Regs = typename std::conditional<FROM_COEF, CoefRegs<CS, NR>, HidRegs<NR, CS>>::type;
    // the scales of the lane's 8 channels, of image bsc; they are loaded where the image changes, and waited for
    // there, so that no wait for them holds up a tile's loads
    [[maybe_unused]] float sc[8];
    [[maybe_unused]] auto scales = [&](int b) {
        const int k0 = 8 * ((int)threadIdx.x % (CS / 8));
#pragma unroll
        for (int c = 0; c < 8; ++c) sc[c] = (k0 + c < a.cin) ? a.scale[b * a.cin + k0 + c] : 0.0f;
#pragma unroll
        for (int c = 0; c < 8; ++c) asm volatile("" : "+v"(sc[c]));
    };
    auto load_rows = [&](Regs& r, int b, int y0, int x0) {  // staged rows R0 .. HH - 1
        if constexpr (FROM_COEF) {
            coef_load<CS, NR>(a, r, b, y0, x0, R0);
        } else {
            hid_load<NR, CS>(a, r, b, y0, x0, R0);
        }
    };
    auto store_rows = [&](const Regs& r, unsigned short* s, [[maybe_unused]] int rb) {
        if constexpr (FROM_COEF) {
            coef_store<CS, NR>(r, sc, s, R0, rb);
        } else {
            hid_store<NR, CS>(r, s, R0);
        }
    };
    [[maybe_unused]] auto stage_top = [&](unsigned short* s, int b, int y0, int x0, int rb) {  // rows 0, 1 (SLIDE)
        CoefRegs<CS, 2> r2;
        coef_load<CS, 2>(a, r2, b, y0, x0, 0);
        coef_store<CS, 2>(r2, sc, s, 0, rb);
    };
    extern __shared__ unsigned short smem[];
    unsigned short* s_in = smem;
    unsigned short* s_w = smem + PLds<CS, FROM_COEF>::in / 2;
    const int tx = a.M / TW, ty = a.N / TH;
    int t, end, stride = 1;
    if constexpr (SLIDE) {
        xcd_chunk(ntiles, t, end);
    } else {
        xcd_range(ntiles, t, end, stride);
    }
    if (t >= end) return;  // the whole block: no tile
    auto tile_origin = [&](int tile, int& b, int& y0, int& x0) {
        if constexpr (SLIDE) {
            y0 = (tile % ty) * TH;
            x0 = ((tile / ty) % tx) * TW;
        } else {
            x0 = (tile % tx) * TW;
            y0 = ((tile / tx) % ty) * TH;
        }
        b = tile / (tx * ty);
    };
    // weights [co][tap][ci] -> LDS rows of WP bf16 (16-byte pieces)
    auto swap_of = [](int co) { return co & 4 ? PLds<CS, FROM_COEF>::WSW : 0; };
    for (int i = (int)threadIdx.x; i < 32 * 9 * CS / 8; i += PTHREADS) {
        const int co = i / (9 * CS / 8), r = i % (9 * CS / 8);
        *reinterpret_cast<uint4*>(s_w + co * WP + ((8 * r) ^ swap_of(co))) = reinterpret_cast<const uint4*>(a.W)[i];
    }
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), l = threadIdx.x % 64;
    const int lr = l % 16, lm = 4 * (l / 16), lk = 8 * (l / 16);
    const int wr = w / (TW / 64), wc = 64 * (w % (TW / 64));  // the wavefront's pixels in the tile
    const int lw = lk ^ swap_of(lr);
    [[maybe_unused]] f32x4 bias[2];
    if constexpr (KIND != GRAD_MASK) {
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) bias[nt] = *reinterpret_cast<const f32x4*>(a.bias + nt * 16 + lm);
    }
    int rb = 0;  // ring slot of staged row 0 (SLIDE)
    auto slot = [&](int yy) { return !SLIDE || yy + rb < HH ? yy + rb : yy + rb - HH; };
    Regs r;
    int b, y0, x0;
    tile_origin(t, b, y0, x0);
    if constexpr (SLIDE) {
        scales(b);
        stage_top(s_in, b, y0, x0, rb);
    }
    load_rows(r, b, y0, x0);
    store_rows(r, s_in, rb);
    if (t + stride < end) {
        int bn, yn, xn;
        tile_origin(t + stride, bn, yn, xn);
        load_rows(r, bn, yn, xn);
    }
    __syncthreads();
    for (;;) {
        if constexpr (KIND == COEF_RELU_Z) {  // the staged tile without its halo
            constexpr int ZU = CS / 8;
            uint4* z = reinterpret_cast<uint4*>(a.z);
#pragma unroll
            for (int j = 0; j < TH * TW * ZU / PTHREADS; ++j) {
                const int i = (int)threadIdx.x + j * PTHREADS, ch = i % ZU, p = i / ZU, px = p % TW, py = p / TW;
                z[(((size_t)b * a.N + y0 + py) * a.M + x0 + px) * ZU + ch] =
                    *reinterpret_cast<const uint4*>(s_in + (slot(py + 1) * HW + px + 1) * PIX + ch * 8);
            }
        }
        // a wavefront: 64 pixels of tile row wr, 4 m-tiles of 16
        f32x4 acc[4][2];
        zero_acc(acc);
#pragma unroll 1
        for (int it = 0; it < STEPS; ++it) {
            // inference takes each tap's channels together, training all taps of 32 channels at a time
            constexpr bool TAP_MAJOR = KIND == COEF_RELU || KIND == HID_RELU;
            const int tap = TAP_MAJOR ? it / KCN : it % 9, kc = TAP_MAJOR ? it % KCN : it / 9;
            const int dy = tap / 3, dx = tap % 3;
            bf16x8 bf[2];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                bf[nt] = *reinterpret_cast<const bf16x8*>(s_w + (nt * 16 + lr) * WP + tap * CS + kc * 32 + lw);
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const bf16x8 afr = *reinterpret_cast<const bf16x8*>(
                    s_in + (slot(wr + dy) * HW + wc + 16 * mt + lr + dx) * PIX + kc * 32 + lk);
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[nt], afr, acc[mt][nt], 0, 0, 0);
            }
        }
        // relu(acc + bias), or the masked gradient: 4 channels of a pixel per lane
        const size_t o8 = (((size_t)b * a.N + y0 + wr) * a.M + x0 + wc + lr) * 8 + l / 16;
        uint2* out = reinterpret_cast<uint2*>(a.out_bf) + o8;
        [[maybe_unused]] uint2 mk[4][2];
        if constexpr (KIND == GRAD_MASK) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) mk[mt][nt] = (reinterpret_cast<const uint2*>(a.mask_act) + o8)[mt * 128 + nt * 4];
        }
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const f32x4 v = acc[mt][nt];
                if constexpr (KIND == GRAD_MASK) {
                    out[mt * 128 + nt * 4] = positive_only(pack_bf16x4(v[0], v[1], v[2], v[3]), mk[mt][nt]);
                } else {
                    const f32x4 c = bias[nt];
                    out[mt * 128 + nt * 4] = pack_bf16x4(fmaxf(v[0] + c[0], 0.0f), fmaxf(v[1] + c[1], 0.0f),
                                                       fmaxf(v[2] + c[2], 0.0f), fmaxf(v[3] + c[3], 0.0f));
                }
            }
        if (t + stride >= end) break;
        const int tn = t + stride;
        int bn, yn, xn;
        tile_origin(tn, bn, yn, xn);
        __syncthreads();  // every wave is done reading the staged tile
        if constexpr (SLIDE) {
            // the next tile continues the strip: its first two staged rows are this one's last two; at the
            // top of a strip they come from memory
            rb = rb + TH < HH ? rb + TH : rb + TH - HH;
            if (bn != b) scales(bn);
            if (yn == 0) stage_top(s_in, bn, yn, xn, rb);
        }
        // The new staged rows of tile tn, loaded during this tile's products, make way for those of the one after,
        // piece by piece: memory is asked again while the rest is still being converted. With all conversions
        // before all loads the network's inference took 846 us against 824 (16 x 512^2 x 49), 713 against 687 (33).
        const bool more = tn + stride < end;
        int bq, yq, xq;
        tile_origin(more ? tn + stride : tn, bq, yq, xq);
        if constexpr (SLIDE) {
            constexpr int NIT = Regs::NIT;
            coef_store<CS, NR, NIT>(r, sc, s_in, R0, rb);
            if (more) coef_load<CS, NR, NIT>(a, r, bq, yq, xq, R0);
            coef_store<CS, NR, 0>(r, sc, s_in, R0, rb);
            if (more) coef_load<CS, NR, 0>(a, r, bq, yq, xq, R0);
            if constexpr (NIT == 2) {
                coef_store<CS, NR, 1>(r, sc, s_in, R0, rb);
                if (more) coef_load<CS, NR, 1>(a, r, bq, yq, xq, R0);
            }
        } else {
            store_rows(r, s_in, rb);
            if (more) load_rows(r, bq, yq, xq);
        }
        t = tn;
        b = bn;
        y0 = yn;
        x0 = xn;
        __syncthreads();  // the next tile is staged
    }
}

// ---------------------------------------------------------------- persistent shrink layer
// The last layer with the shrink decision (and, TAU, the thresholds it is taken with), persistent: two or three
// blocks per CU walk their XCD's range of 8 x 64-pixel tiles. A wavefront keeps the weights of one group of 16
// output channels in registers (36 VGPRs) and takes PTH / RH rows of the tile: per row, 4 m-tiles of 16 pixels x 9 taps of
// products out of the staged activations, then the decision on the row's coefficients where the matrix
// cores leave the outputs (a lane holds 4 consecutive pixels of one channel: 16-byte loads and stores in
// 64-byte runs, two of them to a line), with the next row's coefficients in flight. Nothing but the
// activations passes through LDS, and the wavefronts meet only where the staged tile changes (the
// next tile's activations are in registers by then), so products, decisions and memory overlap freely.
// The low-pass plane, the last, is kept whole: where it would be alone in its group (K = 17, 33, 49) it
// is copied and the group's products and decisions are left out. Per 16 x 512^2 x 49 batch: 0.44-0.46 ms;
// with the coefficients passed through LDS in three barrier phases per 32 channels, one block per CU,
// 0.50 ms. What bounds it: 1.64 GB of coefficients in and out and 0.35 GB of activations. With 256 threads (one,
// two and four groups) a thread holds 11 instead of 7 pieces of the next tile's activations, which with the
// weights pass the 168 registers of three waves per SIMD: 76 to 84 bytes of scratch a lane (three groups: none;
// with TAU 88 to 120, three groups 20). The network is still faster there than with the phases, which did
// not spill (8 x 512^2 images: 282 -> 257 us at 17 planes, 424 -> 351 at 33, 570 -> 527 at 64).
//
// NG groups of 16 output channels
template <int NG>
struct SCfg {
    static constexpr int RH = NG == 3 ? 2 : 4 / NG;  // parts of the tile's rows
    static constexpr int ROWS = PTH / RH, WAVES = NG * RH, THREADS = 64 * WAVES;
    static constexpr int BLOCKS = 12 / WAVES;  // per CU: 12 wavefronts of up to 168 registers
    // three blocks fit in a CU's LDS with 80-byte pixels (96 bytes leave two: the network's
    // inference 487 -> 557 us at 16 x 512^2 x 17); with three groups, two blocks by their registers, the wider
    // pitch takes 873 us against 881 (16 x 512^2 x 49)
    static constexpr int PIX = BLOCKS > 2 ? 40 : Pix<32>::value;
    static constexpr size_t LDS = (size_t)PHH * PHW * PIX * 2;
};

template <int NG, bool TAU>
__global__ __launch_bounds__((SCfg<NG>::THREADS), 3) void k_conv_shrink(ConvArgs a, int ntiles) {
    using C = SCfg<NG>;
    constexpr int PIX = C::PIX, THR = C::THREADS;
    using H = HidRegs<PHH, 32, THR>;
    extern __shared__ unsigned short smem[];
    const int tx = a.M / PTW, ty = a.N / PTH, K = a.cout;
    int t, end, stride;
    xcd_range(ntiles, t, end, stride);
    if (t >= end) return;  // the whole block: no tile
    auto tile_origin = [&](int tile, int& b, int& y0, int& x0) {
        x0 = (tile % tx) * PTW;
        y0 = ((tile / tx) % ty) * PTH;
        b = tile / (tx * ty);
    };
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), l = threadIdx.x % 64;
    const int lr = l % 16, lk = 8 * (l / 16), lm = 4 * (l / 16);
    const int r0 = (w / NG) * C::ROWS;
    // the lane's channel; lanes beyond the last plane repeat it and do not store
    const int kc = (w % NG) * 16 + lr, k = min(kc, K - 1);
    const bool lp_copy = K == 16 * NG + 1;
    bf16x8 wf[9];
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
        wf[tap] = *reinterpret_cast<const bf16x8*>(a.W + ((size_t)kc * 9 + tap) * 32 + lk);
    const bool lowpass = k == a.lowpass;
    const float bias = lowpass && !TAU ? -INFINITY : a.bias[k];
    const size_t plane = (size_t)a.N * a.M;
    auto row_off = [&](int b, int y0, int x0, int r) { return ((size_t)b * K + k) * plane + (size_t)(y0 + r) * a.M + x0 + lm; };
    H hr;
    float4 cv[4];
    int b, y0, x0;
    tile_origin(t, b, y0, x0);
    hid_load<PHH, 32, THR>(a, hr, b, y0, x0, 0);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) cv[mt] = *reinterpret_cast<const float4*>(a.coef + row_off(b, y0, x0, r0) + 16 * mt);
    for (;;) {
        hid_store<PHH, 32, THR, PIX>(hr, smem, 0);
        const float sc = a.scale[b * K + k];
        const int tn = t + stride;
        int bn = b, yn = y0, xn = x0;
        if (tn < end) tile_origin(tn, bn, yn, xn);
        __syncthreads();  // the tile is staged
        if (tn < end) hid_load<PHH, 32, THR>(a, hr, bn, yn, xn, 0);
        float4 lp = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        const size_t lpo = ((size_t)b * K + K - 1) * plane + (size_t)(y0 + (int)threadIdx.x / 16) * a.M + x0 +
                           4 * ((int)threadIdx.x % 16);
        if (lp_copy && threadIdx.x < PTH * PTW / 4) lp = *reinterpret_cast<const float4*>(a.coef + lpo);
#pragma unroll 1
        for (int r = 0; r < C::ROWS; ++r) {
            f32x4 acc[4];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) acc[mt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            const unsigned short* sr = smem + ((r0 + r) * PHW + lr) * PIX + lk;
#pragma unroll
            for (int tap = 0; tap < 9; ++tap)
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) {
                    const bf16x8 af =
                        *reinterpret_cast<const bf16x8*>(sr + ((tap / 3) * PHW + 16 * mt + tap % 3) * PIX);
                    acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, wf[tap], acc[mt], 0, 0, 0);
                }
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const float4 c = cv[mt];
                if constexpr (TAU) {
                    f32x4 t;
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[e] = lowpass ? 0.0f : softplusf(acc[mt][e] + bias);
                    if (kc < K) *reinterpret_cast<f32x4*>(a.tau + row_off(b, y0, x0, r0 + r) + 16 * mt) = t;
                    acc[mt] = f32x4{fabsf(c.x * sc) >= t[0] ? c.x : 0.0f, fabsf(c.y * sc) >= t[1] ? c.y : 0.0f,
                                    fabsf(c.z * sc) >= t[2] ? c.z : 0.0f, fabsf(c.w * sc) >= t[3] ? c.w : 0.0f};
                } else {
                    acc[mt] = f32x4{shrink_keep(c.x, sc, acc[mt][0] + bias), shrink_keep(c.y, sc, acc[mt][1] + bias),
                                    shrink_keep(c.z, sc, acc[mt][2] + bias), shrink_keep(c.w, sc, acc[mt][3] + bias)};
                }
            }
            // the next row's coefficients, of this tile or the first of the next one, in flight during its
            // products; issued before this row's stores, so that they need not wait for those
            const float* cp = a.coef + (r + 1 < C::ROWS ? row_off(b, y0, x0, r0 + r + 1) : row_off(bn, yn, xn, r0));
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) cv[mt] = *reinterpret_cast<const float4*>(cp + 16 * mt);
            float* op = a.out_f + row_off(b, y0, x0, r0 + r);
            if (kc < K) {
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) *reinterpret_cast<f32x4*>(op + 16 * mt) = acc[mt];
            }
        }
        if (lp_copy && threadIdx.x < PTH * PTW / 4) {
            if constexpr (TAU) {
                // the decision with a threshold of 0 that the other planes' lanes take (a NaN is not kept)
                const float ls = a.scale[b * K + K - 1];
                auto kept = [ls](float v) { return fabsf(v * ls) >= 0.0f ? v : 0.0f; };
                lp = make_float4(kept(lp.x), kept(lp.y), kept(lp.z), kept(lp.w));
            }
            *reinterpret_cast<float4*>(a.out_f + lpo) = lp;
            if constexpr (TAU) *reinterpret_cast<float4*>(a.tau + lpo) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        if (tn >= end) break;
        __syncthreads();  // every wavefront is past its products
        t = tn;
        b = bn;
        y0 = yn;
        x0 = xn;
    }
}

// ---------------------------------------------------------------- weight gradients
// dW[co][tap][ci] = sum over pixels p of dy[co](p) x[ci](p + tap offset): an MFMA GEMM with
// M = output channels, N = (tap, input channel), K = pixels. Both operands are channel-last in
// memory and in LDS, so a lane's 8 pixels of one channel are a column of the staged tile; the
// gfx950 transposing LDS read (ds_read_b64_tr_b16: each group of 16 lanes reads 4 pixels x 16
// channels, 8 bytes a lane, and receives one channel's 4 pixels a lane) delivers them without a
// transposed copy, and a tap's column offset is an address offset. Staging is then plain 16-byte
// copies. At 16 x 512^2 x 49 the three layers (64 x 32, 32 x 64 and 32 x 32 channels) take 180, 187
// and 120 us, 4.5 TB/s of operands; staged channel-major with 2-byte copies they took 1320, 1108
// and 723 us.
//
// A block walks units of a 32-pixel column strip by R rows, 4 rows (a chunk) at a time. Row yy of x
// meets the dy rows yy + 1, yy, yy - 1 (taps 0, 1, 2 of the kernel's rows), so each x fragment is read
// from LDS once per kernel column and multiplied with three dy fragments that roll through registers;
// a chunk stages x rows yy and dy rows yy + 1, and a unit begins with a chunk of dy rows alone. The
// chunks are double buffered in LDS, with the next chunk's loads in registers during the products (one
// barrier per chunk); two blocks per CU keep about 50 KB in flight, which is what the path is bound
// by (0.8 GB of operands per layer at 16 x 512^2).
// The staged pixels have a pitch (WgradPitch) that puts the 16 pixels of one read on distinct banks.
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

template <int C>
struct WgradPitch {  // bf16 per staged pixel: an odd multiple of 32 bytes
    static constexpr int value = (C % 32 == 0) ? C + 16 : C;
};

template <int CX, int CY>
struct WgradCfg {
    static constexpr int XP = WgradPitch<CX>::value, YP = WgradPitch<CY>::value;
    static constexpr int RC = 4;                                     // rows per chunk
    static constexpr int XB = RC * HW * XP, YB = RC * TW * YP;       // bf16 per staged chunk
    static constexpr size_t LDS = (size_t)2 * (XB + YB) * 2;         // double buffered
    static constexpr int XU = RC * HW * CX / 8, YU = RC * TW * CY / 8;  // 16-byte units per chunk
    static constexpr int XN = (XU + THREADS - 1) / THREADS, YN = (YU + THREADS - 1) / THREADS;
    static constexpr int NCG = CX / 16, MT = CY / 16;
    static constexpr int WM = 4 / NCG;                // wavefronts that share a group of 16 input channels
    static constexpr int MTW = (MT + WM - 1) / WM;    // groups of 16 output channels of one wavefront
};

// the 32 pixels x 16 channels at s (pitch P bf16 per pixel) as one MFMA operand: lane l holds channel
// l % 16; the order of the pixels is the same for every operand read this way
template <int P>
__device__ __forceinline__ bf16x8 tr_frag(const unsigned short* s) {
    const int l = threadIdx.x % 64;
    const unsigned short* p = s + (l / 4) * P + (l % 4) * 4;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + 16 * P));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// units of R rows (a multiple of 4 that divides N); dy has a.dy_ch >= CY channels per pixel
template <int CX, int CY>
__global__ __launch_bounds__(THREADS, 2) void k_wgrad(WgradArgs a, int R) {
    using C = WgradCfg<CX, CY>;
    constexpr int MTW = C::MTW;
    extern __shared__ unsigned short smem[];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), l = threadIdx.x % 64;
    // output-channel groups m0, m0 + WM, ...; where that passes the last group (a lone or third one), the
    // wavefront repeats the last group and does not write it
    const int cg = w % C::NCG, m0 = C::WM == 1 ? 0 : w / C::NCG;
    auto group = [&](int j) { return C::MT % C::WM == 0 ? m0 + C::WM * j : min(m0 + C::WM * j, C::MT - 1); };
    const int N = a.N, M = a.M;
    const int tx = M / TW, ty = N / R, nunits = a.batch * tx * ty, nc = R / C::RC;
    // each XCD (blocks b, b + 8, ...) takes a contiguous range of units: neighbouring strips, which
    // share halo columns, run on one XCD; gridDim.x is a multiple of 8
    int u, uend;
    {
        const int per = (int)gridDim.x / 8, x = (int)blockIdx.x % 8, j = (int)blockIdx.x / 8;
        const long long lo = ((long long)x * nunits) / 8, hi = ((long long)(x + 1) * nunits) / 8;
        u = (int)(lo + ((hi - lo) * j) / per);
        uend = (int)(lo + ((hi - lo) * (j + 1)) / per);
    }
    f32x4 acc[9][MTW], accb[MTW];
#pragma unroll
    for (int j = 0; j < MTW; ++j) {
        accb[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[t][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    bf16x8 one;
#pragma unroll
    for (int j = 0; j < 8; ++j) one[j] = (__bf16)1.0f;
    // chunk c of unit q: x rows r0 + 4 c .., dy rows r0 + 4 c + 1 .. (the rows wrap around the plane); of chunk
    // -1 only the dy rows r0 - 1 and r0 are used. Lanes past the last unit load it again, so that no load
    // is conditional (conditional loads had put the registers into scratch memory).
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    u32x4 xv[C::XN], yv[C::YN];
    auto load = [&](int q, int c) {
        const int x0 = (q % tx) * TW, b = q / (tx * ty), r = ((q / tx) % ty) * R + C::RC * c + N;
        const u32x4* xs = reinterpret_cast<const u32x4*>(a.xb) + (size_t)b * N * M * (CX / 8);
        const u32x4* ys = reinterpret_cast<const u32x4*>(a.dy) + (size_t)b * N * M * (a.dy_ch / 8);
#pragma unroll
        for (int j = 0; j < C::XN; ++j) {
            const int i = min((int)threadIdx.x + j * THREADS, C::XU - 1);
            const int ch = i % (CX / 8), p = i / (CX / 8), px = p % HW, py = p / HW;
            const int y = (r + py) & (N - 1), x = (x0 + px - 1 + M) & (M - 1);
            xv[j] = xs[((size_t)y * M + x) * (CX / 8) + ch];
        }
#pragma unroll
        for (int j = 0; j < C::YN; ++j) {
            const int i = min((int)threadIdx.x + j * THREADS, C::YU - 1);
            const int ch = i % (CY / 8), p = i / (CY / 8), px = p % TW, py = p / TW;
            const int y = (r + 1 + py) & (N - 1);
            yv[j] = ys[((size_t)y * M + x0 + px) * (a.dy_ch / 8) + ch];
        }
    };
    auto store = [&](unsigned short* sx, unsigned short* sy) {
#pragma unroll
        for (int j = 0; j < C::XN; ++j) {
            const int i = (int)threadIdx.x + j * THREADS;
            if (i < C::XU) *reinterpret_cast<u32x4*>(sx + (i / (CX / 8)) * C::XP + (i % (CX / 8)) * 8) = xv[j];
        }
#pragma unroll
        for (int j = 0; j < C::YN; ++j) {
            const int i = (int)threadIdx.x + j * THREADS;
            if (i < C::YU) *reinterpret_cast<u32x4*>(sy + (i / (CY / 8)) * C::YP + (i % (CY / 8)) * 8) = yv[j];
        }
    };
    bf16x8 af[3][MTW] = {};  // dy rows yy + 1, yy, yy - 1
    auto roll = [&](const unsigned short* row) {
#pragma unroll
        for (int j = 0; j < MTW; ++j) {
            af[2][j] = af[1][j];
            af[1][j] = af[0][j];
            af[0][j] = tr_frag<C::YP>(row + 16 * group(j));
        }
    };
    int c = -1, buf = 0;
    if (u < uend) load(u, c);
    while (u < uend) {
        unsigned short* sx = smem + buf * (C::XB + C::YB);
        unsigned short* sy = sx + C::XB;
        store(sx, sy);
        const int cc = c;
        if (++c == nc) {
            c = -1;
            ++u;
        }
        if (u < uend) load(u, c);
        __syncthreads();
#pragma unroll 1
        for (int r = cc < 0 ? 2 : 0; r < C::RC; ++r) {
            roll(sy + r * TW * C::YP);
            if (cc < 0) continue;
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const bf16x8 bf = tr_frag<C::XP>(sx + (r * HW + dx) * C::XP + 16 * cg);
#pragma unroll
                for (int j = 0; j < MTW; ++j)
#pragma unroll
                    for (int dy = 0; dy < 3; ++dy)
                        acc[3 * dy + dx][j] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[dy][j], bf, acc[3 * dy + dx][j], 0, 0, 0);
            }
            if (cg == 0) {  // the bias gradient: dy times ones, every dy row once
#pragma unroll
                for (int j = 0; j < MTW; ++j)
                    accb[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[0][j], one, accb[j], 0, 0, 0);
            }
        }
        buf ^= 1;
    }
    // partial dW in [co][tap][ci] order, then the bias partial
    float* part = a.part + (size_t)blockIdx.x * (CY * 9 * CX + CY);
#pragma unroll
    for (int j = 0; j < MTW; ++j) {
        const int m = m0 + C::WM * j;
        if (m < C::MT) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int co = m * 16 + 4 * (l / 16) + i;
#pragma unroll
                for (int t = 0; t < 9; ++t) part[((size_t)co * 9 + t) * CX + cg * 16 + l % 16] = acc[t][j][i];
                if (cg == 0 && l % 16 == 0) part[CY * 9 * CX + co] = accb[j][i];
            }
        }
    }
}

// grads in natural order: dW[co][ci][3][3] (co < cout, ci < cin), then db[co]; sums of nblk partials in a
// fixed order. A block sums 32 consecutive values of the partials (128-byte runs), each by 8 threads that
// take every 8th partial, added in order: 8 us for 512 partials of 18464 values (one thread per value,
// in the gradients' order, waited for 512 strided loads in turn: 142 us).
constexpr int RED_V = 32, RED_G = 8;
__global__ __launch_bounds__(RED_V* RED_G) void k_wgrad_reduce(const float* __restrict__ part, float* __restrict__ dW,
                                                             float* __restrict__ db, int nblk, int cout, int cin,
                                                             int coutp, int cinp) {
    __shared__ float s[RED_G][RED_V];
    const int v = (int)threadIdx.x % RED_V, g = (int)threadIdx.x / RED_V;
    const int nw = coutp * 9 * cinp, stride = nw + coutp, src = (int)blockIdx.x * RED_V + v;
    float t = 0.0f;
    if (src < stride) {
#pragma unroll 8
        for (int b = g; b < nblk; b += RED_G) t += part[(size_t)b * stride + src];
    }
    s[g][v] = t;
    __syncthreads();
    if (g != 0 || src >= stride) return;
    t = s[0][v];
#pragma unroll
    for (int i = 1; i < RED_G; ++i) t += s[i][v];
    if (src < nw) {
        const int ci = src % cinp, tap = (src / cinp) % 9, co = src / (9 * cinp);
        if (co < cout && ci < cin) dW[((size_t)co * cin + ci) * 9 + tap] = t;
    } else if (src - nw < cout) {
        db[src - nw] = t;
    }
}

// *loss = scale x the sum of the n tiles' squared residuals, in double precision and a fixed order (one block)
__global__ __launch_bounds__(1024) void k_loss_sum(const float* __restrict__ part, int n, float scale,
                                                float* __restrict__ loss) {
    __shared__ double s[1024];
    double t = 0.0;
    for (int i = (int)threadIdx.x; i < n; i += 1024) t += (double)part[i];
    s[threadIdx.x] = t;
    __syncthreads();
    for (int h = 512; h >= 1; h /= 2) {
        if ((int)threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = (float)(s[0] * (double)scale);
}

// natural W[co][ci][3][3] -> flipped, transposed bf16 [ci][8 - tap][co], padded to cinp' x coutp'
// (the weights of the backward-data correlation)
__global__ void k_pack_weights_t(const float* __restrict__ W, unsigned short* __restrict__ out, int cout, int cin,
                                 int rows, int cols) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * 9 * cols) return;
    const int co = i % cols, tap = (i / cols) % 9, ci = i / (cols * 9);
    out[i] = (ci < cin && co < cout) ? f2bf(W[((size_t)co * cin + ci) * 9 + (8 - tap)]) : (unsigned short)0;
}

// Adam (bias-corrected) on n FP32 parameters; step t >= 1
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                       int n, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// inverse noise scale per (image, filter): 1 / (sigma_b RMS_k)
__global__ void k_inv_scale(const float* __restrict__ sigma, const float* __restrict__ rms, float* __restrict__ out,
                            int B, int K) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < B * K) out[i] = 1.0f / (sigma[i / K] * rms[i % K]);
}

// natural FP32 weights W[co][ci][3][3] -> bf16 [co][tap][ci] padded to COUTP x CINP (zeros)
__global__ void k_pack_weights(const float* __restrict__ W, unsigned short* __restrict__ out, int cout, int cin,
                               int coutp, int cinp) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= coutp * 9 * cinp) return;
    const int ci = i % cinp, tap = (i / cinp) % 9, co = i / (cinp * 9);
    out[i] = (co < cout && ci < cin) ? f2bf(W[((size_t)co * cin + ci) * 9 + tap]) : (unsigned short)0;
}

__global__ void k_pack_bias(const float* __restrict__ b, float* __restrict__ out, int n, int np) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < np) out[i] = i < n ? b[i] : 0.0f;
}

template <int CINP, int COUTP, int MODE, int OUTC = 32>
hipError_t conv_t(const ConvArgs& a, int batch, hipStream_t st) {
    const void* fn = reinterpret_cast<const void*>(&k_conv3x3<CINP, COUTP, MODE, OUTC>);
    const size_t lds = conv_lds_bytes<CINP, OUTC, MODE>();
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    const size_t blocks = (size_t)batch * (a.N / TH) * (a.M / TW);
    hipLaunchKernelGGL((k_conv3x3<CINP, COUTP, MODE, OUTC>), dim3((unsigned)blocks), dim3(THREADS), lds, st,
                       a);
    return hipGetLastError();
}

template <int CINP, ConvKind KIND>
hipError_t conv_relu_t(const ConvArgs& a, int batch, hipStream_t st) {
    using L = PLds<CINP, (KIND < HID_RELU)>;
    const void* fn = reinterpret_cast<const void*>(&k_conv_relu<CINP, KIND>);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)L::bytes);
    if (e != hipSuccess) return e;
    const int ntiles = batch * (a.N / L::TH) * (a.M / L::TW);
    // blocks per CU its registers and LDS allow (64 channels or coefficients: one, 159 KB; 32 bf16
    // channels: two, 82 KB), a multiple of the 8 XCDs
    const int blocks = (CINP == 32 && KIND >= HID_RELU ? 2 : 1) * std::max(8, a.cus / 8 * 8);
    hipLaunchKernelGGL((k_conv_relu<CINP, KIND>), dim3((unsigned)blocks), dim3(PTHREADS), L::bytes, st, a,
                       ntiles);
    return hipGetLastError();
}

template <int NG>
hipError_t conv_shrink_t(const ConvArgs& a, int batch, hipStream_t st) {
    using C = SCfg<NG>;
    const int ntiles = batch * (a.N / PTH) * (a.M / PTW);
    const int blocks = C::BLOCKS * std::max(8, a.cus / 8 * 8);  // a multiple of the 8 XCDs
    const dim3 g((unsigned)blocks), t(C::THREADS);
    if (a.tau) {
        hipLaunchKernelGGL((k_conv_shrink<NG, true>), g, t, C::LDS, st, a, ntiles);
    } else {
        hipLaunchKernelGGL((k_conv_shrink<NG, false>), g, t, C::LDS, st, a, ntiles);
    }
    return hipGetLastError();
}

template <int CX, int CY>
hipError_t wgrad_t(const WgradArgs& a, int blocks, hipStream_t st) {
    using C = WgradCfg<CX, CY>;
    if (blocks % 8 != 0 || a.dy_ch < CY || a.N % 8 != 0 || a.M % TW != 0) return hipErrorInvalidValue;
    const void* fn = reinterpret_cast<const void*>(&k_wgrad<CX, CY>);
    if (C::LDS > 65536) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::LDS);
        if (e != hipSuccess) return e;
    }
    // rows per unit: as many as leave every block two units (each unit begins with a chunk of dy rows
    // alone), at least 8
    int R = 8;
    while (2 * R <= a.N && (long long)a.batch * (a.M / TW) * (a.N / (2 * R)) >= 2LL * blocks) R *= 2;
    hipLaunchKernelGGL((k_wgrad<CX, CY>), dim3((unsigned)blocks), dim3(THREADS), C::LDS, st, a, R);
    return hipGetLastError();
}

}  // namespace

int shrink_cinp(int K) { return K <= 32 ? 32 : 64; }
int shrink_coutp(int K) { return (K + 15) / 16 * 16; }
bool shrink_supported(int K, int N, int M) { return K >= 1 && K <= 64 && N >= TH && N % TH == 0 && M % 128 == 0; }

ShrinkLayout shrink_layout(int K) {
    ShrinkLayout L;
    const int c1 = shrink_cinp(K), c3 = shrink_coutp(K);
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    size_t off = 0;
    L.w1 = off;
    off = al(off + (size_t)32 * 9 * c1 * 2);
    L.w2 = off;
    off = al(off + (size_t)32 * 9 * 32 * 2);
    L.w3 = off;
    off = al(off + (size_t)c3 * 9 * 32 * 2);
    L.b1 = off;
    off = al(off + 32 * 4);
    L.b2 = off;
    off = al(off + 32 * 4);
    L.b3 = off;
    off = al(off + (size_t)c3 * 4);
    L.bytes = off;
    return L;
}

hipError_t launch_shrink_pack(int K, const float* W1, const float* b1, const float* W2, const float* b2,
                              const float* W3, const float* b3, void* packed, hipStream_t st) {
    const ShrinkLayout L = shrink_layout(K);
    char* p = static_cast<char*>(packed);
    const int c1 = shrink_cinp(K), c3 = shrink_coutp(K);
    auto grid = [](int n) { return dim3((unsigned)((n + 255) / 256)); };
    hipLaunchKernelGGL(k_pack_weights, grid(32 * 9 * c1), dim3(256), 0, st, W1, (unsigned short*)(p + L.w1), 32, K, 32, c1);
    hipLaunchKernelGGL(k_pack_weights, grid(32 * 9 * 32), dim3(256), 0, st, W2, (unsigned short*)(p + L.w2), 32, 32, 32, 32);
    hipLaunchKernelGGL(k_pack_weights, grid(c3 * 9 * 32), dim3(256), 0, st, W3, (unsigned short*)(p + L.w3), K, 32, c3, 32);
    hipLaunchKernelGGL(k_pack_bias, grid(32), dim3(256), 0, st, b1, (float*)(p + L.b1), 32, 32);
    hipLaunchKernelGGL(k_pack_bias, grid(32), dim3(256), 0, st, b2, (float*)(p + L.b2), 32, 32);
    hipLaunchKernelGGL(k_pack_bias, grid(c3), dim3(256), 0, st, b3, (float*)(p + L.b3), K, c3);
    return hipGetLastError();
}

hipError_t launch_inv_scale(const float* sigma, const float* rms, float* out, int B, int K, hipStream_t st) {
    hipLaunchKernelGGL(k_inv_scale, dim3((unsigned)((B * K + 255) / 256)), dim3(256), 0, st, sigma, rms, out, B, K);
    return hipGetLastError();
}

hipError_t launch_conv(int layer, int K, const ConvArgs& a, int batch, hipStream_t st) {
    const bool c32 = shrink_cinp(K) == 32;
    if (layer == 0) return c32 ? conv_relu_t<32, COEF_RELU_Z>(a, batch, st) : conv_relu_t<64, COEF_RELU_Z>(a, batch, st);
    if (layer == 1) return conv_relu_t<32, HID_RELU>(a, batch, st);  // h1 -> h2
    if (layer == 6) return c32 ? conv_relu_t<32, COEF_RELU>(a, batch, st) : conv_relu_t<64, COEF_RELU>(a, batch, st);
    if (layer == 3) {  // training: last layer with the loss epilogue, gradient planes of shrink_cinp(K) channels
        // the low-pass plane, the last, has no loss and a zero gradient: groups of 16 channels up to K - 1
        // (at K = 49 three groups of products and epilogue instead of four)
        switch (std::max(16, shrink_coutp(K - 1))) {
            case 16: return conv_t<32, 16, 3, 32>(a, batch, st);
            case 32: return c32 ? conv_t<32, 32, 3, 32>(a, batch, st) : conv_t<32, 32, 3, 64>(a, batch, st);
            case 48: return conv_t<32, 48, 3, 64>(a, batch, st);
            case 64: return conv_t<32, 64, 3, 64>(a, batch, st);
        }
        return hipErrorInvalidValue;
    }
    if (layer == 4 || (layer == 5 && c32)) return conv_relu_t<32, GRAD_MASK>(a, batch, st);  // backward data
    if (layer == 5) return conv_relu_t<64, GRAD_MASK>(a, batch, st);
    // The shrink layer in the persistent kernel or in one-tile blocks of 8 x 32. The persistent kernel's gains are the
    // low-pass plane's group left out where it is alone (17, 33, 49 planes) and less staging and weight traffic;
    // a short call pays for its serial rows and, with one, two and four groups, its spills. So without the
    // thresholds it takes 17 and 33 to 49 planes always, two and four groups from 512 and 256 of its 8 x 64
    // tiles on (2 / groups to a CU), and none of up to 16 planes. With them, which it has to store and to keep
    // in registers, it takes 17, 33 and 49 planes from two tiles per CU on, 50 to 64 from six. The network, us, one-tile /
    // persistent, without and with thresholds:
    //   planes   128 tiles                  256 tiles                  512 tiles                  2048 tiles
    //   16       21.4 / 23.7  22.6 / 25.9   28.2 / 29.2  30.3 / 32.1   39.8 / 39.8  43.0 / 42.8   115 / 115  134 / 138
    //   17       24.4 / 23.7  23.8 / 26.4   32.2 / 29.6  32.7 / 33.0   45.2 / 40.2  46.6 / 43.7   129 / 121  152 / 149
    //   32       24.2 / 28.5  28.6 / 34.8   33.8 / 34.6  37.5 / 40.5   49.5 / 46.3  54.1 / 53.7   173 / 176  215 / 228
    //   33       32.0 / 31.7  35.9 / 38.0   42.3 / 37.6  44.4 / 43.8   59.6 / 51.4  63.0 / 58.8   212 / 191  254 / 243
    //   48       34.1 / 34.3  40.4 / 39.6   44.3 / 40.1  47.9 / 44.3   62.8 / 61.7  69.7 / 70.6   237 / 223  296 / 296
    //   49       37.0 / 34.4  39.5 / 40.2   46.5 / 40.4  48.6 / 45.0   67.9 / 62.4  72.6 / 71.1   256 / 226  322 / 306
    //   50       37.8 / 41.3  42.2 / 50.0   46.9 / 46.4  50.4 / 55.0   67.8 / 62.1  75.0 / 71.2   258 / 231  325 / 308
    //   64       38.4 / 43.1  43.5 / 52.4   49.1 / 49.0  54.4 / 58.9   72.4 / 67.1  82.8 / 81.8   308 / 288  418 / 382
    // Both sum and decide alike, bit by bit.
    const long long tiles = (long long)batch * (a.N / PTH) * (a.M / PTW);
    const int groups = std::max(1, (K - 1 + 15) / 16);  // groups of 16 channels up to the low-pass plane
    const bool alone = K > 1 && K % 16 == 1;
    const bool persistent = a.tau ? (alone ? tiles >= 2LL * a.cus : groups == 4 && tiles >= 6LL * a.cus)
                                  : (alone || groups == 3 || (groups > 1 && tiles * groups >= 4LL * a.cus));
    if (!persistent) {
        switch (shrink_coutp(K)) {
            case 16: return a.tau ? conv_t<32, 16, 5>(a, batch, st) : conv_t<32, 16, 2>(a, batch, st);
            case 32: return a.tau ? conv_t<32, 32, 5>(a, batch, st) : conv_t<32, 32, 2>(a, batch, st);
            case 48: return a.tau ? conv_t<32, 48, 5>(a, batch, st) : hipErrorInvalidValue;  // (without: persistent)
            case 64: return a.tau ? conv_t<32, 64, 5>(a, batch, st) : conv_t<32, 64, 2>(a, batch, st);
        }
        return hipErrorInvalidValue;
    }
    switch (groups) {
        case 1: return conv_shrink_t<1>(a, batch, st);
        case 2: return conv_shrink_t<2>(a, batch, st);
        case 3: return conv_shrink_t<3>(a, batch, st);
        case 4: return conv_shrink_t<4>(a, batch, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_wgrad(int layer, int K, const WgradArgs& a, int blocks, hipStream_t st) {
    if (layer == 0) return shrink_cinp(K) == 32 ? wgrad_t<32, 32>(a, blocks, st) : wgrad_t<64, 32>(a, blocks, st);
    if (layer == 1) return wgrad_t<32, 32>(a, blocks, st);
    switch (shrink_coutp(K)) {
        case 16: return wgrad_t<32, 16>(a, blocks, st);
        case 32: return wgrad_t<32, 32>(a, blocks, st);
        case 48: return wgrad_t<32, 48>(a, blocks, st);
        case 64: return wgrad_t<32, 64>(a, blocks, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_wgrad_reduce(const float* part, float* dW, float* db, int nblk, int cout, int cin, int coutp, int cinp,
                               hipStream_t st) {
    const int n = coutp * 9 * cinp + coutp;
    hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)((n + RED_V - 1) / RED_V)), dim3(RED_V * RED_G), 0, st, part, dW, db,
                       nblk, cout, cin, coutp, cinp);
    return hipGetLastError();
}

hipError_t launch_loss_sum(const float* part, int n, float scale, float* loss, hipStream_t st) {
    hipLaunchKernelGGL(k_loss_sum, dim3(1), dim3(1024), 0, st, part, n, scale, loss);
    return hipGetLastError();
}

hipError_t launch_pack_weights_t(const float* W, unsigned short* out, int cout, int cin, int rows, int cols,
                                 hipStream_t st) {
    const int n = rows * 9 * cols;
    hipLaunchKernelGGL(k_pack_weights_t, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, W, out, cout, cin, rows,
                       cols);
    return hipGetLastError();
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, int n, float lr, float b1, float b2, float eps,
                       int step, hipStream_t st) {
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, g, m, v, n, lr, b1, b2, eps, c1,
                       c2);
    return hipGetLastError();
}

}  // namespace shear
