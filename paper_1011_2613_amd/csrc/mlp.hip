// mlp.hip -- learned drag closure on gfx950 matrix cores.
//
// Network 40 -> 128 -> 128 -> 128 -> 1, SiLU on the hidden layers.  Every
// matrix product uses v_mfma_f32_16x16x32_bf16: bfloat16 operands, binary32
// accumulation.  Operand fragments (one wavefront, 64 lanes):
//   A (16 x 32): lane l holds A[l % 16][8 (l / 16) + j], j = 0..7
//   B (32 x 16): lane l holds B[8 (l / 16) + j][l % 16]
//   D (16 x 16): lane l holds D[4 (l / 16) + i][l % 16], i = 0..3
//
// Large inference batches (k_mlp_forward): the weights stay in LDS (rows padded
// so the 16 rows a fragment touches fall in distinct LDS banks) and each
// wavefront runs its own 32-row tiles through every layer.
// Small batches and training (k_mlp_rows): a workgroup takes a few 16-row tiles
// together, each of its eight wavefronts holding the weights of 16 output
// features in registers; in training the same workgroup runs the backward pass
// of its rows from LDS and leaves one partial gradient, which k_mlp_reduce adds
// up in workgroup order (deterministic, no atomics), with the Adam step on the
// binary32 masters and the refresh of the bfloat16 copies in the same kernel.
#include <math.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <new>

#include "../../include/lbimb.h"
#include "../../include/mlp_closure.h"
#include "internal.h"

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int NIN = MLP_NIN, NH = MLP_NHID, KIN = 64;  // input padded to 64
constexpr int S1 = 72;   // LDS row stride (bf16) of W1 and of the padded input
constexpr int SH = 136;  // LDS row stride (bf16) of 128-wide rows
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + NH * NIN, OFF_W2 = OFF_B1 + NH,
              OFF_B2 = OFF_W2 + NH * NH, OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NH * NH,
              OFF_W4 = OFF_B3 + NH, OFF_B4 = OFF_W4 + NH, NPAR = OFF_B4 + 1;
static_assert(NPAR == MLP_NPARAMS, "parameter count");

// bfloat16 weight copies used by the kernels (global memory):
//   w1 [128][64] (columns 40..63 zero), w2, w3 [128][128], w4 [16][128] (rows 1..15 zero),
//   w2t, w3t the transposes of w2 and w3 (operands of the backward pass)
struct Wbf {
    __bf16 *w1, *w2, *w3, *w4, *w2t, *w3t;
};

// LDS written by some lanes of a wavefront and read by others: order the
// accesses within the wavefront (no cross-wavefront barrier is needed because
// each wavefront owns its activation buffers).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// SiLU of the forward pass from the hardware base-2 exponential and
// reciprocal (e^-z = 2^(-z log2 e)): a few ulp of binary32, far below the
// bfloat16 rounding that follows, and about a fifth of the instructions of
// the correctly rounded form, which made the forward pass ALU-bound.
__device__ __forceinline__ float silu_fwd(float z) {
    const float e = __builtin_amdgcn_exp2f(-z * 1.44269504088896341f);
    return z * __builtin_amdgcn_rcpf(1.0f + e);
}
__device__ __forceinline__ float dsilu(float z) {
    const float s = 1.0f / (1.0f + expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

struct RowArgs {
    const float *X;      // [n][40]
    int64_t n;
    const float *p;      // master parameters (biases are read from here)
    Wbf w;
    const float *norm;   // inference: null, or mu[40], sd[40], lo[40], hi[40]; inputs enter as (X - mu) / sd
    uint8_t *out;        // inference: null, or 1 per row with an input outside [lo, hi] (or NaN)
    float *y;            // inference: [n]
    const float *t;      // training: targets [n]
    float *part;         // training: [gridDim.x][NPART] partial gradients
};

// One dense layer for NS 16-row tiles held in LDS (row stride SIN), computed
// transposed: acc[s][nt] = W[16 nt .. 16 nt + 15] in_s^T, so that a lane's four
// results are four consecutive output features of one row (row l mod 16,
// features 16 nt + 4 (l / 16) + i) and go to LDS as one 8-byte write.  The
// reduction index is outermost, so one fragment of the input feeds NT
// independent MFMA chains and one weight fragment all NS tiles; each output
// element accumulates its K/32 products in ascending order.
template <int K, int SIN, int SW, int NT, int NS>
__device__ __forceinline__ void layer_tiles(const __bf16 *sin, const __bf16 *sw, f32x4 (&acc)[NS][NT]) {
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int s = 0; s < NS; s++)
#pragma unroll
        for (int nt = 0; nt < NT; nt++) acc[s][nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kt = 0; kt < K / 32; kt++) {
        bf16x8 x[NS];
#pragma unroll
        for (int s = 0; s < NS; s++) x[s] = *(const bf16x8 *)(sin + (s * 16 + (l & 15)) * SIN + kt * 32 + 8 * (l >> 4));
#pragma unroll
        for (int nt = 0; nt < NT; nt++) {
            const bf16x8 w = *(const bf16x8 *)(sw + (nt * 16 + (l & 15)) * SW + kt * 32 + 8 * (l >> 4));
#pragma unroll
            for (int s = 0; s < NS; s++) acc[s][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x[s], acc[s][nt], 0, 0, 0);
        }
    }
}

// Large inference batches.  FWD_WAVES wavefronts share the bfloat16 weights
// and the hidden biases in LDS; each wavefront owns FWD_SUB 16-row tiles at a
// time, which every layer overwrites in place once its products are in
// registers.  A weight fragment read from LDS feeds FWD_SUB products, which
// halves the LDS traffic per row that one tile at a time needs.  NORM applies
// the normaliser and raises the envelope flags from the values already in
// registers.  Bound by the SiLU's vector instructions (its exponential and
// reciprocal issue at a quarter of the rate: about 300 issue cycles per row and
// SIMD, 128 us at 1 048 576 rows) with the products' 36 us mostly beside them.
// Measured at 1 048 576 rows with flags: 187 us (5.6 G rows/s; 185 us on inputs
// that lie in the Infinity Cache, 188 us on inputs that do not) against 231 us
// with one tile per wavefront and twelve wavefronts, and 561 us for a separate
// pass over X for the flags.
constexpr int FWD_WAVES = 8;
constexpr int FWD_SUB = 2;

template <bool NORM>
__global__ __launch_bounds__(64 * FWD_WAVES) void k_mlp_forward(RowArgs a) {
    constexpr int NS = FWD_SUB, TR = 16 * NS;
    __shared__ __attribute__((aligned(16))) __bf16 sW1[NH * S1];
    __shared__ __attribute__((aligned(16))) __bf16 sW2[NH * SH];
    __shared__ __attribute__((aligned(16))) __bf16 sW3[NH * SH];
    __shared__ __attribute__((aligned(16))) __bf16 sAct[FWD_WAVES][TR * SH];
    __shared__ __attribute__((aligned(16))) float sBias[3 * NH];
    __shared__ f32x4 sNorm[NORM ? NIN : 1];  // mu, 1 / sd, lo, hi of an input
    __shared__ uint32_t sRows[FWD_WAVES];
    static_assert(TR <= 32, "a mask bit per row");
    const int tid = threadIdx.x, l = tid & 63, wv = tid >> 6;
    // weights -> LDS, 8 bf16 per copy
    for (int c = tid; c < NH * KIN / 8; c += blockDim.x) {
        const int r = c / (KIN / 8), k = (c % (KIN / 8)) * 8;
        *(bf16x8 *)(sW1 + r * S1 + k) = *(const bf16x8 *)(a.w.w1 + r * KIN + k);
    }
    for (int c = tid; c < NH * NH / 8; c += blockDim.x) {
        const int r = c / (NH / 8), k = (c % (NH / 8)) * 8;
        *(bf16x8 *)(sW2 + r * SH + k) = *(const bf16x8 *)(a.w.w2 + r * NH + k);
        *(bf16x8 *)(sW3 + r * SH + k) = *(const bf16x8 *)(a.w.w3 + r * NH + k);
    }
    for (int c = tid; c < 3 * NH; c += blockDim.x) {
        const int layer = c / NH, col = c % NH;
        sBias[c] = a.p[(layer == 0 ? OFF_B1 : (layer == 1 ? OFF_B2 : OFF_B3)) + col];
    }
    // the output layer's weights (padded to 16 rows) stay in registers
    bf16x8 w4f[NH / 32];
#pragma unroll
    for (int kt = 0; kt < NH / 32; kt++)
        w4f[kt] = *(const bf16x8 *)(a.w.w4 + (l & 15) * NH + kt * 32 + 8 * (l >> 4));
    const float b4 = a.p[OFF_B4];
    if (NORM)
        for (int k = tid; k < NIN; k += blockDim.x)
            sNorm[k] = f32x4{a.norm[k], 1.0f / a.norm[NIN + k], a.norm[2 * NIN + k], a.norm[3 * NIN + k]};
    __syncthreads();
    __bf16 *buf = sAct[wv];
    const int64_t ntiles = (a.n + TR - 1) / TR;
    // the rows of a tile are consecutive binary32 values of X: coalesced loads
    // issued one tile ahead
    constexpr int XL = TR * NIN / 64;
    auto load_tile = [&](int64_t t, float (&xv)[XL]) {
        const float *src = a.X + t * TR * NIN + l;
        if ((t + 1) * TR <= a.n) {
#pragma unroll
            for (int j = 0; j < XL; j++) xv[j] = src[j * 64];
        } else {
            const int64_t lim = a.n * NIN - t * TR * NIN - l;
#pragma unroll
            for (int j = 0; j < XL; j++) xv[j] = j * 64 < lim ? src[j * 64] : 0.0f;
        }
    };
    // places in the input tile of the lane's first five values; five loads on
    // is eight rows on
    int at[5];
#pragma unroll
    for (int j = 0; j < 5; j++) at[j] = (j * 64 + l) / NIN * S1 + (j * 64 + l) % NIN;
    float xv[XL];
    int64_t tile = (int64_t)blockIdx.x * FWD_WAVES + wv;
    load_tile(tile, xv);
    // this lane's row of a tile and the first of its four features
    const int lr = l & 15, lf = 4 * (l >> 4);
    for (; tile < ntiles; tile += (int64_t)gridDim.x * FWD_WAVES) {
        const int64_t r0 = tile * TR;
        // input tile: rows x 64 (40 features, zero padded), binary32 -> bfloat16;
        // bit j of `bad`: this lane's j-th value lies outside the envelope
        // (value 64 j + l is column (64 j + l) mod 40, which repeats every five j)
        uint32_t bad = 0;
#pragma unroll
        for (int c = 0; c < 5; c++) {
            f32x4 nm;
            if (NORM) nm = sNorm[(c * 64 + l) % NIN];
#pragma unroll
            for (int j = c; j < XL; j += 5) {
                float xk = xv[j];
                if (NORM) {
                    if (!(xk >= nm[2] && xk <= nm[3])) bad |= 1u << j;
                    xk = (xk - nm[0]) * nm[1];
                }
                buf[at[c] + (j / 5) * 8 * S1] = (__bf16)xk;
            }
        }
        for (int c = l; c < TR * (KIN - NIN) / 8; c += 64) {
            constexpr int PV = (KIN - NIN) / 8;
            *(bf16x8 *)(buf + (c / PV) * S1 + NIN + (c % PV) * 8) = bf16x8{};
        }
        if (NORM && a.out) {
            // bit r of the mask: row r has an input outside the envelope
            uint32_t mask = 0;
            if (__any(bad != 0)) {
                if (l == 0) sRows[wv] = 0;
                wave_sync();
                for (; bad; bad &= bad - 1) atomicOr(&sRows[wv], 1u << (((__ffs(bad) - 1) * 64 + l) / NIN));
                wave_sync();
                mask = sRows[wv];
            }
            if (l < TR && r0 + l < a.n) a.out[r0 + l] = (uint8_t)((mask >> l) & 1u);
        }
        load_tile(tile + (int64_t)gridDim.x * FWD_WAVES, xv);
        wave_sync();
        // hidden layers
#pragma unroll 1
        for (int layer = 0; layer < 3; layer++) {
            f32x4 acc[NS][NH / 16];
            if (layer == 0) layer_tiles<KIN, S1, S1, NH / 16, NS>(buf, sW1, acc);
            else layer_tiles<NH, SH, SH, NH / 16, NS>(buf, layer == 1 ? sW2 : sW3, acc);
            wave_sync();  // every lane's reads of the input tile are done
#pragma unroll
            for (int nt = 0; nt < NH / 16; nt++) {
                const int f0 = nt * 16 + lf;
                const f32x4 b = *(const f32x4 *)(sBias + layer * NH + f0);
#pragma unroll
                for (int s = 0; s < NS; s++) {
                    bf16x4 h;
#pragma unroll
                    for (int i = 0; i < 4; i++) h[i] = (__bf16)silu_fwd(acc[s][nt][i] + b[i]);
                    *(bf16x4 *)(buf + (s * 16 + lr) * SH + f0) = h;
                }
            }
            wave_sync();
        }
        // output layer: output feature 0 of row l (l < 16) is y
#pragma unroll
        for (int s = 0; s < NS; s++) {
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kt = 0; kt < NH / 32; kt++)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    w4f[kt], *(const bf16x8 *)(buf + (s * 16 + lr) * SH + kt * 32 + 8 * (l >> 4)), acc, 0, 0, 0);
            if (l < 16 && r0 + s * 16 + l < a.n) a.y[r0 + s * 16 + l] = acc[0] + b4;
        }
        wave_sync();
    }
}

// ------------------------------------------------- small batches and training
// A workgroup of eight wavefronts takes RT 16-row tiles together.  Wavefront w
// computes the output features 16 w .. 16 w + 15 of every layer for all rows,
// its weights in registers (10 fragments), so nothing is staged before the
// first product and a batch of a few thousand rows spreads over as many CUs as
// it has tiles; the activations pass between the wavefronts through LDS.  The
// products and their order are those of k_mlp_forward, so both give the same
// bits.
//
// TRAIN: the backward pass follows in the same workgroup.  A wavefront's
// pre-activations stay in its registers; dZ goes to LDS in both orders (rows
// for dH = dZ W, features for dW = dZ^T H, whose reduction runs over the
// workgroup's rows).  No activation or dZ goes to memory: a workgroup reads
// its 64 rows and the weights and writes one partial gradient (154 KB).
// 4 096 rows: 26 us with the reduction and the Adam step 6 us; one workgroup
// per CU at a time leaves the chain of layers exposed, which bounds it.  The
// same gradients from a GEMM per product, with column sums in row order by one
// workgroup, took 3 750 us over 18 launches.
constexpr int ST = 72;          // LDS row stride (bf16) of the feature-major copies (64 rows)
constexpr int GRAD_TILES = 4;   // 16-row tiles per workgroup in training
constexpr int NPART = 38464;    // values per partial: the parameters, the loss sum, padding
static_assert(NPART > NPAR, "room for the loss");

constexpr int64_t grad_groups(int64_t n) { return (n + 16 * GRAD_TILES - 1) / (16 * GRAD_TILES); }

__device__ __forceinline__ bf16x8 frag(const __bf16 *base, int row, int stride, int kt) {
    const int l = threadIdx.x & 63;
    return *(const bf16x8 *)(base + (row + (l & 15)) * stride + kt * 32 + 8 * (l >> 4));
}

template <int RT, bool TRAIN>
__global__ __launch_bounds__(512) void k_mlp_rows(RowArgs a) {
    static_assert(!TRAIN || RT == GRAD_TILES, "the weight gradients reduce over 64 rows");
    constexpr int R = 16 * RT;
    __shared__ __attribute__((aligned(16))) __bf16 sX[R * S1];
    __shared__ __attribute__((aligned(16))) __bf16 sH[TRAIN ? 3 : 2][R * SH];
    __shared__ __attribute__((aligned(16))) __bf16 sXT[TRAIN ? KIN * ST : 8];
    __shared__ __attribute__((aligned(16))) __bf16 sHT[TRAIN ? 2 : 1][TRAIN ? NH * ST : 8];
    __shared__ __attribute__((aligned(16))) __bf16 sDT[TRAIN ? NH * ST : 8];
    __shared__ float sGq[R], sSum[2][RT];
    __shared__ int sBad[R];
    const int tid = threadIdx.x, l = tid & 63, wv = tid >> 6;
    const int lr = l & 15, f0 = 16 * wv + 4 * (l >> 4);  // this lane's row of a tile, first of its features
    const int64_t r0 = (int64_t)blockIdx.x * R;
    const int rows = a.n - r0 < R ? (int)(a.n - r0) : R;
    // fragments and biases of the hidden layers, loaded beside the input rows
    bf16x8 wf[3][NH / 32];
    float b[3][4];
#pragma unroll
    for (int kt = 0; kt < NH / 32; kt++) {
        if (kt < KIN / 32) wf[0][kt] = frag(a.w.w1, 16 * wv, KIN, kt);
        wf[1][kt] = frag(a.w.w2, 16 * wv, NH, kt);
        wf[2][kt] = frag(a.w.w3, 16 * wv, NH, kt);
    }
#pragma unroll
    for (int i = 0; i < 4; i++) {
        b[0][i] = a.p[OFF_B1 + f0 + i];
        b[1][i] = a.p[OFF_B2 + f0 + i];
        b[2][i] = a.p[OFF_B3 + f0 + i];
    }
    // input rows: binary32 -> bfloat16, zero padded to 64 columns
    if (!TRAIN && a.out) {
        if (tid < R) sBad[tid] = 0;
        __syncthreads();
    }
    for (int idx = tid; idx < R * NIN; idx += 512) {
        const int r = idx / NIN, k = idx % NIN;
        float xk = r < rows ? a.X[r0 * NIN + idx] : 0.0f;
        if (!TRAIN && a.norm) {
            if (a.out && r < rows && !(xk >= a.norm[2 * NIN + k] && xk <= a.norm[3 * NIN + k])) sBad[r] = 1;
            xk = (xk - a.norm[k]) * (1.0f / a.norm[NIN + k]);
        }
        sX[r * S1 + k] = (__bf16)xk;
        if (TRAIN) sXT[k * ST + r] = (__bf16)xk;
    }
    for (int c = tid; c < R * (KIN - NIN); c += 512) {
        const int r = c / (KIN - NIN), k = NIN + c % (KIN - NIN);
        sX[r * S1 + k] = (__bf16)0.0f;
        if (TRAIN) sXT[k * ST + r] = (__bf16)0.0f;
    }
    __syncthreads();
    if (!TRAIN && a.out && tid < rows) a.out[r0 + tid] = (uint8_t)sBad[tid];
    // hidden layers
    float z[TRAIN ? 3 : 1][RT][4];
    bf16x4 h3[TRAIN ? RT : 1];
#pragma unroll
    for (int layer = 0; layer < 3; layer++) {
        __bf16 *ho = sH[TRAIN ? layer : layer & 1];
        const __bf16 *hi = layer == 0 ? sX : sH[TRAIN ? layer - 1 : (layer - 1) & 1];
#pragma unroll
        for (int rt = 0; rt < RT; rt++) {
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kt = 0; kt < (layer == 0 ? KIN : NH) / 32; kt++) {
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[layer][kt], frag(hi, rt * 16, layer == 0 ? S1 : SH, kt), acc, 0, 0, 0);
            }
            // rows beyond n hold zeros, as the reductions over rows need
            const bool in = rt * 16 + lr < rows;
            bf16x4 h;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float zi = acc[i] + b[layer][i];
                h[i] = in ? (__bf16)silu_fwd(zi) : (__bf16)0.0f;
                if (TRAIN) {
                    z[layer][rt][i] = zi;
                    if (layer == 2) h3[rt][i] = h[i];
                    else sHT[layer][(f0 + i) * ST + rt * 16 + lr] = h[i];
                }
            }
            *(bf16x4 *)(ho + (rt * 16 + lr) * SH + f0) = h;
        }
        __syncthreads();
    }
    // output layer, tile w by wavefront w (W4 padded to 16 rows): output
    // feature 0 of row l (l < 16) is y
    float gsum = 0.0f, qsum = 0.0f;
    if (wv < RT) {
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        const __bf16 *hi = sH[TRAIN ? 2 : 0];
#pragma unroll
        for (int kt = 0; kt < NH / 32; kt++)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(a.w.w4, 0, NH, kt), frag(hi, wv * 16, SH, kt), acc, 0, 0, 0);
        const int r = wv * 16 + l;
        if (l < 16) {
            const float y = acc[0] + a.p[OFF_B4];
            if (!TRAIN) {
                if (r < rows) a.y[r0 + r] = y;
            } else {
                // g = 2/n (y - t) in binary32, its bfloat16 feeds the layers below
                float g = 0.0f, q = 0.0f;
                if (r < rows) {
                    const float d = y - a.t[r0 + r];
                    g = (2.0f / (float)a.n) * d;
                    q = d * d;
                }
                sGq[r] = (float)(__bf16)g;
                gsum = g;
                qsum = q;
            }
        }
    }
    if (!TRAIN) return;
    __syncthreads();
    float *part = a.part + (int64_t)blockIdx.x * NPART;
    // sum over the 16 lanes that hold a feature's rows
    auto lane_sum = [](float v) {
#pragma unroll
        for (int d = 8; d >= 1; d >>= 1) v = v + __shfl_xor(v, d, 64);
        return v;
    };
    // dZ3 = (gq w4) silu'(z3); dZ of the lower layers = dH silu'(z), dH = dZ W
#pragma unroll
    for (int layer = 2; layer >= 0; layer--) {
        // dZ3 and dZ2 in row order take the tiles of h3 and h2, which no wavefront reads any more
        const __bf16 *up = sH[layer == 1 ? 2 : 1];
        bf16x8 wt[NH / 32];
        if (layer < 2)
#pragma unroll
            for (int kt = 0; kt < NH / 32; kt++) wt[kt] = frag(layer == 1 ? a.w.w3t : a.w.w2t, 16 * wv, NH, kt);
        float dz[RT][4], db[4] = {0.0f, 0.0f, 0.0f, 0.0f}, dw4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int rt = 0; rt < RT; rt++) {
            const bool in = rt * 16 + lr < rows;
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
            if (layer < 2)
#pragma unroll
                for (int kt = 0; kt < NH / 32; kt++)
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[kt], frag(up, rt * 16, SH, kt), acc, 0, 0, 0);
            const float gq = sGq[rt * 16 + lr];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float dh = layer == 2 ? gq * (float)a.w.w4[f0 + i] : acc[i];
                dz[rt][i] = in ? dh * dsilu(z[layer][rt][i]) : 0.0f;
                db[i] = db[i] + dz[rt][i];
                if (layer == 2) dw4[i] = dw4[i] + gq * (float)h3[rt][i];
            }
        }
        wave_sync();  // this wavefront's reads of its previous dZ^T are done
#pragma unroll
        for (int rt = 0; rt < RT; rt++) {
            bf16x4 d;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                d[i] = (__bf16)dz[rt][i];
                sDT[(f0 + i) * ST + rt * 16 + lr] = d[i];
            }
            if (layer > 0) *(bf16x4 *)(sH[layer] + (rt * 16 + lr) * SH + f0) = d;
        }
        __syncthreads();
        // dW = dZ^T H over the workgroup's rows: this wavefront's 16 features
        const __bf16 *ht = layer == 0 ? sXT : sHT[layer - 1];
        constexpr int off[3] = {OFF_W1, OFF_W2, OFF_W3}, offb[3] = {OFF_B1, OFF_B2, OFF_B3};
        const int nin = layer == 0 ? NIN : NH;
#pragma unroll
        for (int nt = 0; nt < (layer == 0 ? KIN : NH) / 16; nt++) {
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kt = 0; kt < R / 32; kt++)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(sDT, 16 * wv, ST, kt), frag(ht, nt * 16, ST, kt), acc, 0, 0, 0);
            if (nt * 16 + lr < nin)
#pragma unroll
                for (int i = 0; i < 4; i++) part[off[layer] + (f0 + i) * nin + nt * 16 + lr] = acc[i];
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float s = lane_sum(db[i]);
            if (lr == 0) part[offb[layer] + f0 + i] = s;
            if (layer == 2) {
                const float s4 = lane_sum(dw4[i]);
                if (lr == 0) part[OFF_W4 + f0 + i] = s4;
            }
        }
    }
    gsum = lane_sum(gsum);
    qsum = lane_sum(qsum);
    if (wv < RT && l == 0) {
        sSum[0][wv] = gsum;
        sSum[1][wv] = qsum;
    }
    __syncthreads();
    if (tid < 2) {
        float s = 0.0f;
        for (int k = 0; k < RT; k++) s = s + sSum[tid][k];
        part[tid == 0 ? OFF_B4 : NPAR] = s;
    }
}

struct ReduceArgs {
    const float *part;   // [groups][NPART]
    int64_t groups, n;
    float *g;            // gradient out (without the update)
    float *loss;
    float *p, *m, *v;    // masters and moments (with the update)
    Wbf w;
    float lr, c1, c2;    // rate, 1 - beta1^t, 1 - beta2^t
};

// Sum of the partial gradients in workgroup order, one thread per parameter
// (consecutive threads read consecutive values).  UPDATE: the Adam step on the
// masters and their bfloat16 copies; otherwise the gradient goes to g.
template <bool UPDATE>
__global__ __launch_bounds__(256) void k_mlp_reduce(ReduceArgs a) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i > NPAR) return;
    float g = 0.0f;
#pragma unroll 16
    for (int64_t k = 0; k < a.groups; k++) g = g + a.part[k * NPART + i];
    if (i == NPAR) {
        *a.loss = g / (float)a.n;
        return;
    }
    if (!UPDATE) {
        a.g[i] = g;
        return;
    }
    const float mi = 0.9f * a.m[i] + (1.0f - 0.9f) * g;
    const float vi = 0.999f * a.v[i] + (1.0f - 0.999f) * g * g;
    a.m[i] = mi;
    a.v[i] = vi;
    const float mh = mi / a.c1, vh = vi / a.c2;
    const float p = a.p[i] - a.lr * mh / (sqrtf(vh) + 1e-8f);
    a.p[i] = p;
    const __bf16 q = (__bf16)p;
    if (i < OFF_B1) {
        a.w.w1[(i / NIN) * KIN + i % NIN] = q;
    } else if (i >= OFF_W2 && i < OFF_B2) {
        const int j = i - OFF_W2;
        a.w.w2[j] = a.w.w2t[(j % NH) * NH + j / NH] = q;
    } else if (i >= OFF_W3 && i < OFF_B3) {
        const int j = i - OFF_W3;
        a.w.w3[j] = a.w.w3t[(j % NH) * NH + j / NH] = q;
    } else if (i >= OFF_W4 && i < OFF_B4) {
        a.w.w4[i - OFF_W4] = q;
    }
}

// Inference.  k_mlp_forward stages 88 KB of weights per workgroup, which takes
// 14 us whatever the batch up to 65 536 rows; k_mlp_rows starts at once, with
// as few tiles per workgroup as leave one workgroup per CU.  Measured (us, 1 /
// 2 / 4 tiles per workgroup / k_mlp_forward): 16 rows 5.6 / 6.5 / 7.9 / 10.2,
// 4 096 rows 6.2 / 7.3 / 9.7 / 14.2, 8 317 rows 11.6 / 10.4 / 9.8 / 14.2,
// 16 384 rows 15.8 / 10.6 / 10.0 / 14.3, 24 000 rows 20.9 / 13.9 / 14.1 / 14.3,
// 65 536 rows 57 / 36 / 24 / 14.5.
constexpr int64_t FWD_SMALL = 64 * 256;

hipError_t launch_forward(const RowArgs &a, hipStream_t s) {
    if (a.n > FWD_SMALL) {
        const int64_t tiles = (a.n + 16 * FWD_SUB - 1) / (16 * FWD_SUB);
        const dim3 g((unsigned)std::min<int64_t>((tiles + FWD_WAVES - 1) / FWD_WAVES, 256)), b(64 * FWD_WAVES);
        if (a.norm) hipLaunchKernelGGL(k_mlp_forward<true>, g, b, 0, s, a);
        else hipLaunchKernelGGL(k_mlp_forward<false>, g, b, 0, s, a);
    } else if (a.n > 2 * 16 * 256) {
        hipLaunchKernelGGL((k_mlp_rows<4, false>), dim3((unsigned)((a.n + 63) / 64)), dim3(512), 0, s, a);
    } else if (a.n > 16 * 256) {
        hipLaunchKernelGGL((k_mlp_rows<2, false>), dim3((unsigned)((a.n + 31) / 32)), dim3(512), 0, s, a);
    } else {
        hipLaunchKernelGGL((k_mlp_rows<1, false>), dim3((unsigned)((a.n + 15) / 16)), dim3(512), 0, s, a);
    }
    return hipGetLastError();
}

// binary32 masters -> padded bfloat16 copies.
__global__ void k_pack(const float *p, Wbf w) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < NH * KIN) {
        const int r = i / KIN, k = i % KIN;
        w.w1[i] = (__bf16)(k < NIN ? p[OFF_W1 + r * NIN + k] : 0.0f);
    }
    if (i < NH * NH) {
        const int t = (i % NH) * NH + i / NH;
        w.w2[i] = w.w2t[t] = (__bf16)p[OFF_W2 + i];
        w.w3[i] = w.w3t[t] = (__bf16)p[OFF_W3 + i];
    }
    if (i < 16 * NH) w.w4[i] = (__bf16)(i < NH ? p[OFF_W4 + i] : 0.0f);
}

constexpr size_t AL = 256;
constexpr size_t al(size_t v) { return (v + AL - 1) / AL * AL; }

struct Lay {
    int64_t B;  // batch capacity, multiple of 32
    size_t p, m, v, g, w1, w2, w3, w4, w2t, w3t, part, loss, norm, total;
};

// masters: whether the binary32 parameters, their gradient and the Adam
// moments live here too (a context) or stay with the caller (a bare gradient
// evaluation).
constexpr Lay layout(int64_t max_batch, bool masters = true) {
    Lay L{};
    L.B = (max_batch + 31) / 32 * 32;
    size_t o = 0;
    auto take = [&](size_t b) { size_t r = o; o = al(o + b); return r; };
    const size_t mp = masters ? (size_t)NPAR * 4 : 0;
    L.p = take(mp); L.m = take(mp); L.v = take(mp); L.g = take(mp);
    L.w1 = take(NH * KIN * 2); L.w2 = take(NH * NH * 2); L.w3 = take(NH * NH * 2); L.w4 = take(16 * NH * 2);
    L.w2t = take(NH * NH * 2); L.w3t = take(NH * NH * 2);
    L.part = take((size_t)grad_groups(L.B) * NPART * 4);
    L.loss = take(64);
    L.norm = masters ? take(4 * NIN * 4) : 0;
    L.total = o;
    return L;
}

}  // namespace

struct mlp_ctx {
    Lay L;
    char *ws;
    hipStream_t s;
    int t;
    Wbf w;
    bool have_norm;  // mlp_set_normaliser was called
};

namespace {
template <class T> T *P(mlp_ctx *c, size_t off) { return (T *)(c->ws + off); }

Wbf weights_at(char *base, const Lay &L) {
    auto at = [&](size_t off) { return (__bf16 *)(base + off); };
    return Wbf{at(L.w1), at(L.w2), at(L.w3), at(L.w4), at(L.w2t), at(L.w3t)};
}

hipError_t pack_to(const float *p, Wbf w, hipStream_t s) {
    hipLaunchKernelGGL(k_pack, dim3((NH * NH + 255) / 256), dim3(256), 0, s, p, w);
    return hipGetLastError();
}

hipError_t pack(mlp_ctx *c) { return pack_to(P<float>(c, c->L.p), c->w, c->s); }

hipError_t zero(mlp_ctx *c, size_t off, size_t bytes) {
    return lbimb::launch_fill_u32(P<uint32_t>(c, off), 0u, (int64_t)(bytes / 4), c->s);
}

// Partial gradients of the mean squared error, one per workgroup, into
// `part`; the workgroups used.  They depend on n alone, so that every caller
// sums the same partials in the same order.
hipError_t partial_grads(const float *p, const Wbf &w, const float *X, const float *y, int64_t n, float *part,
                         hipStream_t s, int64_t &groups) {
    RowArgs a{};
    a.X = X; a.t = y; a.n = n; a.p = p; a.w = w; a.part = part;
    groups = grad_groups(n);
    hipLaunchKernelGGL((k_mlp_rows<GRAD_TILES, true>), dim3((unsigned)groups), dim3(512), 0, s, a);
    return hipGetLastError();
}

// Gradient and loss from the partials, without an update.
hipError_t grads(const float *p, const Wbf &w, const float *X, const float *y, int64_t n, float *part, float *g,
                 float *loss, hipStream_t s) {
    ReduceArgs r{};
    hipError_t e = partial_grads(p, w, X, y, n, part, s, r.groups);
    if (e != hipSuccess) return e;
    r.part = part; r.n = n; r.g = g; r.loss = loss;
    hipLaunchKernelGGL(k_mlp_reduce<false>, dim3((NPAR + 256) / 256), dim3(256), 0, s, r);
    return hipGetLastError();
}

// ------------------------------------------------ allocation-free gradients
// The intermediates of mlp_gradients_noalloc: one fixed array per GPU, held
// until the process ends.  Host code never passes `scratch` itself to a kernel
// (on the host that name is only a stand-in); it passes the device address
// that hipGetSymbolAddress returns for the current GPU, looked up once per
// device and kept in scratch_ptr.
constexpr Lay NOALLOC_LAY = layout(MLP_NOALLOC_MAX_ROWS, false);
static_assert(NOALLOC_LAY.total <= MLP_NOALLOC_SCRATCH_BYTES, "scratch size in mlp_closure.h");
static __device__ __align__(256) char scratch[MLP_NOALLOC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
char *scratch_ptr[MAX_DEVICES];

// Device address of this GPU's scratch array (looked up on the first call on
// each device, with that device current).
hipError_t scratch_for_current_device(char **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr || (uintptr_t)ptr % AL) return hipErrorInvalidSymbol;
        scratch_ptr[dev] = (char *)ptr;
    }
    *out = scratch_ptr[dev];
    return hipSuccess;
}
}  // namespace

extern "C" {

int mlp_workspace_bytes(int64_t max_batch, size_t *bytes) {
    if (max_batch < 1 || !bytes) return LBM_E_INVALID;
    *bytes = layout(max_batch).total;
    return LBM_OK;
}

int mlp_create(int64_t max_batch, void *workspace, size_t ws_bytes, void *hip_stream, mlp_ctx **out) {
    if (!out || max_batch < 1) return LBM_E_INVALID;
    Lay L = layout(max_batch);
    if (!workspace || ws_bytes < L.total) return LBM_E_NOMEM;
    if ((uintptr_t)workspace % AL) return LBM_E_INVALID;
    mlp_ctx *c = new (std::nothrow) mlp_ctx();
    if (!c) return LBM_E_NOMEM;
    c->L = L;
    c->ws = (char *)workspace;
    c->s = (hipStream_t)hip_stream;
    c->t = 0;
    c->have_norm = false;
    c->w = weights_at(c->ws, L);
    if (zero(c, 0, L.total) != hipSuccess || hipStreamSynchronize(c->s) != hipSuccess) {
        delete c;
        return LBM_E_HIP;
    }
    *out = c;
    return LBM_OK;
}

void mlp_destroy(mlp_ctx *c) {
    if (!c) return;
    (void)hipStreamSynchronize(c->s);
    delete c;
}

int mlp_set_params(mlp_ctx *c, const float *params, int ptr_kind) {
    if (!c || !params) return LBM_E_INVALID;
    const hipMemcpyKind k = ptr_kind == LBM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
    if (hipMemcpyAsync(P<float>(c, c->L.p), params, NPAR * 4, k, c->s) != hipSuccess) return LBM_E_HIP;
    if (zero(c, c->L.m, NPAR * 4) != hipSuccess || zero(c, c->L.v, NPAR * 4) != hipSuccess) return LBM_E_HIP;
    c->t = 0;
    if (pack(c) != hipSuccess) return LBM_E_HIP;
    if (ptr_kind == LBM_HOST && hipStreamSynchronize(c->s) != hipSuccess) return LBM_E_HIP;
    return LBM_OK;
}

int mlp_get_params(mlp_ctx *c, float *params, int ptr_kind) {
    if (!c || !params) return LBM_E_INVALID;
    const hipMemcpyKind k = ptr_kind == LBM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice;
    if (hipMemcpyAsync(params, P<float>(c, c->L.p), NPAR * 4, k, c->s) != hipSuccess) return LBM_E_HIP;
    if (ptr_kind == LBM_HOST && hipStreamSynchronize(c->s) != hipSuccess) return LBM_E_HIP;
    return LBM_OK;
}

int mlp_forward(mlp_ctx *c, const float *X, int64_t n, float *y) {
    if (!c || !X || !y || n < 0) return LBM_E_INVALID;
    if (n == 0) return LBM_OK;
    RowArgs a{};
    a.X = X; a.n = n; a.p = P<float>(c, c->L.p); a.w = c->w; a.y = y;
    return launch_forward(a, c->s) == hipSuccess ? LBM_OK : LBM_E_HIP;
}

int mlp_set_normaliser(mlp_ctx *c, const float *mu, const float *sd, const float *lo, const float *hi,
                       int ptr_kind) {
    if (!c || !mu || !sd || !lo || !hi || (ptr_kind != LBM_HOST && ptr_kind != LBM_DEVICE)) return LBM_E_INVALID;
    if (ptr_kind == LBM_HOST)
        for (int k = 0; k < NIN; k++)
            if (!(sd[k] > 0.0f) || !std::isfinite(sd[k]) || !std::isfinite(mu[k])) return LBM_E_INVALID;
    const hipMemcpyKind kind = ptr_kind == LBM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
    const float *src[4] = {mu, sd, lo, hi};
    for (int j = 0; j < 4; j++)
        if (hipMemcpyAsync(P<float>(c, c->L.norm) + j * NIN, src[j], NIN * 4, kind, c->s) != hipSuccess)
            return LBM_E_HIP;
    if (ptr_kind == LBM_HOST && hipStreamSynchronize(c->s) != hipSuccess) return LBM_E_HIP;
    c->have_norm = true;
    return LBM_OK;
}

int mlp_infer(mlp_ctx *c, const float *X, int64_t n, float *y, uint8_t *out_of_envelope) {
    if (!c || !X || !y || n < 0) return LBM_E_INVALID;
    if (!c->have_norm) return LBM_E_STATE;
    if (n == 0) return LBM_OK;
    const float *nb = P<float>(c, c->L.norm);
    RowArgs a{};
    a.X = X; a.n = n; a.p = P<float>(c, c->L.p); a.w = c->w; a.y = y;
    a.norm = nb; a.out = out_of_envelope;
    return launch_forward(a, c->s) == hipSuccess ? LBM_OK : LBM_E_HIP;
}

int mlp_gradients(mlp_ctx *c, const float *X, const float *y, int64_t n, float *out_grads, float *loss,
                  int ptr_kind) {
    if (!c || !X || !y || n < 1 || n > c->L.B) return LBM_E_INVALID;
    if (grads(P<float>(c, c->L.p), c->w, X, y, n, P<float>(c, c->L.part), P<float>(c, c->L.g),
              P<float>(c, c->L.loss), c->s) != hipSuccess)
        return LBM_E_HIP;
    const hipMemcpyKind k = ptr_kind == LBM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice;
    if (out_grads && hipMemcpyAsync(out_grads, P<float>(c, c->L.g), NPAR * 4, k, c->s) != hipSuccess) return LBM_E_HIP;
    if (loss && hipMemcpyAsync(loss, P<float>(c, c->L.loss), 4, k, c->s) != hipSuccess) return LBM_E_HIP;
    if (ptr_kind == LBM_HOST && hipStreamSynchronize(c->s) != hipSuccess) return LBM_E_HIP;
    return LBM_OK;
}

int mlp_train_step(mlp_ctx *c, const float *X, const float *y, int64_t n, float lr, float *loss) {
    if (!c || !X || !y || n < 1 || n > c->L.B) return LBM_E_INVALID;
    ReduceArgs r{};
    if (partial_grads(P<float>(c, c->L.p), c->w, X, y, n, P<float>(c, c->L.part), c->s, r.groups) != hipSuccess)
        return LBM_E_HIP;
    c->t += 1;
    r.part = P<float>(c, c->L.part); r.n = n; r.loss = P<float>(c, c->L.loss);
    r.p = P<float>(c, c->L.p); r.m = P<float>(c, c->L.m); r.v = P<float>(c, c->L.v); r.w = c->w; r.lr = lr;
    r.c1 = 1.0f - powf(0.9f, (float)c->t);
    r.c2 = 1.0f - powf(0.999f, (float)c->t);
    hipLaunchKernelGGL(k_mlp_reduce<true>, dim3((NPAR + 256) / 256), dim3(256), 0, c->s, r);
    if (hipGetLastError() != hipSuccess) return LBM_E_HIP;
    if (loss) {
        if (hipMemcpyAsync(loss, P<float>(c, c->L.loss), 4, hipMemcpyDeviceToHost, c->s) != hipSuccess) return LBM_E_HIP;
        if (hipStreamSynchronize(c->s) != hipSuccess) return LBM_E_HIP;
    }
    return LBM_OK;
}

int mlp_gradients_noalloc(const float *params, const float *X, const float *y, int64_t n, float *grads_out,
                          float *loss, void *hip_stream) {
    if (!params || !X || !y || !grads_out) return LBM_E_INVALID;
    if (n < 1 || n > MLP_NOALLOC_MAX_ROWS) return LBM_E_INVALID;
    char *base = nullptr;
    if (scratch_for_current_device(&base) != hipSuccess) return LBM_E_HIP;
    const Lay &L = NOALLOC_LAY;
    const hipStream_t s = (hipStream_t)hip_stream;
    const Wbf w = weights_at(base, L);
    if (pack_to(params, w, s) != hipSuccess) return LBM_E_HIP;
    if (grads(params, w, X, y, n, (float *)(base + L.part), grads_out, loss ? loss : (float *)(base + L.loss), s) !=
        hipSuccess)
        return LBM_E_HIP;
    return LBM_OK;
}

}  // extern "C"
