// Per-point warm-start MLP on gfx950: 5 -> 128 -> 128 -> 128 -> 4, GELU (erf
// form) on the hidden layers, bfloat16 weights/activations with fp32
// accumulation, Adam on fp32 master weights.
//
// Every product of bf16 operands runs on the matrix cores
// (v_mfma_f32_16x16x32_bf16): one wavefront computes one 16 x 16 output tile,
// K is walked 32 at a time.  Operand registers: lane l holds row (A) or column
// (B) l % 16 and the eight K entries of group g = l / 16; the accumulator lane
// l holds column l % 16 of rows 4 g .. 4 g + 3.
//
// Layers are evaluated transposed, Z^T = W H^T: units along the matrix rows,
// data rows along its columns.  A lane then holds units 16 c + 4 g + 0..3 of
// data row l % 16 for every 16-unit tile c, and the next layer's B operand (units
// 32 s + 8 g + 0..7 of the same row) is one exchange between the four lanes of a
// row.  Weights are kept operand by operand (64 lanes x 16 bytes, "fragments").
//
// Quantisation points (shared with the float64 reference of the tests):
// bf16 copies of W1..W4, of the input features and of each hidden activation;
// the backward pass rounds the pre-activation gradients of layers 3 and 2 to
// bf16 before their products; everything else is fp32.  What is rounded is
// computed in one order everywhere (K ascending from zero, then the bias; layer
// 1 and the gradient of layer 4 term by term), because one activation rounded
// the other way moves a row's outputs by up to a percent.
#include "lskum_mlp.h"

#include <cmath>

namespace lskum {
namespace mlp {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

constexpr float kInvSqrt2 = 0.70710678118654752f;
constexpr float kInvSqrt2Pi = 0.39894228040143268f;

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * kInvSqrt2)); }
__device__ __forceinline__ float gelu_prime(float z) {
    return 0.5f * (1.0f + erff(z * kInvSqrt2)) + z * expf(-0.5f * z * z) * kInvSqrt2Pi;
}

typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;

// Phi(-a) for a >= 0 (the normal CDF's lower half) as 2^P(a), P a degree-10
// fit of log2 Phi(-a) on [0, 6] (gen_lskum_gelu.py), minimax in the error of
// Phi(-a); beyond 6, P falls on and 2^P is below 1e-9.  (Degree 9 turns upwards there.)
__device__ __forceinline__ float phi_lower(float a) {
    float p = -6.841560207e-08f;
    p = fmaf(p, a, 1.628766199e-06f);
    p = fmaf(p, a, -1.707519550e-05f);
    p = fmaf(p, a, 1.021452845e-04f);
    p = fmaf(p, a, -3.417893604e-04f);
    p = fmaf(p, a, 8.748981782e-05f);
    p = fmaf(p, a, 6.877615582e-03f);
    p = fmaf(p, a, -5.241313577e-02f);
    p = fmaf(p, a, -4.592256248e-01f);
    p = fmaf(p, a, -1.151103973e+00f);
    p = fmaf(p, a, -1.000000000e+00f);
    return __builtin_amdgcn_exp2f(p);
}

// bf16(gelu(z)) of four values, mostly without erff but with its bits:
// max(z, 0) - |z| Phi(-|z|) is within 1.8e-7 |z| of gelu(z) (with the fit above, and
// erff and 2^P rounded correctly, at most 1.48e-7 |z| over the floats), so where both
// ends of that interval round to the same bf16, gelu(z) does too; every float from
// 1e-30 to 1e30 gives erff's bits.  Elsewhere (one value in 10,000 at z = 1, in 300 at
// z = -2, all below -5 or so) the lane takes gelu itself.  So does the whole wave
// where no |z| exceeds kNear, since there erff is the quicker one (1,000,003 rows: 221
// against 257 us; with inputs that spread z beyond, 297 against 260 us), and
// where one exceeds kFar: some lane's fit would settle nothing, and the wave pay for
// both (1,000,003 rows, weights and inputs three times the initial ones: 512 us, with
// this rule 378, with erff throughout 372).  Infinities are beyond kFar, and NaNs
// pass through Phi.  (Zeros may differ in sign.  A median in place of the maximum
// with zero: that function would first bring its operand to a canonical form.)
__device__ __forceinline__ bf16x4 gelu_bf16(const f32x4& z) {
    constexpr float kDiff = 1.8e-7f, kNear = 1.4f, kFar = 4.0f;
    bf16x4 up, down;
    const float far = fmaxf(fmaxf(fabsf(z[0]), fabsf(z[1])), fmaxf(fabsf(z[2]), fabsf(z[3])));
    bool exact = true;
    if (__any(far > kNear) && !__any(far > kFar)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float relu = __builtin_amdgcn_fmed3f(z[k], 0.0f, __builtin_inff());
            const float a = fabsf(z[k]);
            const float v = fmaf(-a, phi_lower(a), relu);
            up[k] = (__bf16)fmaf(kDiff, a, v);
            down[k] = (__bf16)fmaf(-kDiff, a, v);
        }
        exact = __builtin_bit_cast(uint64_t, up) != __builtin_bit_cast(uint64_t, down);
    }
    if (exact)
#pragma unroll
        for (int k = 0; k < 4; ++k) up[k] = (__bf16)gelu(z[k]);
    return up;
}

// Place of W[row][k] (a 128 x 128 matrix used as A operand, contraction over
// k) in its fragments: tile row / 16, K block k / 32, lane, place.
__device__ __forceinline__ int fragment(int row, int k) {
    return ((row / 16 * 4 + k / 32) * 64 + k % 32 / 8 * 16 + row % 16) * 8 + k % 8;
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// W fragments (c, s) times the four K blocks of a B operand, onto z.
__device__ __forceinline__ f32x4 row_tile(const __bf16* frag, int c, int l, const bf16x8 h[4],
                                          f32x4 z) {
#pragma unroll
    for (int s = 0; s < 4; ++s) z = mfma(*(const bf16x8*)&frag[((c * 4 + s) * 64 + l) * 8], h[s], z);
    return z;
}

// A row's features, rounded.
__device__ __forceinline__ void load_row(const float* __restrict__ X, float x[kIn]) {
#pragma unroll
    for (int f = 0; f < kIn; ++f) x[f] = (float)(__bf16)X[f];
}

// Layer 1 for one unit, w its weights and bias.
__device__ __forceinline__ float layer1(const float w[8], const float x[kIn]) {
    float z = w[kIn];
#pragma unroll
    for (int f = 0; f < kIn; ++f) z = fmaf(x[f], w[f], z);
    return z;
}

// The accumulator tiles c = 2 s, 2 s + 1 of a row, as bf16, to K block s of the
// next layer's B operand: of the row's four lanes, g receives what lanes
// 2 (g % 2) and 2 (g % 2) + 1 hold of tile 2 s + g / 2.
__device__ __forceinline__ bf16x8 to_operand(bf16x4 even, bf16x4 odd) {
    typedef __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned u32x2;
    typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
    const u32x2 e = __builtin_bit_cast(u32x2, even), o = __builtin_bit_cast(u32x2, odd);
    u32x4 h;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const auto a = __builtin_amdgcn_permlane32_swap(e[q], o[q], false, false);
        const auto b = __builtin_amdgcn_permlane16_swap(a[0], a[1], false, false);
        h[q] = b[0];
        h[2 + q] = b[1];
    }
    return __builtin_bit_cast(bf16x8, h);
}

// Whole forward pass: W2 and W3 in LDS as fragments (a wave's 1 KiB operand
// reads are then linear), blocks of eight waves walking over the rows 16 at a
// time per wave; the four outputs, padded to one tile, run on the matrix cores
// too.  Layer 1 is evaluated in the operand's own order, its weights as fp32 rows
// in LDS (one address for 16 lanes).
// Bound by the vector instructions of GELU (384 a row): 1,000,003 rows take 260
// us with the call, 370 with activations passed through LDS between layers, one
// weight buffer for both layers and layer 4 on the vector units.  Layers unrolled
// (twice the code), other occupancy, two tiles a wave: the same to 5% more.
constexpr int kFwdWaves = 8;

__global__ void __launch_bounds__(64 * kFwdWaves, 4) k_mlp_forward(
    int M, const float* __restrict__ X, const float* __restrict__ W1f,
    const __bf16* __restrict__ W2f, const float* __restrict__ b2,
    const __bf16* __restrict__ W3f, const float* __restrict__ b3, const __bf16* __restrict__ W4f,
    const float* __restrict__ b4, float* __restrict__ Y) {
    __shared__ __attribute__((aligned(16))) __bf16 sW[2][kWidth * kWidth];
    __shared__ __attribute__((aligned(16))) __bf16 sW4[kW4Frag];
    __shared__ __attribute__((aligned(16))) float sW1[kWidth][8], sB[2][kWidth];
    auto stage = [](__bf16* dst, const __bf16* __restrict__ src, int n) {  // 16-byte chunks
        for (int k = 8 * threadIdx.x; k < n; k += 8 * 64 * kFwdWaves)
            *(bf16x8*)&dst[k] = *(const bf16x8*)&src[k];
    };
    stage(sW[0], W2f, kWidth * kWidth);
    stage(sW[1], W3f, kWidth * kWidth);
    stage(sW4, W4f, kW4Frag);
    for (int k = threadIdx.x; k < kWidth * 8; k += 64 * kFwdWaves) (&sW1[0][0])[k] = W1f[k];
    for (int k = threadIdx.x; k < kWidth; k += 64 * kFwdWaves) {
        sB[0][k] = b2[k];
        sB[1][k] = b3[k];
    }
    __syncthreads();
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, r = l & 15, g = l >> 4;
    const f32x4 out0 = g == 0 ? f32x4{b4[0], b4[1], b4[2], b4[3]} : f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t row0 = ((int64_t)blockIdx.x * kFwdWaves + w) * 16; row0 < M;
         row0 += (int64_t)gridDim.x * kFwdWaves * 16) {
        const int64_t m = row0 + r;
        // an opaque zero in the LDS addresses: the weights' operands are read
        // where they are used, not all held in registers across the row loop
        int at = 0;
        asm volatile("" : "+v"(at));
        bf16x8 h[4];
        // ---- layer 1, in the operand's order
        float x[kIn];
        load_row(X + (m < M ? m : 0) * kIn, x);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                f32x4 z;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    z[k] = layer1(&sW1[0][0] + at + (32 * s + 8 * g + 4 * j + k) * 8, x);
                const bf16x4 v = gelu_bf16(z);
#pragma unroll
                for (int k = 0; k < 4; ++k) h[s][4 * j + k] = v[k];
            }
#pragma unroll 1
        for (int n = 0; n < 2; ++n) {
            bf16x8 hn[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                bf16x4 v[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int c = 2 * s + i;
                    const f32x4 bias = *(const f32x4*)&sB[n][at + 16 * c + 4 * g];
                    const f32x4 z = row_tile(sW[n] + at, c, l, h, f32x4{0.f, 0.f, 0.f, 0.f});
                    v[i] = gelu_bf16(z + bias);
                }
                hn[s] = to_operand(v[0], v[1]);
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) h[s] = hn[s];
        }
        // ---- layer 4: outputs 0..3 of a row are the accumulators of its lane g = 0
        const f32x4 y = row_tile(sW4 + at, 0, l, h, out0);
        if (g == 0 && m < M) {
            float* o = Y + m * kOut;  // the caller's pointer: four-byte alignment
            o[0] = y[0];
            o[1] = y[1];
            o[2] = y[2];
            o[3] = y[3];
        }
    }
}

__device__ __forceinline__ uint64_t splitmix64(uint64_t z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// The rows of a training pass: row r of a given array, or of a data set of n
// rows the row floor(h n / 2^64), h the splitmix64 hash of seed + step batch + r.
struct Rows {
    const float* X;
    const float* T;
    int64_t n;  // 0: the arrays hold the rows themselves
    uint64_t first;  // seed + step * batch
};
__device__ __forceinline__ int64_t data_row(const Rows& R, int64_t r) {
    return R.n ? (int64_t)__umul64hi(splitmix64(R.first + (uint64_t)r), (uint64_t)R.n) : r;
}

// Forward and backward of kTrainRows rows a turn in one block, blocks walking
// over the rows: loss and the gradient's partial sums over the block's rows,
// part[block][parameter].  Wave w takes the 16 units of tile w of every layer
// and all rows of the turn, so that a block reads each weight fragment once.
// Activations and pre-activation gradients pass from layer to layer as operand
// fragments in LDS (two buffers in turn, one barrier a layer) and are kept as
// [unit][row] for the products over rows at the end;
// GELU' of the three layers stays in registers.  The 128 x 128 weight gradients
// accumulate in registers over the block's turns, one row of 16 x 16 tiles a
// wave and matrix; the sums that have fp32 factors (W1, W4, biases) run on the
// vector units, four threads a unit.
// Bound by the path of one wave: 30 KB of code met once, eight barriers, 24
// GELU evaluations a lane.  A training step of 8,192 rows (one turn, a block on
// every CU) takes 32 us, 9 of them for the 35 MB of partial sums; with a launch
// for each product and sum it took 103 us.  64 rows a turn (half the partial sums,
// half of the CUs): 5 us more.
constexpr int kTrainRows = 32;
constexpr int kTrainThreads = 512;
constexpr int kLdB = kTrainRows + 8;  // row strides: 16-byte reads of neighbouring units fall in
constexpr int kLdF = kTrainRows + 4;  // distinct banks

struct TrainLds {
    __bf16 H[3][kWidth * kLdB];
    __bf16 dZ[2][kWidth * kLdB];  // layers 3, 2
    union {
        __bf16 pass[2][kTrainRows * kWidth];  // fragments between layers
        float dZ1[kWidth * kLdF];             // then layer 1's gradient
        float col[3][12][kWidth];             // at the end: sums of the unit's other threads
    };
    float x[kTrainRows][8];
    float dY[kTrainRows][kOut];
    float W1[kWidth][8], W4[kWidth][kOut], B[2][kWidth];
    double loss[kTrainRows];
};
static_assert(sizeof(TrainLds) <= 160 * 1024, "the LDS of a CU");

__global__ void __launch_bounds__(kTrainThreads, 2) k_mlp_train(
    int Mvalid, Rows R, const float* __restrict__ W1f, const __bf16* __restrict__ W2f, const float* __restrict__ b2, const __bf16* __restrict__ W3f,
    const float* __restrict__ b3, const __bf16* __restrict__ W4f, const float* __restrict__ b4,
    const __bf16* __restrict__ W2t, const __bf16* __restrict__ W3t, float* __restrict__ part,
    double* __restrict__ loss_part) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    TrainLds& L = *reinterpret_cast<TrainLds*>(lds_raw);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int k = threadIdx.x; k < kWidth; k += kTrainThreads) {
        L.B[0][k] = b2[k];
        L.B[1][k] = b3[k];
    }
    for (int k = threadIdx.x; k < kWidth * 8; k += kTrainThreads) (&L.W1[0][0])[k] = W1f[k];
    for (int k = threadIdx.x; k < kWidth * kOut; k += kTrainThreads)
        L.W4[k / kOut][k % kOut] = (float)W4f[fragment(k % kOut, k / kOut)];
    __syncthreads();
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 dW[2][8];  // layers 3, 2: tiles (w, c)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int c = 0; c < 8; ++c) dW[n][c] = zero;
    float col[12];  // per unit: W4 (4), b3, b2, W1 (5), b1
#pragma unroll
    for (int k = 0; k < 12; ++k) col[k] = 0.0f;
    f32x4 db4 = zero;  // and the loss: of the rows whose outputs the thread sums
    double loss = 0.0;
    const f32x4 bias4 = {b4[0], b4[1], b4[2], b4[3]};
    const int part_u = w >> 1;  // sums over rows: unit threadIdx.x % 128, a quarter of the rows
    for (int64_t row0 = (int64_t)blockIdx.x * kTrainRows; row0 < Mvalid;
         row0 += (int64_t)gridDim.x * kTrainRows) {
        // Nothing that depends on the lane is computed once for all turns: the
        // many LDS addresses would fill the registers.
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int l = lane, r = l & 15, g = l >> 4, u = 64 * (w & 1) + l;
        // Operands of one layer, read a layer ahead of their use: the opaque zero
        // in their addresses keeps them from being read all at once, or once for
        // all rows, which the registers have no room for.
        int at = 0;
        bf16x8 wf[4];
        auto ahead = [&](const __bf16* __restrict__ W) {
            asm volatile("" : "+v"(at));
#pragma unroll
            for (int s = 0; s < 4; ++s) wf[s] = *(const bf16x8*)&W[at + ((4 * w + s) * 64 + l) * 8];
        };
        // Rows beyond the last are zeros (they read row 0): their gradient is zero, but
        // zero times the infinities that a row of the data may give is not.
        float x[2][kIn];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int64_t m = row0 + 16 * t + r;
            load_row(R.X + (m < Mvalid ? data_row(R, m) : 0) * kIn, x[t]);
            if (m >= Mvalid)
#pragma unroll
                for (int f = 0; f < kIn; ++f) x[t][f] = 0.0f;
            if (w == 0 && g == 0)
#pragma unroll
                for (int f = 0; f < kIn; ++f) L.x[16 * t + r][f] = x[t][f];
        }
        // the row whose outputs this thread sums over units u % 16 == r
        const int my = 4 * w + g;
        const bool valid = row0 + my < Mvalid;
        const float* target = R.T + (valid ? data_row(R, row0 + my) : 0) * kOut;
        f32x4 t4;
#pragma unroll
        for (int o = 0; o < kOut; ++o) t4[o] = target[o];
        bf16x8 h[2][4];
        // values v of units 16 w + 4 g + 0..3, row 16 t + r
        auto keep = [&](__bf16* rows, __bf16* pass, int t, bf16x4 v) {
#pragma unroll
            for (int k = 0; k < 4; ++k) rows[(16 * w + 4 * g + k) * kLdB + 16 * t + r] = v[k];
            *(bf16x4*)&pass[((4 * t + (w >> 1)) * 64 + (2 * (w & 1) + (g >> 1)) * 16 + r) * 8 + 4 * (g & 1)] = v;
        };
        auto take = [&](const __bf16* pass) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    h[t][s] = *(const bf16x8*)&pass[((4 * t + s) * 64 + l) * 8];
        };
        auto product = [&](int t) {
            f32x4 z = zero;
#pragma unroll
            for (int s = 0; s < 4; ++s) z = mfma(wf[s], h[t][s], z);
            return z;
        };
        f32x4 gp[3][2];
        // ---- forward, keeping GELU'
        auto activate = [&](int n, int t, const f32x4& z) {
            bf16x4 v;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = (__bf16)gelu(z[k]);
                gp[n][t][k] = gelu_prime(z[k]);
            }
            keep(L.H[n], L.pass[n % 2], t, v);
        };
        ahead(W2f);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x4 z;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                z[k] = layer1(&L.W1[0][0] + at + (16 * w + 4 * g + k) * 8, x[t]);
            activate(0, t, z);
        }
        __syncthreads();
#pragma unroll
        for (int n = 1; n < 3; ++n) {
            take(L.pass[n - 1]);
            f32x4 z[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
                z[t] = product(t) + *(const f32x4*)&L.B[n - 1][at + 16 * w + 4 * g];
            ahead(n == 1 ? W3f : W3t);
#pragma unroll
            for (int t = 0; t < 2; ++t) activate(n, t, z[t]);
            __syncthreads();
        }
        // ---- outputs, loss and its gradient: 16 threads a row, eight units each
        f32x4 y = zero;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const float h3 = (float)L.H[2][(16 * c + r) * kLdB + my];
            const f32x4 w4 = *(const f32x4*)L.W4[at + 16 * c + r];
#pragma unroll
            for (int o = 0; o < kOut; ++o) y[o] = fmaf(h3, w4[o], y[o]);
        }
#pragma unroll
        for (int step = 8; step > 0; step >>= 1)
#pragma unroll
            for (int o = 0; o < kOut; ++o) y[o] += __shfl_xor(y[o], step, 64);
        if (r == 0) {
            f32x4 e;
#pragma unroll
            for (int o = 0; o < kOut; ++o) {
                const float d = valid ? y[o] + bias4[o] - t4[o] : 0.0f;
                loss += (double)(d * d);
                e[o] = 2.0f * d / (4.0f * (float)Mvalid);
                db4[o] += e[o];
            }
            *(f32x4*)L.dY[my] = e;
        }
        __syncthreads();
        // ---- dZ3 = bf16((dY W4) GELU'), then down through W3 and W2
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const f32x4 dy = *(const f32x4*)L.dY[16 * t + r];
            bf16x4 v;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const f32x4 w4 = *(const f32x4*)L.W4[at + 16 * w + 4 * g + k];
                float s = 0.0f;
#pragma unroll
                for (int o = 0; o < kOut; ++o) s = fmaf(dy[o], w4[o], s);
                v[k] = (__bf16)(s * gp[2][t][k]);
            }
            keep(L.dZ[0], L.pass[1], t, v);
        }
        __syncthreads();
        take(L.pass[1]);
        f32x4 d[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) d[t] = product(t);
        ahead(W2t);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            bf16x4 v;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = (__bf16)(d[t][k] * gp[1][t][k]);
            keep(L.dZ[1], L.pass[0], t, v);
        }
        __syncthreads();
        take(L.pass[0]);
        __syncthreads();  // dZ1 takes the place of the fragments
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            d[t] = product(t);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                L.dZ1[(16 * w + 4 * g + k) * kLdF + 16 * t + r] = d[t][k] * gp[0][t][k];
        }
        __syncthreads();
        // ---- weight gradients over the block's rows: dZ^T H, K = rows
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const bf16x8 a = *(const bf16x8*)&L.dZ[n][(16 * w + r) * kLdB + 8 * g];
#pragma unroll
            for (int c = 0; c < 8; ++c)
                dW[n][c] = mfma(a, *(const bf16x8*)&L.H[1 - n][(16 * c + r) * kLdB + 8 * g], dW[n][c]);
        }
        // ---- sums over rows with fp32 factors: unit u, a quarter of the rows
        {
            const int m0 = part_u * 8;
            const bf16x8 h3 = *(const bf16x8*)&L.H[2][u * kLdB + m0];
            const bf16x8 z3 = *(const bf16x8*)&L.dZ[0][u * kLdB + m0];
            const bf16x8 z2 = *(const bf16x8*)&L.dZ[1][u * kLdB + m0];
            const f32x4 za = *(const f32x4*)&L.dZ1[u * kLdF + m0];
            const f32x4 zb = *(const f32x4*)&L.dZ1[u * kLdF + m0 + 4];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const f32x4 d = *(const f32x4*)L.dY[m0 + k];
                const f32x4 xa = *(const f32x4*)L.x[m0 + k];
                const float x4 = L.x[m0 + k][4], z1 = k < 4 ? za[k % 4] : zb[k % 4];
#pragma unroll
                for (int o = 0; o < kOut; ++o) col[o] += d[o] * (float)h3[k];
                col[4] += (float)z3[k];
                col[5] += (float)z2[k];
#pragma unroll
                for (int f = 0; f < 4; ++f) col[6 + f] += z1 * xa[f];
                col[10] += z1 * x4;
                col[11] += z1;
            }
        }
        __syncthreads();
    }
    // ---- the block's partial sums
    const int l = threadIdx.x & 63, r = l & 15, g = l >> 4, u = threadIdx.x & (kWidth - 1);
    float* P = part + (int64_t)blockIdx.x * kParams;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                P[(n == 0 ? kOffW3 : kOffW2) + (16 * w + 4 * g + k) * kWidth + 16 * c + r] =
                    dW[n][c][k];
    if (part_u > 0)
#pragma unroll
        for (int k = 0; k < 12; ++k) L.col[part_u - 1][k][u] = col[k];
    if (r == 0) {
        L.loss[4 * w + g] = loss;
        *(f32x4*)L.dY[4 * w + g] = db4;
    }
    __syncthreads();
    if (part_u == 0) {
#pragma unroll
        for (int k = 0; k < 12; ++k) col[k] += (L.col[0][k][u] + L.col[1][k][u]) + L.col[2][k][u];
#pragma unroll
        for (int o = 0; o < kOut; ++o) P[kOffW4 + o * kWidth + u] = col[o];
        P[kOffB3 + u] = col[4];
        P[kOffB2 + u] = col[5];
#pragma unroll
        for (int f = 0; f < kIn; ++f) P[kOffW1 + u * kIn + f] = col[6 + f];
        P[kOffB1 + u] = col[11];
    }
    if (threadIdx.x < kOut) {
        float s = 0.0f;
        for (int m = 0; m < kTrainRows; ++m) s += L.dY[m][threadIdx.x];
        P[kOffB4 + threadIdx.x] = s;
    }
    if (threadIdx.x == 64) {
        double s = 0.0;
        for (int m = 0; m < kTrainRows; ++m) s += L.loss[m];
        loss_part[blockIdx.x] = s;
    }
}

// The bf16 copies of parameter k with value t that the kernels read: weights
// as operand fragments, W2 and W3 in both orientations.
__device__ __forceinline__ void store_copies(int k, float t, const WeightCopies& C) {
    const __bf16 q = (__bf16)t;
    if (k >= kOffW1 && k < kOffW1 + kWidth * kIn) {
        const int row = (k - kOffW1) / kIn, f = (k - kOffW1) % kIn;
        C.W1f[row * 8 + f] = (float)q;
    } else if (k >= kOffB1 && k < kOffB1 + kWidth) {
        C.W1f[(k - kOffB1) * 8 + kIn] = t;
    } else if (k >= kOffW2 && k < kOffW2 + kWidth * kWidth) {
        const int o = (k - kOffW2) / kWidth, i = (k - kOffW2) % kWidth;
        C.W2f[fragment(o, i)] = q;
        C.W2t[fragment(i, o)] = q;
    } else if (k >= kOffW3 && k < kOffW3 + kWidth * kWidth) {
        const int o = (k - kOffW3) / kWidth, i = (k - kOffW3) % kWidth;
        C.W3f[fragment(o, i)] = q;
        C.W3t[fragment(i, o)] = q;
    } else if (k >= kOffW4 && k < kOffW4 + kOut * kWidth) {
        const int o = (k - kOffW4) / kWidth, i = (k - kOffW4) % kWidth;
        C.W4f[fragment(o, i)] = q;
    }
}

__global__ void __launch_bounds__(256) k_refresh(const float* __restrict__ theta, WeightCopies C) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < kParams) store_copies(k, theta[k], C);
}

// Adam (fp32): m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2,
// theta -= lr * (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps).
struct Adam {
    float lr, b1, b2, eps, c1, c2;
    float* m;
    float* v;
    float* theta;
};

// The gradient from the blocks' partial sums: block b covers parameters
// [64 b, 64 b + 64) with four thread groups, group g adding parts g, g + 4, ...
// in order, the four group sums in group order (fixed throughout; in double
// precision, rounded once: 8,192 rows are 256 parts, and in fp32 their sum was off
// by 7e-8, with the same time); the last block adds the loss.  Into grad (may be
// NULL), and with STEP into an Adam step of the parameters and their copies.
template <bool STEP>
__global__ void __launch_bounds__(256) k_grad_sum(int nparts, const float* __restrict__ part,
                                                  const double* __restrict__ loss_part,
                                                  float* __restrict__ grad,
                                                  double* __restrict__ loss, Adam A,
                                                  WeightCopies C) {
    __shared__ double group[4][64];
    const int j = threadIdx.x & 63, g = threadIdx.x >> 6;
    if (blockIdx.x == gridDim.x - 1) {
        if (g != 0) return;
        double t = 0.0;
        for (int b = j; b < nparts; b += 64) t += loss_part[b];
        for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
        if (j == 0) loss[0] = t;
        return;
    }
    const int k = blockIdx.x * 64 + j;
    double s = 0.0;
    if (k < kParams)
#pragma unroll 8
        for (int b = g; b < nparts; b += 4) s += part[(int64_t)b * kParams + k];
    group[g][j] = s;
    __syncthreads();
    if (g != 0 || k >= kParams) return;
    const float gk = (float)(((group[0][j] + group[1][j]) + group[2][j]) + group[3][j]);
    if (grad) grad[k] = gk;
    if (STEP) {
        const float mk = A.b1 * A.m[k] + (1.0f - A.b1) * gk;
        const float vk = A.b2 * A.v[k] + (1.0f - A.b2) * gk * gk;
        A.m[k] = mk;
        A.v[k] = vk;
        const float t = A.theta[k] - A.lr * (mk / A.c1) / (sqrtf(vk / A.c2) + A.eps);
        A.theta[k] = t;
        store_copies(k, t, C);
    }
}

// Squared distance from c to the nearest wall point, by runs of kWallRun wall
// points (consecutive along the contour, so a run is compact).  The wavefront's
// points share a bounding box.  Lane j bounds the distances between the box and
// run j from both sides; the smallest upper bound rules out most runs at once,
// its run is searched first, and of the others those that the box and then the
// lane's own best point do not rule out.  Bounds are moved apart by far more than
// their rounding, so no point that could be the nearest is passed over.  Runs,
// boxes and points to search are read at wave-uniform addresses (scalar loads).
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) f64x2 ConstD2;  // read by scalar loads
typedef const __attribute__((address_space(4))) f64x4 ConstD4;
typedef const __attribute__((address_space(4))) int32_t ConstI32;

// A wave-uniform value kept apart from the per-lane value it was compared
// with: in a branch on their equality the compiler takes one for the other,
// and addresses formed from it are no longer uniform.
__device__ __forceinline__ int uniform(int v) {
    asm volatile("" : "+s"(v));
    return v;
}

__device__ __forceinline__ double box_bound(f64x4 b, const D2& c) {
    const double dx = fmax(fmax(b.x - c.x, c.x - b.y), 0.0);
    const double dy = fmax(fmax(b.z - c.y, c.y - b.w), 0.0);
    return (dx * dx + dy * dy) * (1.0 - 1e-12);
}

__device__ __forceinline__ double run_min(double d2, int r, ConstD2* wall_xy,
                                          const D2& c) {
#pragma unroll 16
    for (int w = 0; w < kWallRun; ++w) {
        const f64x2 q = wall_xy[(int64_t)r * kWallRun + w];
        const double dx = c.x - q.x, dy = c.y - q.y;
        d2 = fmin(d2, dx * dx + dy * dy);
    }
    return d2;
}

// Smallest (largest) value of the wavefront in fp32, rounded down (up).
template <bool MAX>
__device__ __forceinline__ float wave_extreme(double x) {
    float v = MAX ? __double2float_ru(x) : __double2float_rd(x);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float w = __shfl_xor(v, o, 64);
        v = MAX ? fmaxf(v, w) : fminf(v, w);
    }
    return v;
}

// Called by whole wavefronts; `mine` lanes ask, runs r0 .. r1 - 1.
__device__ __forceinline__ double nearest_wall(bool mine, int r0, int r1, const D2& c,
                                               const D4* wall_box, ConstD2* run_xy,
                                               ConstD4* run_box) {
    const int lane = threadIdx.x & 63;
    const double x0 = wave_extreme<false>(mine ? c.x : HUGE_VAL);
    const double x1 = wave_extreme<true>(mine ? c.x : -HUGE_VAL);
    const double y0 = wave_extreme<false>(mine ? c.y : HUGE_VAL);
    const double y1 = wave_extreme<true>(mine ? c.y : -HUGE_VAL);
    // bounds of the distances between the box and run b + lane
    auto bounds = [&](int b, double& lower, double& upper) {
        const D4 w = wall_box[min(b + lane, r1 - 1)];
        const double dx = fmax(fmax(w.x - x1, x0 - w.y), 0.0), ex = fmax(w.y - x0, x1 - w.x);
        const double dy = fmax(fmax(w.z - y1, y0 - w.w), 0.0), ey = fmax(w.w - y0, y1 - w.z);
        lower = (dx * dx + dy * dy) * (1.0 - 1e-12);
        upper = (ex * ex + ey * ey) * (1.0 + 1e-12);
    };
    double lower, upper;
    float most = HUGE_VALF;
    int first = r0;
    for (int b = r0; b < r1; b += 64) {
        bounds(b, lower, upper);
        const float u = wave_extreme<false>(upper);
        if (u < most) {  // uniform
            most = u;
            first = b + __builtin_ctzll(__ballot(__double2float_rd(upper) == u));
        }
    }
    first = uniform(__builtin_amdgcn_readfirstlane(min(first, r1 - 1)));
    double d2 = run_min(1e300, first, run_xy, c);
    most = wave_extreme<true>(mine ? d2 : 0.0);
    for (int b = r0; b < r1; b += 64) {
        if (r1 - r0 > 64) bounds(b, lower, upper);
        uint64_t todo = __ballot(lower <= most && b + lane < r1);
        if (first >= b && first < b + 64) todo &= ~(1ull << (first - b));
        for (; todo; todo &= todo - 1) {
            const int r = uniform(__builtin_amdgcn_readfirstlane(b + __builtin_ctzll(todo)));
            if (box_bound(run_box[r], c) < d2) d2 = run_min(d2, r, run_xy, c);
        }
    }
    return d2;
}

// Features of a point: position squashed into the unit disc about mid-chord,
// distance to the nearest wall point of its own cloud, Mach number and angle
// of attack recovered from the free-stream velocity.
// Bound by the search's vector instructions (about 20 boxes looked at and 5 runs
// searched by a wavefront around 1,280 wall points): 2,621,440 points about 2,560
// wall points 197 us, 640,000 about 1,280 62 us with the call.  Every point
// visiting every wall point: 3,725 and 580 us; every point visiting every box:
// 343 and 82 us.
__global__ void __launch_bounds__(256) k_features(int64_t p0, int64_t m, const D2* __restrict__ xy,
                                                  const int32_t* __restrict__ comp,
                                                  const D2* __restrict__ wall_xy,
                                                  const D4* __restrict__ wall_box,
                                                  const int32_t* __restrict__ run_off,
                                                  const double* __restrict__ vinf,
                                                  const D4* __restrict__ U, double gamma,
                                                  float* __restrict__ X, float* __restrict__ T) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t p = p0 + min(r, m - 1);  // whole wavefronts search
    const int k = comp ? comp[p] : 0;
    const D2 c = xy[p];
    // one component at a time (a wavefront may straddle two or more)
    double d2 = 1e300;
    for (uint64_t todo = __ballot(true); todo;) {
        const int ku = __builtin_amdgcn_readlane(k, __builtin_ctzll(todo)), kr = uniform(ku);
        const bool mine = k == ku;
        ConstI32* ro = (ConstI32*)run_off;
        const int r0 = ro[kr], r1 = ro[kr + 1];
        if (r1 > r0) {
            const double t = nearest_wall(mine, r0, r1, c, wall_box, (ConstD2*)wall_xy,
                                          (ConstD4*)wall_box);
            if (mine) d2 = t;
        }
        todo &= ~__ballot(mine);
    }
    if (r >= m) return;
    const double d = run_off[k + 1] > run_off[k] ? sqrt(d2) : 1e3;
    const double ex = c.x - 0.5, rc = sqrt(ex * ex + c.y * c.y);
    const double u1 = vinf[2 * k], u2 = vinf[2 * k + 1];
    const double mach = sqrt(u1 * u1 + u2 * u2);
    const double aoa = atan2(u2, u1) * (180.0 / 3.14159265358979323846);
    float* x = X + r * kIn;
    x[0] = (float)(ex / (1.0 + rc));
    x[1] = (float)(c.y / (1.0 + rc));
    x[2] = (float)(2.0 * d / (d + 0.1) - 1.0);
    x[3] = (float)((mach - 0.6) / 0.25);
    x[4] = (float)((aoa - 2.0) / 6.0);
    if (T) {
        const D4 u = U[p];
        const double irho = 1.0 / u.x, v1 = u.y * irho, v2 = u.z * irho;
        const double pr = (gamma - 1.0) * (u.w - 0.5 * u.x * (v1 * v1 + v2 * v2));
        float* t = T + r * kOut;
        t[0] = (float)(u.x - 1.0);
        t[1] = (float)(v1 - u1);
        t[2] = (float)(v2 - u2);
        t[3] = (float)(gamma * pr - 1.0);
    }
}

// U of points [p0, p0 + m) from predicted deviations from the free stream
// (rho - 1, u - u_inf, v - v_inf, gamma p - 1).  Outer points stay at the free
// stream and wall points keep only the tangential velocity.  With FALLBACK,
// only points of components flagged in bad are written, at the free stream.
template <bool FALLBACK>
__global__ void __launch_bounds__(256) k_pred_to_U(int64_t p0, int64_t m, const float* __restrict__ Y,
                                                   const int8_t* __restrict__ type,
                                                   const D2* __restrict__ frame,
                                                   const int32_t* __restrict__ comp,
                                                   const double* __restrict__ vinf, double gamma,
                                                   int32_t* __restrict__ bad, D4* __restrict__ U) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= m) return;
    const int64_t p = p0 + r;
    const int k = comp ? comp[p] : 0;
    if (FALLBACK && !bad[k]) return;
    double rho = 1.0, u1 = vinf[2 * k], u2 = vinf[2 * k + 1], gp = 1.0;
    if (!FALLBACK && type[p] != 2) {
        const float* y = Y + r * kOut;
        rho += (double)y[0];
        u1 += (double)y[1];
        u2 += (double)y[2];
        gp += (double)y[3];
        // unusable prediction: the residual check sends the whole component back to the free stream
        if (!(rho > 0.05) || !(gp > 0.05) || !(fabs(u1) + fabs(u2) < 1e3)) {
            bad[k] = 1;
            rho = 1.0;
            u1 = vinf[2 * k];
            u2 = vinf[2 * k + 1];
            gp = 1.0;
        }
    }
    if (type[p] == 0) {
        const D2 t = frame[p];
        const double ut = u1 * t.x + u2 * t.y;
        u1 = ut * t.x;
        u2 = ut * t.y;
    }
    const double pr = gp / gamma;
    U[p] = {rho, rho * u1, rho * u2, pr / (gamma - 1.0) + 0.5 * rho * (u1 * u1 + u2 * u2)};
}

__global__ void k_vet(int ncomp, const double* __restrict__ res, const double* __restrict__ res_fs,
                      int32_t* __restrict__ bad) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= ncomp) return;
    if (!(res[k] < res_fs[k])) bad[k] = 1;
}

}  // namespace

hipError_t refresh_weights(Net& net) {
    hipLaunchKernelGGL(k_refresh, dim3(nblk(kParams, 256)), dim3(256), 0, net.stream, net.theta,
                       net.copies);
    return hipGetLastError();
}

// Blocks for rows: all of them while there is a CU for each, then two a CU
// that walk over the rows.
hipError_t forward(Net& net, const float* X, int M, float* Y) {
    const float* th = net.theta;
    const WeightCopies& C = net.copies;
    const unsigned nb = std::min(nblk(M, 16 * kFwdWaves), 512u);
    hipLaunchKernelGGL(k_mlp_forward, dim3(nb), dim3(64 * kFwdWaves), 0, net.stream, M, X,
                       C.W1f, C.W2f, th + kOffB2, C.W3f, th + kOffB3, C.W4f,
                       th + kOffB4, Y);
    return hipGetLastError();
}

int part_count(int64_t rows) {
    return (int)std::min<int64_t>((rows + kTrainRows - 1) / kTrainRows, kMaxParts);
}

// Gradient (fp32, into grad) and sum of squared errors of m rows, two launches;
// lr: also an Adam step.
static hipError_t gradient_rows(Net& net, const Rows& R, int m, float* grad, double* loss,
                                const float* lr) {
    const float* th = net.theta;
    const WeightCopies& C = net.copies;
    const int nparts = part_count(m);
    hipLaunchKernelGGL(k_mlp_train, dim3(nparts), dim3(kTrainThreads), sizeof(TrainLds), net.stream, m, R,
                       C.W1f, C.W2f, th + kOffB2, C.W3f, th + kOffB3, C.W4f,
                       th + kOffB4, C.W2t, C.W3t, net.part, net.loss_part);
    const dim3 g(nblk(kParams, 64) + 1), b(256);
    if (lr) {
        net.step += 1;
        const float b1 = 0.9f, b2 = 0.999f;
        const Adam A{*lr, b1, b2, 1e-8f, 1.0f - std::pow(b1, (float)net.step),
                     1.0f - std::pow(b2, (float)net.step), net.m, net.v, net.theta};
        hipLaunchKernelGGL(k_grad_sum<true>, g, b, 0, net.stream, nparts, net.part, net.loss_part,
                           grad, loss, A, C);
    } else {
        hipLaunchKernelGGL(k_grad_sum<false>, g, b, 0, net.stream, nparts, net.part, net.loss_part,
                           grad, loss, Adam{}, C);
    }
    return hipGetLastError();
}

hipError_t gradient(Net& net, const float* X, const float* T, int m, float* grad, double* loss,
                    const float* lr) {
    return gradient_rows(net, Rows{X, T, 0, 0}, m, grad, loss, lr);
}

hipError_t minibatch_step(Net& net, int64_t n, const float* X, const float* T, int B, uint64_t seed,
                          int64_t step, double* loss, float lr) {
    return gradient_rows(net, Rows{X, T, n, seed + (uint64_t)step * (uint64_t)B}, B, nullptr, loss,
                         &lr);
}

hipError_t prepare_kernels() {
    return hipFuncSetAttribute((const void*)k_mlp_train, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)sizeof(TrainLds));
}

hipError_t features(const State& s, int64_t p0, int64_t m, float* Xout, float* Tout) {
    const Cloud& c = *s.cloud;
    hipLaunchKernelGGL(k_features, dim3(nblk(m, 256)), dim3(256), 0, s.stream, p0, m, c.xy, c.comp,
                       c.wall_xy, c.wall_box, c.wall_run_off, s.vinf, s.U, s.prm.gamma, Xout, Tout);
    return hipGetLastError();
}

hipError_t pred_to_U(Net& net, const State& s, int64_t p0, int64_t m, const float* Y) {
    const Cloud& c = *s.cloud;
    hipLaunchKernelGGL(k_pred_to_U<false>, dim3(nblk(m, 256)), dim3(256), 0, s.stream, p0, m, Y,
                       c.type, c.frame, c.comp, s.vinf, s.prm.gamma, net.d_bad, s.U);
    return hipGetLastError();
}

hipError_t vet_and_fallback(Net& net, const State& s, const double* res) {
    const Cloud& c = *s.cloud;
    hipLaunchKernelGGL(k_vet, dim3(nblk(c.ncomp, 256)), dim3(256), 0, s.stream, c.ncomp, res,
                       net.d_res_fs, net.d_bad);
    hipLaunchKernelGGL(k_pred_to_U<true>, dim3(nblk(c.n, 256)), dim3(256), 0, s.stream, (int64_t)0,
                       c.n, (const float*)nullptr, c.type, c.frame, c.comp, s.vinf, s.prm.gamma,
                       net.d_bad, s.U);
    return hipGetLastError();
}

}  // namespace mlp
}  // namespace lskum
