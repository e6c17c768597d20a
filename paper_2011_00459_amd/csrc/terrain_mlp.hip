// terrain_mlp.hip -- the learned warm start: a 12 -> 64 -> 64 -> 3 SiLU MLP
// that predicts each contact's initial impulses (lambda_n, lambda_t1,
// lambda_t2) / (m_eff g dt) in the contact frame.
//
//   k_mlp_bf16    inference on MFMA (v_mfma_f32_32x32x16_bf16): one wave per 32
//                 contacts, weights and activations in BF16, FP32 accumulate
//   k_mlp_f32     the same network in FP32 on the vector ALU (reference)
//   k_learned_lam lambda^0 = frame x output x scale, projected onto the bounds
//   k_mlp_train   FP32 forward + backward of 0.5 mean ||y - label||^2 on
//                 MFMA (FP32), per-block gradient partials reduced in fixed order
//   k_adam        Adam update
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "terrain_internal.h"

namespace trk {

namespace {

constexpr int kIn = 12, kH = 64, kOut = 3;
// offsets of the flat parameter vector
constexpr int oW1 = 0, ob1 = oW1 + kH * kIn, oW2 = ob1 + kH, ob2 = oW2 + kH * kH, oW3 = ob2 + kH,
              ob3 = oW3 + kOut * kH, oScale = ob3 + kOut;
constexpr int kNP = oScale;  // trainable parameters (in_scale is fixed)
static_assert(oScale + kIn == kMlpParams, "parameter layout");

typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ inline float silu(float z) { return z / (1.0f + __expf(-z)); }
__device__ inline float dsilu(float z)
{
    float s = 1.0f / (1.0f + __expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

// SiLU of the BF16 inference: the hardware reciprocal (about 1 ulp) in place
// of a full division
__device__ inline float silu_fast(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

}  // namespace

// ---------------------------------------------------------------------------
// BF16 MFMA inference.  Each wave works alone on tiles of 32 contacts and
// computes the transposed layers, units x contacts, so that nothing of a tile
// passes through LDS: the weights are the A operands and stay in registers,
// a lane's accumulators are units of one contact, and the pair of lanes that
// shares a contact trades half of its packed units (v_permlane32_swap) to
// have the next layer's B operand.  The input tile is read straight into the
// first B operand (the next tile's rows in flight meanwhile).
//   layer 1: W1[64 x 16] (12 inputs padded) . X^T[16 x 32]: 2 M-tiles x 1 K-step
//   layer 2: W2[64 x 64] . H1^T[64 x 32]: 2 M-tiles x 4 K-steps
//   layer 3: W3[32 x 64] (3 of 32 rows used) . H2^T[64 x 32]: 4 K-steps
// Operand layouts of v_mfma_f32_32x32x16_bf16 (A 32x16, B 16x32, D 32x32):
//   A[i][k] -> lane i + 32 (k / 8), element k % 8
//   B[k][j] -> lane j + 32 (k / 8), element k % 8
//   D[i][j] -> lane j + 32 ((i / 4) % 2), element (i % 4) + 4 (i / 8)
// Bound by the vector ALU: 128 SiLUs a contact, each an exponential and a
// reciprocal at a quarter of the rate and four or five plain operations, is
// about 3,300 cycles a tile of a SIMD, where a tile takes 3,280.  2^22
// contacts take 184 us; with weights and layers in LDS they took 202, and
// three waves a SIMD, for which the registers spill, take 215.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));

constexpr int kMlpWaves = 4;

__global__ __launch_bounds__(64 * kMlpWaves, 2) void k_mlp_bf16(const float* __restrict__ W,
                                                                const float* __restrict__ feat,
                                                                float* __restrict__ out, const uint32_t* d_n,
                                                                int64_t cap)
{
    // the weights come through LDS (rows of 64 + 8 BF16), one reading of them a block
    __shared__ __attribute__((aligned(16))) __bf16 w1s[kH][16 + 8], w2s[kH][kH + 8], w3s[kOut + 1][kH + 8];
    __shared__ __attribute__((aligned(16))) float bias[2][kH];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int half = lane >> 5, col = lane & 31;
    for (int t = tid; t < kH * 16; t += blockDim.x)
        w1s[t / 16][t % 16] = (__bf16)(t % 16 < kIn ? W[oW1 + t / 16 * kIn + t % 16] : 0.0f);
    for (int t = tid; t < kH * kH; t += blockDim.x) w2s[t / kH][t % kH] = (__bf16)W[oW2 + t];
    for (int t = tid; t < (kOut + 1) * kH; t += blockDim.x)
        w3s[t / kH][t % kH] = (__bf16)(t < kOut * kH ? W[oW3 + t] : 0.0f);
    for (int t = tid; t < 2 * kH; t += blockDim.x) bias[t / kH][t % kH] = W[(t < kH ? ob1 : ob2) + t % kH];
    __syncthreads();  // the only block barrier: the weights are read-only afterwards
    // lane (col, half) holds weights 8 half .. 8 half + 7 of each K-step into
    // unit col (W1 padded to K = 16, W3 to 32 rows)
    auto row = [&](const __bf16* r, int k0) { return *reinterpret_cast<const bf16x8*>(r + k0 + half * 8); };
    bf16x8 w1[2], w2[2][4], w3[4];
    for (int m = 0; m < 2; ++m) {
        w1[m] = row(w1s[m * 32 + col], 0);
        for (int ks = 0; ks < 4; ++ks) w2[m][ks] = row(w2s[m * 32 + col], ks * 16);
    }
    for (int ks = 0; ks < 4; ++ks) w3[ks] = row(w3s[min(col, kOut)], ks * 16);
    const float b3[kOut] = {W[ob3], W[ob3 + 1], W[ob3 + 2]};
    float scl[8];  // scales of this lane's input columns 8 half .. 8 half + 7
    for (int q = 0; q < 8; ++q) scl[q] = half * 8 + q < kIn ? W[oScale + half * 8 + q] : 0.0f;

    const uint64_t n = d_n ? (uint64_t)min((uint64_t)*d_n, (uint64_t)cap) : (uint64_t)cap;
    const uint64_t ntiles = (n + 31) / 32;
    const uint64_t nwaves = (uint64_t)gridDim.x * kMlpWaves;
    // the input row of a tile: lane (col, half) holds features 8 half .. 8 half + 7
    // (only 8 .. 11 of the second half are inside the 12)
    auto load_x = [&](uint64_t tile, float4& x0, float4& x1) {
        const uint64_t c = tile * 32 + col;
        x0 = make_float4(0.f, 0.f, 0.f, 0.f);
        x1 = x0;
        if (tile < ntiles && c < n) {
            const float4* f = reinterpret_cast<const float4*>(feat + c * kIn);
            x0 = f[2 * half];
            if (half == 0) x1 = f[1];
        }
    };
    // M-tile (+ bias, SiLU) in BF16 -> the next layer's B operands of its two
    // K-steps.  The lane's units of a K-step are 4 half .. 4 half + 3 and 8 more;
    // the swap gives the lower lanes 0 .. 7 and the upper ones 8 .. 15.
    // Accumulator element e is unit 8 (e / 4) + 4 half + e % 4.
    auto activate = [&](const floatx16& acc, const float* bs, bf16x8* B) {
        for (int ks = 0; ks < 2; ++ks) {
            unsigned p[4];
            for (int t = 0; t < 2; ++t) {
                const int e = ks * 8 + 4 * t;
                const float4 q = *reinterpret_cast<const float4*>(bs + 2 * e + 4 * half);
                const bf16x2 h0 = {(__bf16)silu_fast(acc[e] + q.x), (__bf16)silu_fast(acc[e + 1] + q.y)};
                const bf16x2 h1 = {(__bf16)silu_fast(acc[e + 2] + q.z), (__bf16)silu_fast(acc[e + 3] + q.w)};
                p[2 * t] = __builtin_bit_cast(unsigned, h0);
                p[2 * t + 1] = __builtin_bit_cast(unsigned, h1);
            }
            const uintx2 s0 = __builtin_amdgcn_permlane32_swap(p[0], p[2], false, false);
            const uintx2 s1 = __builtin_amdgcn_permlane32_swap(p[1], p[3], false, false);
            const uint4 v = make_uint4(s0[0], s1[0], s0[1], s1[1]);
            B[ks] = __builtin_bit_cast(bf16x8, v);
        }
    };
    uint64_t tile = (uint64_t)blockIdx.x * kMlpWaves + wave;
    float4 x0, x1;
    load_x(tile, x0, x1);
    for (; tile < ntiles; tile += nwaves) {
        bf16x8 X, H1[4], H2[4];
        X[0] = (__bf16)(x0.x * scl[0]); X[1] = (__bf16)(x0.y * scl[1]);
        X[2] = (__bf16)(x0.z * scl[2]); X[3] = (__bf16)(x0.w * scl[3]);
        X[4] = (__bf16)(x1.x * scl[4]); X[5] = (__bf16)(x1.y * scl[5]);
        X[6] = (__bf16)(x1.z * scl[6]); X[7] = (__bf16)(x1.w * scl[7]);
        load_x(tile + nwaves, x0, x1);  // the next tile's rows, in flight meanwhile
        floatx16 d[2] = {};
        for (int m = 0; m < 2; ++m) {
            d[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1[m], X, d[m], 0, 0, 0);
            activate(d[m], bias[0] + 32 * m, H1 + 2 * m);
        }
        for (int m = 0; m < 2; ++m) {
            d[m] = floatx16{};
            for (int ks = 0; ks < 4; ++ks)
                d[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w2[m][ks], H1[ks], d[m], 0, 0, 0);
        }
        for (int m = 0; m < 2; ++m) activate(d[m], bias[1] + 32 * m, H2 + 2 * m);
        floatx16 y = {};
        for (int ks = 0; ks < 4; ++ks) y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w3[ks], H2[ks], y, 0, 0, 0);
        // units 0 .. 2 of the lower lanes are the contact's outputs
        const uint64_t c = tile * 32 + col;
        if (half == 0 && c < n)
            for (int q = 0; q < kOut; ++q) out[c * kOut + q] = y[q] + b3[q];
    }
}

// FP32 reference inference: one thread per contact
__global__ __launch_bounds__(256) void k_mlp_f32(const float* __restrict__ W, const float* __restrict__ feat,
                                                 float* __restrict__ out, const uint32_t* d_n, int64_t cap)
{
    __shared__ float w[kMlpParams];
    for (int t = threadIdx.x; t < kMlpParams; t += blockDim.x) w[t] = W[t];
    __syncthreads();
    uint64_t n = d_n ? (uint64_t)min((uint64_t)*d_n, (uint64_t)cap) : (uint64_t)cap;
    for (uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (uint64_t)gridDim.x * blockDim.x) {
        float x0[kIn], h1[kH];
        for (int k = 0; k < kIn; ++k) x0[k] = feat[c * kIn + k] * w[oScale + k];
        for (int o = 0; o < kH; ++o) {
            float z = w[ob1 + o];
            for (int k = 0; k < kIn; ++k) z += w[oW1 + o * kIn + k] * x0[k];
            h1[o] = silu(z);
        }
        float y[kOut] = {w[ob3], w[ob3 + 1], w[ob3 + 2]};
        for (int o = 0; o < kH; ++o) {
            float z = w[ob2 + o];
            for (int k = 0; k < kH; ++k) z += w[oW2 + o * kH + k] * h1[k];
            float h = silu(z);
            for (int q = 0; q < kOut; ++q) y[q] += w[oW3 + q * kH + o] * h;
        }
        for (int q = 0; q < kOut; ++q) out[c * kOut + q] = y[q];
    }
}

void launch_mlp_infer(const float* W, const float* feat, float* out, const uint32_t* d_n, int64_t cap, bool bf16,
                      hipStream_t s)
{
    if (cap <= 0) return;
    if (bf16) {
        // one round of resident blocks, each wave looping over tiles
        static int resident = 0;
        if (!resident) {
            int dev = 0, per_cu = 0;
            (void)hipGetDevice(&dev);
            hipDeviceProp_t pr;
            (void)hipGetDeviceProperties(&pr, dev);
            (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_mlp_bf16, 64 * kMlpWaves, 0);
            resident = std::max(1, per_cu) * pr.multiProcessorCount;
        }
        int64_t tiles = (cap + 31) / 32;
        int grid = (int)std::min<int64_t>((tiles + kMlpWaves - 1) / kMlpWaves, resident);
        hipLaunchKernelGGL(k_mlp_bf16, dim3(grid), dim3(64 * kMlpWaves), 0, s, W, feat, out, d_n, cap);
    } else {
        int grid = (int)std::min<int64_t>((cap + 255) / 256, 2048);
        hipLaunchKernelGGL(k_mlp_f32, dim3(grid), dim3(256), 0, s, W, feat, out, d_n, cap);
    }
}

// ---------------------------------------------------------------------------
// lambda^0 of the learned start (colour order): world impulse from the
// previous-step impulse plus the network output in the contact frame, projected
// onto {ln >= lo, |lt| <= mu |ln|}
// ---------------------------------------------------------------------------
__global__ void k_learned_lam(DevBuffers b, StepParams p, int64_t cap)
{
    uint32_t nc = b.cnt->n_raw < (uint64_t)cap ? b.cnt->n_raw : (uint32_t)cap;
    uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nc || b.cnt->overflow) return;
    float4 f1 = b.frm1[c], f2 = b.frm2[c], a = b.r0[c], q = b.r2[c];
    // residual form: the output corrects the previous-step impulse in the
    // contact frame (inputs 3-5), so a zero output is the previous-step start
    const float* fc = b.feat + (size_t)c * 12;
    float y0 = fc[3] + b.mlp_out[3 * (size_t)c], y1 = fc[4] + b.mlp_out[3 * (size_t)c + 1],
          y2 = fc[5] + b.mlp_out[3 * (size_t)c + 2];
    float ls = f1.w;
    float ln = y0 * ls;
    float t0 = (y1 * f1.x + y2 * f2.x) * ls, t1 = (y1 * f1.y + y2 * f2.y) * ls, t2 = (y1 * f1.z + y2 * f2.z) * ls;
    if (!(isfinite(ln) && isfinite(t0) && isfinite(t1) && isfinite(t2))) {
        atomicOr(&b.ustats[__float_as_int(f2.w)].learn_bad, 1u);
        ln = 0.f; t0 = t1 = t2 = 0.f;
    }
    ln = fmaxf(ln, q.y);
    float tn = a.x * t0 + a.y * t1 + a.z * t2;
    t0 -= tn * a.x; t1 -= tn * a.y; t2 -= tn * a.z;
    float lim = p.mu * fabsf(ln);
    float m2 = t0 * t0 + t1 * t1 + t2 * t2;
    if (m2 > lim * lim) {
        float sc = m2 > 0.f ? lim * rsqrtf(m2) : 0.f;
        t0 *= sc; t1 *= sc; t2 *= sc;
    }
    b.lamL[c] = make_float4(ln, t0, t1, t2);
}

void launch_learned_lam(const DevBuffers& b, const StepParams& p, const Sizes& z, hipStream_t s)
{
    hipLaunchKernelGGL(k_learned_lam, dim3((unsigned)((z.C + 255) / 256)), dim3(256), 0, s, b, p, z.C);
}

// ---------------------------------------------------------------------------
// training: forward + backward of 0.5 mean ||y - label||^2 in FP32 on MFMA
// (v_mfma_f32_16x16x4f32, FP32 products and sums).  A block's 16 waves are
// four groups of four; a group takes tiles of 32 samples, R of them (128 R
// samples a block, R from 1 to 4 so that a call fills the 256 CUs where the
// batch allows), and each of its waves a quarter of every product: 16 units
// of a layer, 16 rows of a weight gradient.  Per tile:
//   layer 1   Z1[32 x 64] = X[32 x 12] . W1^T          2 x 4 tiles x 3 K-steps
//   layer 2   Z2 = H1 . W2^T                           2 x 4 tiles x 16 K-steps
//   layer 3   y = H2 . W3^T (3 outputs: vector ALU)
//   backward  gZ2 = (gy . W3) o silu'(Z2) (vector ALU)
//             gZ1 = (gZ2 . W2) o silu'(Z1)             2 x 4 tiles x 16 K-steps
//   gradients dW2 += gZ2^T . H1  (64 x 64, K = 32 samples: 4 x 4 tiles x 8)
//             dW1 += gZ1^T . X   (64 x 12 of one 16-wide tile: 4 tiles x 8)
//             dW3, the biases and the loss on the vector ALU
// The gradient accumulators stay in registers across a group's tiles; the
// groups' sums are added in a fixed order and written as the block's partial
// to part[block][kNP] (loss at part[.][kNP]).
// Operand layouts (A 16x4, B 4x16, D 16x16): A[i][k] -> lane i + 16 k,
// B[k][j] -> lane j + 16 k, D[i][j] -> lane j + 16 (i / 4), element i % 4.
//
// A batch of 4,096 is 32 blocks, and what bounds it is the chain of one tile:
// with one wave a tile, and the rows of W2 in LDS all starting at one bank, it
// took 49 us, now 22.
// ---------------------------------------------------------------------------
constexpr int kTrainWaves = 4;  // tiles of a block at once: groups of kTrainQ waves
constexpr int kTrainQ = 4;
// LDS pitch of the 64-wide rows: 16 rows by 4 columns, an operand's lanes, fall into 64 banks
constexpr int kTP = kH + 4;
constexpr int kXP = kIn + 1;    // of the 12-wide ones

// tiles per group and blocks of a batch of B samples
__host__ __device__ constexpr int train_tiles(int64_t B)
{
    return B > (int64_t)3 * kTrainWaves * 32 * 256 ? 4 : (B > (int64_t)kTrainWaves * 32 * 256 ? 2 : 1);
}
__host__ __device__ constexpr int64_t train_blocks(int64_t B)
{
    return (B + (int64_t)kTrainWaves * 32 * train_tiles(B) - 1) / ((int64_t)kTrainWaves * 32 * train_tiles(B));
}

typedef float floatx4 __attribute__((ext_vector_type(4)));
__device__ inline floatx4 mfma16(float a, float b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// LDS of a group.  h1, h2 and g hold H1, H2 then gZ1, and gZ2; at the end the
// group's gradients (kNP values) and what its waves add to dW3, b3 and the loss.
struct TrainGroup {
    float h1[32][kTP], h2[32][kTP], g[32][kTP];
    float xs[32][kXP];
    float gy[32][kOut + 1];
    float yp[kTrainQ][32][kOut];
};
constexpr int kTail = kOut * kH + kOut + 1;  // dW3, b3, loss of one wave
static_assert(kNP + kTrainQ * kTail <= 3 * 32 * kTP, "a group's gradients take the place of its activations");

__global__ __launch_bounds__(64 * kTrainQ * kTrainWaves) void k_mlp_train(const float* __restrict__ W,
                                                                          const float* __restrict__ feat,
                                                                          const float* __restrict__ label, int64_t B,
                                                                          int tiles, float* __restrict__ part)
{
    __shared__ float w1[kH][kXP], w2[kH][kTP], w3[kOut][kH], bias[2][kH], b3[kOut];
    __shared__ TrainGroup gm[kTrainWaves];
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63, grp = wave / kTrainQ, wq = wave % kTrainQ;
    const int l16 = lane & 15, q4 = lane >> 4, s32 = lane & 31;
    const int u0 = 16 * wq, u = u0 + l16;  // the wave's units, the lane's
    TrainGroup& G = gm[grp];
    const float inv_b = 1.0f / (float)B;
    // two of the group's 32 x 12 inputs a lane (the second of half the lanes) and, for its first wave, the labels
    const int e0 = wq * 64 + lane, e1 = min(e0 + 64 * kTrainQ, 32 * kIn - 1);
    const float sc0 = W[oScale + e0 % kIn], sc1 = W[oScale + e1 % kIn];
    float x0 = 0.0f, x1 = 0.0f, lab[kOut] = {0.0f, 0.0f, 0.0f};
    auto read_tile = [&](int r) {
        const int64_t s0 = (((int64_t)blockIdx.x * tiles + r) * kTrainWaves + grp) * 32;
        x0 = s0 + e0 / kIn < B ? feat[s0 * kIn + e0] : 0.0f;
        x1 = s0 + e1 / kIn < B ? feat[s0 * kIn + e1] : 0.0f;
        if (wq == 0)
            for (int q = 0; q < kOut; ++q) lab[q] = s0 + s32 < B ? label[(s0 + s32) * kOut + q] : 0.0f;
    };
    read_tile(0);
    {
        // every load of the weights in flight at once: one after the other they would cost 10 us
        static_assert(kH * kIn <= 1024 && kH * kH == 4096 && 64 * kTrainQ * kTrainWaves == 1024, "one pass each");
        float v2[4];
        for (int k = 0; k < 4; ++k) v2[k] = W[oW2 + t + 1024 * k];
        const float v1 = W[oW1 + min(t, kH * kIn - 1)], v3 = W[oW3 + min(t, kOut * kH - 1)];
        const float vb = W[(t < kH ? ob1 : ob2) + t % kH], v4 = W[ob3 + min(t, kOut - 1)];
        for (int k = 0; k < 4; ++k) w2[(t + 1024 * k) / kH][t % kH] = v2[k];
        if (t < kH * kIn) w1[t / kIn][t % kIn] = v1;
        if (t < kOut * kH) w3[t / kH][t % kH] = v3;
        if (t < 2 * kH) bias[t / kH][t % kH] = vb;
        if (t < kOut) b3[t] = v4;
    }
    floatx4 dW2[4], dW1 = {};
    for (int n = 0; n < 4; ++n) dW2[n] = floatx4{};
    float dW3[kOut] = {0.0f, 0.0f, 0.0f}, db1 = 0.0f, db2 = 0.0f, db3 = 0.0f, loss = 0.0f;
    for (int r = 0; r < tiles; ++r) {
        // (opaque here: the addresses of all LDS operands would else be kept
        // across tiles, and spill)
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int l16 = ln & 15, q4 = ln >> 4, s32 = ln & 31, half = ln >> 5, u = u0 + l16;
        const int64_t s0 = (((int64_t)blockIdx.x * tiles + r) * kTrainWaves + grp) * 32;
        G.xs[e0 / kIn][e0 % kIn] = x0 * sc0;
        if (e1 == e0 + 64 * kTrainQ) G.xs[e1 / kIn][e1 % kIn] = x1 * sc1;
        __syncthreads();
        // layers 1 and 2: the wave's 16 units of Z in registers (D layout), H into LDS
        floatx4 z1[2], z2[2];
        for (int m = 0; m < 2; ++m) {
            floatx4 acc = {};
            for (int kk = 0; kk < kIn / 4; ++kk)
                acc = mfma16(G.xs[m * 16 + l16][4 * kk + q4], w1[u][4 * kk + q4], acc);
            for (int e = 0; e < 4; ++e) {
                z1[m][e] = acc[e] + bias[0][u];
                G.h1[m * 16 + 4 * q4 + e][u] = silu(z1[m][e]);
            }
        }
        __syncthreads();
        {
            floatx4 acc[2] = {};
#pragma unroll 4
            for (int kk = 0; kk < kH / 4; ++kk) {
                const float bw = w2[u][4 * kk + q4];
                for (int m = 0; m < 2; ++m) acc[m] = mfma16(G.h1[m * 16 + l16][4 * kk + q4], bw, acc[m]);
            }
            for (int m = 0; m < 2; ++m)
                for (int e = 0; e < 4; ++e) {
                    z2[m][e] = acc[m][e] + bias[1][u];
                    G.h2[m * 16 + 4 * q4 + e][u] = silu(z2[m][e]);
                }
        }
        __syncthreads();
        // layer 3: sample s32, an eighth of H2's columns a lane
        {
            float y[kOut] = {0.0f, 0.0f, 0.0f};
            const int k0 = u0 + 8 * half;
            for (int k = k0; k < k0 + 8; ++k) {
                const float h = G.h2[s32][k];
                for (int q = 0; q < kOut; ++q) y[q] += w3[q][k] * h;
            }
            for (int q = 0; q < kOut; ++q) {
                y[q] += __shfl_xor(y[q], 32);
                if (half == 0) G.yp[wq][s32][q] = y[q];
            }
        }
        __syncthreads();
        if (wq == 0 && half == 0)
            for (int q = 0; q < kOut; ++q) {
                const float y = (G.yp[0][s32][q] + G.yp[1][s32][q]) + (G.yp[2][s32][q] + G.yp[3][s32][q]);
                const float e = s0 + s32 < B ? (y + b3[q]) - lab[q] : 0.0f;
                G.gy[s32][q] = e * inv_b;
                loss += 0.5f * e * e;
            }
        if (r + 1 < tiles) read_tile(r + 1);
        __syncthreads();
        // dW3 (row q, column lane) and db3 over a quarter of the samples
        for (int i = 8 * wq; i < 8 * wq + 8; ++i) {
            const float h = G.h2[i][ln];
            for (int q = 0; q < kOut; ++q) dW3[q] += G.gy[i][q] * h;
            if (ln < kOut) db3 += G.gy[i][ln];
        }
        // gZ2 = (gy . W3) o silu'(Z2)
        for (int m = 0; m < 2; ++m)
            for (int e = 0; e < 4; ++e) {
                const int i = m * 16 + 4 * q4 + e;
                float gh = 0.0f;
                for (int q = 0; q < kOut; ++q) gh += G.gy[i][q] * w3[q][u];
                const float g = gh * dsilu(z2[m][e]);
                G.g[i][u] = g;
                db2 += g;
            }
        __syncthreads();
        // dW2 += gZ2^T . H1, rows u0 .. u0 + 15
#pragma unroll 4
        for (int kk = 0; kk < 8; ++kk) {
            const int i = 4 * kk + q4;
            const float ag = G.g[i][u];
            for (int n = 0; n < 4; ++n) dW2[n] = mfma16(ag, G.h1[i][n * 16 + l16], dW2[n]);
        }
        // gZ1 = (gZ2 . W2) o silu'(Z1), in H2's place
        {
            floatx4 acc[2] = {};
#pragma unroll 4
            for (int kk = 0; kk < kH / 4; ++kk) {
                const float bw = w2[4 * kk + q4][u];
                for (int m = 0; m < 2; ++m) acc[m] = mfma16(G.g[m * 16 + l16][4 * kk + q4], bw, acc[m]);
            }
            for (int m = 0; m < 2; ++m)
                for (int e = 0; e < 4; ++e) {
                    const float g = acc[m][e] * dsilu(z1[m][e]);
                    G.h2[m * 16 + 4 * q4 + e][u] = g;
                    db1 += g;
                }
        }
        // dW1 += gZ1^T . X, rows u0 .. u0 + 15 (of this wave's own units), columns l16 < 12
        __syncthreads();
#pragma unroll 4
        for (int kk = 0; kk < 8; ++kk) {
            const int i = 4 * kk + q4;
            dW1 = mfma16(G.h2[i][u], l16 < kIn ? G.xs[i][l16] : 0.0f, dW1);
        }
        __syncthreads();  // the group's buffers are rewritten by its next tile
    }
    // the group's gradients over its activations; dW3, b3 and the loss a wave at a time behind them
    float* red = &G.h1[0][0];
    for (int e = 0; e < 4; ++e) {
        const int o = u0 + 4 * q4 + e;
        for (int n = 0; n < 4; ++n) red[oW2 + o * kH + n * 16 + l16] = dW2[n][e];
        if (l16 < kIn) red[oW1 + o * kIn + l16] = dW1[e];
    }
    db1 += __shfl_xor(db1, 16);
    db1 += __shfl_xor(db1, 32);
    db2 += __shfl_xor(db2, 16);
    db2 += __shfl_xor(db2, 32);
    if (q4 == 0) {
        red[ob1 + u] = db1;
        red[ob2 + u] = db2;
    }
    float* tail = red + kNP + wq * kTail;
    for (int q = 0; q < kOut; ++q) tail[q * kH + lane] = dW3[q];
    if (lane < kOut) tail[kOut * kH + lane] = db3;
    for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o);
    if (lane == 0) tail[kTail - 1] = loss * inv_b;
    __syncthreads();
    float* out = part + (size_t)blockIdx.x * (kNP + 1);
    for (int k = t; k <= kNP; k += blockDim.x) {
        const int at = k >= oW3 && k < oW3 + kOut * kH ? k - oW3
                       : k >= ob3 && k < ob3 + kOut    ? kOut * kH + k - ob3
                                                       : (k == kNP ? kTail - 1 : -1);
        float v = 0.0f;
        for (int gq = 0; gq < kTrainWaves; ++gq) {
            const float* rg = &gm[gq].h1[0][0];
            if (at < 0) v += rg[k];
            else
                for (int q = 0; q < kTrainQ; ++q) v += rg[kNP + q * kTail + at];
        }
        out[k] = v;
    }
}

// the blocks' partials summed in a fixed order: 64 parameters per block of
// 1024 threads, 16 groups each summing every 16th partial (64 consecutive
// parameters per load: coalesced), then the 16 group sums in group order
constexpr int kRedGroups = 16;
__global__ __launch_bounds__(64 * kRedGroups) void k_grad_reduce(const float* __restrict__ part, int nblocks,
                                                                   float* __restrict__ grad, float* loss)
{
    __shared__ float gs[kRedGroups][64];
    const int j = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int pidx = blockIdx.x * 64 + j;
    float g = 0.0f;
    if (pidx <= kNP)
        for (int b = grp; b < nblocks; b += kRedGroups) g += part[(size_t)b * (kNP + 1) + pidx];
    gs[grp][j] = g;
    __syncthreads();
    if (grp == 0 && pidx <= kNP) {
        float t = 0.0f;
        for (int k = 0; k < kRedGroups; ++k) t += gs[k][j];
        if (pidx < kNP) grad[pidx] = t;
        else if (loss) *loss = t;
    }
}

__global__ void k_adam(float* W, const float* g, float* m, float* v, int n, float lr, float b1, float b2, float eps,
                       float c1, float c2)
{
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    float gk = g[k];
    float mk = b1 * m[k] + (1.0f - b1) * gk;
    float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    W[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

int64_t mlp_grad_scratch(int64_t B) { return train_blocks(B) * (int64_t)(kNP + 1); }
int mlp_trainable() { return kNP; }

void launch_mlp_grad(const float* W, const float* feat, const float* label, int64_t B, float* grad, float* loss,
                     float* scratch, hipStream_t s)
{
    const int nb = (int)train_blocks(B);
    hipLaunchKernelGGL(k_mlp_train, dim3(nb), dim3(64 * kTrainQ * kTrainWaves), 0, s, W, feat, label, B, train_tiles(B),
                       scratch);
    hipLaunchKernelGGL(k_grad_reduce, dim3((kNP + 1 + 63) / 64), dim3(64 * kRedGroups), 0, s, scratch, nb, grad, loss);
}

void launch_adam(float* W, const float* g, float* m, float* v, int n, float lr, float b1, float b2, float eps, int t,
                 hipStream_t s)
{
    float c1 = 1.0f - powf(b1, (float)t), c2 = 1.0f - powf(b2, (float)t);
    hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, s, W, g, m, v, n, lr, b1, b2, eps, c1, c2);
}

}  // namespace trk

// ---------------------------------------------------------------------------
// Loss gradient without allocation: the per-block gradient partials live in a
// file-scope device array of fixed size instead of a caller workspace.
// ---------------------------------------------------------------------------
namespace {
constexpr int64_t kNoAllocMaxBatch = TR_MLP_NOALLOC_MAX_BATCH;
constexpr int64_t kNoAllocFloats = trk::train_blocks(kNoAllocMaxBatch) * (int64_t)(trk::kNP + 1);
constexpr int kMaxDevices = 64;

// One copy per GPU, held until the process ends.  Host code never passes the
// array's name to a kernel: the device address of each GPU's copy comes from
// hipGetSymbolAddress on that GPU.
static __device__ __align__(256) float g_train_scratch[kNoAllocFloats];

std::mutex g_scratch_mu;
float* g_scratch_ptr[kMaxDevices] = {};

// Device address of this GPU's copy (looked up once per device, with the
// device current).  nullptr on failure.
float* train_scratch_ptr(int dev)
{
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_train_scratch)) != hipSuccess || !p) return nullptr;
        g_scratch_ptr[dev] = static_cast<float*>(p);
    }
    return g_scratch_ptr[dev];
}
}  // namespace

extern "C" int mlp_loss_grad_noalloc(const float* weights, const float* feat, const float* label, int64_t B,
                                     float* grad, float* loss, void* stream)
{
    if (!weights || !feat || !label || !grad || B <= 0) return TR_E_INVAL;
    if (B > kNoAllocMaxBatch) return TR_E_CAPACITY;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return TR_E_DEVICE;
    float* scratch = train_scratch_ptr(dev);
    if (!scratch) return TR_E_DEVICE;
    trk::launch_mlp_grad(weights, feat, label, B, grad, loss, scratch, (hipStream_t)stream);
    return hipGetLastError() == hipSuccess ? TR_OK : TR_E_DEVICE;
}
