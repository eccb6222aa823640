// Learned cost model: per-point features from the cover tree, a 16-64-64-2
// perceptron (SiLU) with hand-written forward, backward and Adam kernels,
// and inference.  It predicts, for every point, log1p of the number of
// block pairs its query pack takes part in ("visits") and log1p of its
// neighbour count.  The predictions only size CSR rows and order work; no
// edge decision depends on them.
//
// Parameter layout (row-major, one contiguous float buffer):
//   W1 [64][16], b1 [64], W2 [64][64], b2 [64], W3 [2][64], b3 [2].
// Loss: L = 1/(2B) * sum_b sum_o (y_bo - t_bo)^2.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "learn.h"

namespace fnn {

constexpr int OW1 = 0, OB1 = OW1 + MLP_H * MLP_F, OW2 = OB1 + MLP_H,
              OB2 = OW2 + MLP_H * MLP_H, OW3 = OB2 + MLP_H,
              OB3 = OW3 + MLP_O * MLP_H;
static_assert(OB3 + MLP_O == MLP_NPAR, "parameter layout");

__device__ __forceinline__ float silu(float z) { return z / (1.f + expf(-z)); }

// ------------------------------------------------------------- features --

__global__ void k_parent(const int32_t *__restrict__ cbeg,
                         const int32_t *__restrict__ ccnt, int nn,
                         int32_t *__restrict__ parent)
{
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < nn;
         v += gridDim.x * blockDim.x) {
        if (v == 0)
            parent[0] = -1;
        for (int c = 0; c < ccnt[v]; ++c)
            parent[cbeg[v] + c] = v;
    }
}

__global__ void k_depth(const int32_t *__restrict__ parent, int nn,
                        int32_t *__restrict__ depth)
{
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < nn;
         v += gridDim.x * blockDim.x) {
        int d = 0, u = v;
        while (parent[u] >= 0 && d < 4096) {
            u = parent[u];
            ++d;
        }
        depth[v] = d;
    }
}

// owner[pos] = id of the range [pb, pe) holding pos, for ranges that tile
// the positions (leaf blocks, or packs).
__global__ void k_owner(const int32_t *__restrict__ pb, const int32_t *__restrict__ pe,
                        const int32_t *__restrict__ ccnt, int first, int count,
                        int only_leaves, int32_t *__restrict__ owner)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const int wpb = blockDim.x / WAVE;
    for (int k = blockIdx.x * wpb + threadIdx.x / WAVE; k < count;
         k += gridDim.x * wpb) {
        const int v = first + k;
        if (only_leaves && ccnt[v] != 0)
            continue;
        for (int p = pb[v] + lane; p < pe[v]; p += WAVE)
            owner[p] = v;
    }
}

// Per-point features (16, scale-free; eps is the point's own cloud's):
//  0 log2(1 + pack size) / 6        1 depth of the point's leaf / 8
//  2 log2(r_pack / eps)             3 d(p, pack centre) / eps (<= 16)
//  4 log2(r / eps) of the parent    5 the same for the grandparent
//  6 d(p, centre) / r of the parent 7 the same for the grandparent (<= 2)
//  8, 9, 10 log1p(pack members within eps, 2 eps, eps / 2) / 6
// 11 mean distance to the pack members / eps (each <= 16)
// 12 log2(1 + size of the smallest ancestor with r >= eps) / 20
// 13 log2(1 + the parent's child count) / 8
// 14 log2(1 + the parent's size) / 20
// 15 distance to the nearest other pack member / eps (<= 4)
// No feature is constant over a whole tree (such a value would let the
// network recognise the training set instead of the point's surroundings).
template <int M>
__global__ void k_features(Pts P, FeatArgs A, int local_done, float *__restrict__ feat)
{
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < P.n;
         p += gridDim.x * blockDim.x) {
        float f[MLP_F];
        const int pk = A.pack_of[p];
        const int v0 = A.leaf_of[p];
        const int cl = A.pcl ? A.pcl[p] : -1;
        const float eps = cl >= 0 ? A.ct[cl].feps : A.eps;
        const float tiny = 1.0f / 1048576.0f;
        const int qb = A.q_pb[pk], qe = A.q_pe[pk];
        f[0] = log2f(1.f + (float)(qe - qb)) / 6.f;
        f[1] = (float)A.depth[v0] / 8.f;
        f[2] = log2f(A.q_rad[pk] / eps + tiny);
        f[3] = fminf(key_to_dist<M>(key32<M>(P, p, A.q_cpos[pk])) / eps, 16.f);
        int v = v0;
        for (int k = 0; k < 2; ++k) {
            if (A.parent[v] >= 0)
                v = A.parent[v];
            const float r = A.radius[v];
            f[4 + k] = log2f(r / eps + tiny);
            const float d = key_to_dist<M>(key32<M>(P, p, A.center_pos[v]));
            f[6 + k] = fminf(d / (r + 1e-30f), 2.f);
        }
        // the point's own pack as a local sample of its neighbourhood: the
        // whole pack when it holds at most 64 points (then the lanes of a
        // pack read the same member rows in step), else 64 members around p
        // (a duplicate leaf can be larger)
        // packs of at most 64 points get these from k_pack_local when it runs
        const bool mine = !local_done || qe - qb > 64;
        const int lo = qe - qb <= 64 ? qb : max(qb, min(p - 32, qe - 64));
        const int hi = mine ? min(qe, lo + 64) : lo;
        int c1 = 0, c2 = 0, ch = 0;
        float sum = 0.f, dmin = 4.f * eps;
        for (int q = lo; q < hi; ++q) {
            if (q == p)
                continue;
            const float d = key_to_dist<M>(key32<M>(P, p, q));
            c1 += d <= eps;
            c2 += d <= 2.f * eps;
            ch += d <= 0.5f * eps;
            sum += fminf(d, 16.f * eps);
            dmin = fminf(dmin, d);
        }
        const int others = max(hi - lo - 1, 1);
        f[8] = log1pf((float)c1) / 6.f;
        f[9] = log1pf((float)c2) / 6.f;
        f[10] = log1pf((float)ch) / 6.f;
        f[11] = sum / ((float)others * eps);
        int u = v0;
        while (A.radius[u] < eps && A.parent[u] >= 0)
            u = A.parent[u];
        f[12] = log2f(1.f + (float)(A.pe[u] - A.pb[u])) / 20.f;
        const int v1 = A.parent[v0] >= 0 ? A.parent[v0] : v0;
        f[13] = log2f(1.f + (float)A.ccnt[v1]) / 8.f;
        f[14] = log2f(1.f + (float)(A.pe[v1] - A.pb[v1])) / 20.f;
        f[15] = dmin / eps;
#pragma unroll
        for (int k = 0; k < MLP_F; ++k)
            if (mine || (k != 8 && k != 9 && k != 10 && k != 11 && k != 15))
                feat[(size_t)p * MLP_F + k] = f[k];
    }
}

// Features 8-11 and 15 (the pack as a local sample) for vector rows of at
// most LOC_MAXD floats: one work-group per pack of at most 64 points, its
// rows staged in LDS (odd row stride: lanes reading one coordinate of
// different rows hit different banks); thread t takes point t / 4 against
// every fourth member, and the four partial results meet by shuffles.
constexpr int LOC_MAXD = 128;
template <int M>
__global__ void __launch_bounds__(256)
k_pack_local(Pts P, FeatArgs A, float *__restrict__ feat)
{
    __shared__ float rows[64 * (LOC_MAXD + 1)];
    const float *X = M == M_L2 ? P.x : P.xn;
    const int dp = P.dp, ld = dp + 1, t = threadIdx.x;
    const int npk = A.npacks;
    for (int k = blockIdx.x; k < npk; k += gridDim.x) {
        const int pk = A.first_pack + k;
        const int qb = A.q_pb[pk], qe = A.q_pe[pk], m = qe - qb;
        __syncthreads();  // rows of the previous pack are no longer read
        if (m > 64)
            continue;     // k_features handles large packs
        for (int e = t; e < m * dp; e += blockDim.x)
            rows[(e / dp) * ld + e % dp] = X[(size_t)qb * dp + e];
        __syncthreads();
        const int i = t >> 2, j0 = t & 3;
        const int p = qb + i;
        const int cl = A.pcl ? A.pcl[min(p, qe - 1)] : -1;
        const float eps = cl >= 0 ? A.ct[cl].feps : A.eps;
        int c1 = 0, c2 = 0, ch = 0;
        float sum = 0.f, dmin = 4.f * eps;
        if (i < m)
            for (int j = j0; j < m; j += 4) {
                if (j == i)
                    continue;
                const float *a = rows + i * ld, *b = rows + j * ld;
                float acc = 0.f;
                for (int c = 0; c < dp; ++c) {
                    const float d = a[c] - b[c];
                    acc = fmaf(d, d, acc);
                }
                const float d = key_to_dist<M>(acc);
                c1 += d <= eps;
                c2 += d <= 2.f * eps;
                ch += d <= 0.5f * eps;
                sum += fminf(d, 16.f * eps);
                dmin = fminf(dmin, d);
            }
        // the four threads of a point are adjacent lanes
#pragma unroll
        for (int o = 1; o < 4; o <<= 1) {
            c1 += __shfl_xor(c1, o, WAVE);
            c2 += __shfl_xor(c2, o, WAVE);
            ch += __shfl_xor(ch, o, WAVE);
            sum += __shfl_xor(sum, o, WAVE);
            dmin = fminf(dmin, __shfl_xor(dmin, o, WAVE));
        }
        if (i < m && j0 == 0) {
            float *f = feat + (size_t)p * MLP_F;
            f[8] = log1pf((float)c1) / 6.f;
            f[9] = log1pf((float)c2) / 6.f;
            f[10] = log1pf((float)ch) / 6.f;
            f[11] = sum / ((float)max(m - 1, 1) * eps);
            f[15] = dmin / eps;
        }
    }
}

// ------------------------------------------------------------------ MLP --
//
// Both directions run on the FP32 matrix instructions (operands, products and
// sums in FP32).  A wave takes MT = 32 samples as the 32 columns of
// v_mfma_f32_32x32x2_f32 products Z^T = W X^T: in the result a lane holds
// sample lane % 32 and, in register r of tile t, neuron
// 32 t + 8 (r / 4) + 4 (lane / 32) + r % 4.  That register is, as it stands,
// the other operand of the next layer's product for the pair of k values
// (n, n + 4) of its two lane halves, so activations and their gradients pass
// from layer to layer without leaving the registers; only the operand read
// from the weights follows that order of k.  The weight gradients contract
// over the samples instead: there a wave turns one 64 x 32 array at a time
// through its LDS tile (row stride 33: both sides free of bank conflicts).
//
// What bounds it: 80 (forward) or 272 (with the gradient) matrix
// instructions of 64 cycles per 32 samples against 64 logistic functions per
// lane.  1M samples, against one sample per thread on the vector units (the
// gradient with 32 of 256 threads in its forward part): forward 0.847 -> 0.212
// ms, gradient 9.63 -> 0.50 ms (60 TFLOP/s; the matrix instructions alone
// 0.18 ms), error against FP64 2.5e-7 -> 2.1e-7 and 2.2e-6 -> 8.5e-8.
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4u __attribute__((ext_vector_type(4), aligned(4)));  // 4-byte aligned rows

constexpr int MT = 32;                             // samples of a wave's tile
constexpr int LW1 = MLP_F + 1, LW2 = MLP_H + 1;    // LDS row strides of the weights
constexpr int LT = MT + 1;                         // and of the turned arrays
static_assert(MLP_F == 16 && MLP_H == 64 && MLP_O == 2, "tile layout");

struct MlpW {
    float w1[MLP_H * LW1], w2[MLP_H * LW2];
    __align__(16) float w3[MLP_O * MLP_H];
    __align__(16) float b1[MLP_H];
    __align__(16) float b2[MLP_H];
    float b3[MLP_O];
};

__device__ __forceinline__ void mlp_stage(const float *__restrict__ th, MlpW &w)
{
    for (int i = threadIdx.x; i < MLP_NPAR; i += blockDim.x) {
        const float v = th[i];
        if (i < OB1)
            w.w1[(i / MLP_F) * LW1 + i % MLP_F] = v;
        else if (i < OW2)
            w.b1[i - OB1] = v;
        else if (i < OB2)
            w.w2[((i - OW2) / MLP_H) * LW2 + (i - OW2) % MLP_H] = v;
        else if (i < OW3)
            w.b2[i - OB2] = v;
        else if (i < OB3)
            w.w3[i - OW3] = v;
        else
            w.b3[i - OB3] = v;
    }
    __syncthreads();
}

// One wave's LDS accesses complete in order: only the compiler must keep
// reads after writes (and the next writes after them).
__device__ __forceinline__ void lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// The same value, which the compiler takes for a new one: LDS addresses
// formed from it are formed where they are used, not held in registers from
// phase to phase (there are more of them than registers).
__device__ __forceinline__ int fresh(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// z[2] of a 64-neuron layer: the bias in the result's layout.
__device__ __forceinline__ void mlp_bias(const float *b, int half, v16f (&z)[2])
{
    half = fresh(half);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const float4 v = *reinterpret_cast<const float4 *>(b + 32 * t + 8 * a + 4 * half);
            z[t][4 * a] = v.x;
            z[t][4 * a + 1] = v.y;
            z[t][4 * a + 2] = v.z;
            z[t][4 * a + 3] = v.w;
        }
}

// z += W1 x for the lane's sample (x: inputs 8 half .. 8 half + 7).
__device__ __forceinline__ void mlp_layer1(const MlpW &w, const float (&x)[8], int col,
                                           int half, v16f (&z)[2])
{
    col = fresh(col);
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int t = 0; t < 2; ++t)
            z[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                w.w1[(32 * t + col) * LW1 + 8 * half + k], x[k], z[t], 0, 0, 0);
}

// z += W2 h (TR: z += W2^T h).
template <bool TR>
__device__ __forceinline__ void mlp_layer2(const MlpW &w, const v16f (&h)[2], int col,
                                           int half, v16f (&z)[2])
{
    col = fresh(col);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int k = 32 * u + 8 * (r / 4) + r % 4 + 4 * half;
#pragma unroll
            for (int t = 0; t < 2; ++t)
                z[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                    w.w2[TR ? k * LW2 + 32 * t + col : (32 * t + col) * LW2 + k], h[u][r],
                    z[t], 0, 0, 0);
            if (r % 4 == 3)  // weights for a few products at a time, not all 64
                __builtin_amdgcn_sched_barrier(0);
        }
}

// Output o of the lane's sample, the same in both halves.
__device__ __forceinline__ float mlp_out(const MlpW &w, const v16f (&h)[2], int half, int o)
{
    half = fresh(half);
    float y = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const float4 v = *reinterpret_cast<const float4 *>(w.w3 + o * MLP_H + 32 * t +
                                                               8 * a + 4 * half);
            y = fmaf(v.x, h[t][4 * a], y);
            y = fmaf(v.y, h[t][4 * a + 1], y);
            y = fmaf(v.z, h[t][4 * a + 2], y);
            y = fmaf(v.w, h[t][4 * a + 3], y);
        }
    return y + __shfl_xor(y, 32, WAVE) + w.b3[o];
}

// y = W3 silu(W2 silu(W1 x + b1) + b2) + b3, 32 samples per wave.
__global__ void __launch_bounds__(256)
k_mlp_fwd(const float *__restrict__ th, const float *__restrict__ X, long long n,
          float *__restrict__ Y)
{
    __shared__ MlpW w;
    mlp_stage(th, w);
    const int lane = threadIdx.x & (WAVE - 1), col = lane & 31, half = lane >> 5;
    const long long tiles = (n + MT - 1) / MT, wpb = blockDim.x / WAVE;
    for (long long q = (long long)blockIdx.x * wpb + threadIdx.x / WAVE; q < tiles;
         q += (long long)gridDim.x * wpb) {
        const long long s = q * MT + col;
        const bool in = s < n;
        const v4u *xr = reinterpret_cast<const v4u *>(X + (in ? s : n - 1) * MLP_F + 8 * half);
        const v4u xa = xr[0], xb = xr[1];
        const float x[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
        v16f z1[2], z2[2];
        asm volatile("" ::: "memory");  // the weights stay in LDS, not in registers
        mlp_bias(w.b1, half, z1);
        mlp_layer1(w, x, col, half, z1);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                z1[t][r] = silu(z1[t][r]);
        mlp_bias(w.b2, half, z2);
        mlp_layer2<false>(w, z1, col, half, z2);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                z2[t][r] = silu(z2[t][r]);
        const float y0 = mlp_out(w, z2, half, 0), y1 = mlp_out(w, z2, half, 1);
        if (in)  // the lower half writes y0, the upper y1
            Y[s * 2 + half] = half ? y1 : y0;
    }
}

// Gradient of the loss over the samples idx[0..B) (or 0..B if idx is NULL):
// work-group b writes its waves' sum to row b of part ([gridDim][NPAR]) and
// its loss to ploss[b], in a fixed order; k_mlp_grad_reduce adds the rows.
// A wave keeps the whole gradient in its registers over all its tiles (the
// 64 x 64 block as four 32 x 32 results, the 64 x 16 one as four 16 x 16).
// NW = 4 waves, one per SIMD, share one copy of the weights: two per SIMD
// would halve the registers, and the 81 that then spill cost more than the
// second wave hides (1M samples: 0.55 against 0.50 ms).  NW = 1 is for few
// tiles, one per work-group, where spreading over the CUs counts (4096
// samples, whole call: 178 -> 61 us).
template <int NW>
__global__ void __launch_bounds__(NW *WAVE)
k_mlp_grad(const float *__restrict__ th, const float *__restrict__ X,
           const float *__restrict__ T, const int32_t *__restrict__ idx, long long B,
           float invB, float *__restrict__ part, double *__restrict__ ploss)
{
    constexpr int SLOTS = NW / 2;  // partial gradients in LDS while the waves' are added
    constexpr int POOL = 2 * NW * MLP_H * LT;
    static_assert(POOL >= SLOTS * MLP_NPAR, "slots fit the tiles' space");
    __shared__ MlpW w;
    __shared__ float pool[POOL];
    __shared__ double wl[NW];
    mlp_stage(th, w);
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    const int col = lane & 31, half = lane >> 5, c16 = lane & 15, q16 = lane >> 4;
    // this wave's tiles, [neuron][sample]: h1 (kept out of the registers from
    // layer 2 to the W2 gradient), and the others one after another
    float *t1 = pool + 2 * wv * MLP_H * LT, *tt = t1 + MLP_H * LT;
    v16f g2[2][2] = {};                  // W2: rows 32 i .., columns 32 j ..
    v4f g1[4] = {};                      // W1: rows 16 i ..
    float gb1[4] = {}, gb2[2] = {}, g3[2] = {}, gb3[2] = {};
    double lsum = 0.0;
    auto turn = [&](float *tt, const v16f (&v)[2]) {
        lds_order();
        const int c = fresh(col);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                tt[(32 * t + 8 * (r / 4) + r % 4 + 4 * half) * LT + c] = v[t][r];
        lds_order();
    };
    const long long tiles = (B + MT - 1) / MT;
    for (long long q = (long long)blockIdx.x * NW + wv; q < tiles;
         q += (long long)gridDim.x * NW) {
        const long long b0 = q * MT;
        const int ns = (int)std::min<long long>(MT, B - b0);
        const bool in = col < ns;
        const long long at = b0 + (in ? col : 0);
        const long long s = idx ? (long long)idx[at] : at;  // idx: below 2^31
        // samples past the end: zero inputs and a zero output gradient
        float x[8], xc[8];
        {
            const v4u *xr = reinterpret_cast<const v4u *>(X + s * MLP_F + 8 * half);
            const v4u xa = xr[0], xb = xr[1];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                x[k] = in ? xa[k] : 0.f;
                x[4 + k] = in ? xb[k] : 0.f;
            }
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {  // input c16 of sample 4 k + q16
            const int j = 4 * k + q16;
            const int d = __shfl((int)(s - b0), j, WAVE);  // of a valid sample
            const float v = X[(b0 + d) * MLP_F + c16];
            xc[k] = j < ns ? v : 0.f;
        }
        v16f h1[2], d1[2], h2[2], d2[2];
        asm volatile("" ::: "memory");  // the weights stay in LDS, not in registers
        mlp_bias(w.b1, half, h1);
        mlp_layer1(w, x, col, half, h1);
        mlp_bias(w.b2, half, h2);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float z = h1[t][r], g = 1.f / (1.f + expf(-z));
                h1[t][r] = z * g;
                d1[t][r] = g * (1.f + z * (1.f - g));
                if (r % 4 == 3)
                    __builtin_amdgcn_sched_barrier(0);
            }
        turn(t1, h1);
        mlp_layer2<false>(w, h1, col, half, h2);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float z = h2[t][r], g = 1.f / (1.f + expf(-z));
                h2[t][r] = z * g;
                d2[t][r] = g * (1.f + z * (1.f - g));
                if (r % 4 == 3)
                    __builtin_amdgcn_sched_barrier(0);
            }
        const float e0 = mlp_out(w, h2, half, 0) - T[s * 2];
        const float e1 = mlp_out(w, h2, half, 1) - T[s * 2 + 1];
        const float gy0 = in ? e0 * invB : 0.f, gy1 = in ? e1 * invB : 0.f;
        if (in && !half) {
            lsum += 0.5 * ((double)e0 * e0 + (double)e1 * e1);
            gb3[0] += gy0;
            gb3[1] += gy1;
        }
        // W3: neuron = lane, the samples one after another
        turn(tt, h2);
        const int ln = fresh(lane);
#pragma unroll
        for (int j = 0; j < MT; ++j) {
            const float v = tt[ln * LT + j];
            g3[0] = fmaf(__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(gy0), j)), v,
                         g3[0]);
            g3[1] = fmaf(__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(gy1), j)), v,
                         g3[1]);
            if (j % 8 == 7)
                __builtin_amdgcn_sched_barrier(0);
        }
        // d2 <- the gradient at z2
        const int hf = fresh(half);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = 32 * t + 8 * (r / 4) + r % 4 + 4 * hf;
                d2[t][r] *= w.w3[k] * gy0 + w.w3[MLP_H + k] * gy1;
            }
        // W2: rows from the gradient at z2, columns from h1
        turn(tt, d2);
        float a2[2][16];
        const int ca = fresh(col), ch = fresh(col), cd = fresh(c16);
#pragma unroll
        for (int k = 0; k < 16; ++k)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                a2[t][k] = tt[(32 * t + ca) * LT + 2 * k + half];
                gb2[t] += a2[t][k];
            }
#pragma unroll
        for (int k = 0; k < 16; ++k)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float v = t1[(32 * j + ch) * LT + 2 * k + half];
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    g2[i][j] =
                        __builtin_amdgcn_mfma_f32_32x32x2f32(a2[i][k], v, g2[i][j], 0, 0, 0);
                if (k % 4 == 3 && j == 1)
                    __builtin_amdgcn_sched_barrier(0);
            }
        // d1 <- the gradient at z1
        v16f gh[2] = {};
        mlp_layer2<true>(w, d2, col, half, gh);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                d1[t][r] *= gh[t][r];
        __builtin_amdgcn_sched_barrier(0);
        turn(tt, d1);
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float v = tt[(16 * i + cd) * LT + 4 * k + q16];
                gb1[i] += v;
                g1[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, xc[k], g1[i], 0, 0, 0);
                if (i == 3)
                    __builtin_amdgcn_sched_barrier(0);
            }
    }
    // x = f(parameter, x) for every parameter's sum x of this wave, each held
    // by one lane
    auto each = [&](auto f) {
        auto put = [&](int i, auto &v, int r) { v[r] = f(i, v[r]); };
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    put(OW2 + (32 * i + 8 * (r / 4) + r % 4 + 4 * half) * MLP_H + 32 * j + col,
                        g2[i][j], r);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                put(OW1 + (16 * i + 4 * q16 + r) * MLP_F + c16, g1[i], r);
#pragma unroll
        for (int o = 0; o < 2; ++o)
            put(OW3 + o * MLP_H + lane, g3, o);
        if (lane < 32)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                put(OB2 + 32 * i + col, gb2, i);
        if (lane < 16)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                put(OB1 + 16 * i + c16, gb1, i);
        if (lane == 0)
#pragma unroll
            for (int o = 0; o < 2; ++o)
                put(OB3 + o, gb3, o);
    };
#pragma unroll
    for (int i = 0; i < 2; ++i)
        gb2[i] += __shfl_xor(gb2[i], 32, WAVE);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        gb1[i] += __shfl_xor(gb1[i], 16, WAVE);
        gb1[i] += __shfl_xor(gb1[i], 32, WAVE);
    }
#pragma unroll
    for (int o = 0; o < 2; ++o)
        gb3[o] = wave_sum(gb3[o]);
    lsum = wave_sum(lsum);
    if (lane == 0)
        wl[wv] = lsum;
#pragma unroll
    for (int m = NW / 2; m >= 1; m >>= 1) {
        __syncthreads();  // the tiles, or the slots of the last step, are consumed
        if (wv >= m && wv < 2 * m) {
            float *p = pool + (wv - m) * MLP_NPAR;
            each([&](int i, float v) { return p[i] = v; });
        }
        __syncthreads();
        if (wv < m) {
            const float *p = pool + wv * MLP_NPAR;
            each([&](int i, float v) { return v + p[i]; });
        }
    }
    if (wv == 0) {
        float *p = part + (size_t)blockIdx.x * MLP_NPAR;
        each([&](int i, float v) { return p[i] = v; });
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < NW; ++i)
            t += wl[i];
        ploss[blockIdx.x] = t;
    }
}

// Fixed-order sums of the per-work-group partials: grad[p] = sum over g of
// part[g][p], four rows at a time per work-group of 64 parameters; *loss =
// (sum over g of ploss[g]) / n, or added to *loss undivided when n is 0.
__global__ void __launch_bounds__(256)
k_mlp_grad_reduce(const float *__restrict__ part, const double *__restrict__ ploss,
                  int groups, long long n, float *__restrict__ grad,
                  double *__restrict__ loss)
{
    __shared__ float s[4][WAVE];
    const int lane = threadIdx.x & (WAVE - 1), q = threadIdx.x / WAVE;
    const int p = blockIdx.x * WAVE + lane;
    float g = 0.f;
    if (p < MLP_NPAR) {
#pragma unroll 8
        for (int k = q; k < groups; k += 4)
            g += part[(size_t)k * MLP_NPAR + p];
    }
    s[q][lane] = g;
    __syncthreads();
    if (q == 0 && p < MLP_NPAR)
        grad[p] = (s[0][lane] + s[1][lane]) + (s[2][lane] + s[3][lane]);
    if (blockIdx.x == 0 && q == 1) {
        double t = 0.0;
        for (int k = lane; k < groups; k += WAVE)
            t += ploss[k];
        t = wave_sum(t);
        if (lane == 0)
            *loss = n > 0 ? t / (double)n : *loss + t;
    }
}

// Adam (Kingma & Ba), bias-corrected; step counts from 1.
__global__ void k_adam(float *__restrict__ th, const float *__restrict__ g,
                       float *__restrict__ m, float *__restrict__ v, int n,
                       float lr, float b1, float b2, float eps, float c1,
                       float c2)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float mh = mi / c1, vh = vi / c2;
        th[i] -= lr * mh / (sqrtf(vh) + eps);
    }
}

// SplitMix64 (Steele, Lea, Flood 2014) keys for a seeded shuffle.
__global__ void k_shuffle_keys(long long n, unsigned long long seed,
                               uint32_t *__restrict__ key, uint32_t *__restrict__ val)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        unsigned long long z = seed + 0x9E3779B97F4A7C15ull * (unsigned long long)(i + 1);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z = z ^ (z >> 31);
        key[i] = (uint32_t)(z >> 32);
        val[i] = (uint32_t)i;
    }
}

// ------------------------------------------------------------ host side --

// At most this many rows of partial gradients: a work-group of four waves
// per CU for many samples, one wave per work-group while the tiles are no
// more than the CUs.
constexpr int GRAD_GROUPS = 256;

static int grad_groups(long long B)
{
    const long long tiles = cdiv(std::max<long long>(B, 1), MT);
    return tiles <= GRAD_GROUPS ? (int)tiles
                                : (int)std::min<long long>(cdiv(tiles, 4), GRAD_GROUPS);
}

// Partial gradients and losses of B samples into grad_groups(B) rows.
static void grad_rows(const float *theta, const float *X, const float *T,
                      const int32_t *idx, long long B, float *part, double *ploss,
                      hipStream_t s)
{
    const int groups = grad_groups(B);
    const float invB = B > 0 ? 1.0f / (float)B : 0.f;
    if (cdiv(std::max<long long>(B, 1), MT) <= GRAD_GROUPS)
        FNN_LAUNCH(k_mlp_grad<1>, dim3(groups), dim3(WAVE), 0, s, theta, X, T, idx, B, invB,
                   part, ploss);
    else
        FNN_LAUNCH(k_mlp_grad<4>, dim3(groups), dim3(4 * WAVE), 0, s, theta, X, T, idx, B,
                   invB, part, ploss);
}

static void grad_reduce(const float *part, const double *ploss, int groups, long long n,
                        float *grad, double *loss, hipStream_t s)
{
    FNN_LAUNCH(k_mlp_grad_reduce, dim3((unsigned)cdiv(MLP_NPAR, WAVE)), dim3(4 * WAVE), 0, s,
               part, ploss, groups, n, grad, loss);
}

void mlp_forward(const float *theta, const float *X, long long n, float *Y,
                 hipStream_t s)
{
    if (n <= 0)
        return;
    FNN_LAUNCH(k_mlp_fwd, dim3(grid_cap(cdiv(n, MT), 4, 1024)), dim3(256), 0, s, theta, X, n,
               Y);
}

double mlp_loss_grad(const float *theta, const float *X, const float *T,
                     long long n, float *grad, Scratch &S)
{
    hipStream_t s = S.stream();
    if (n <= 0) {
        fill(grad, 0.f, MLP_NPAR, s);
        FNN_HIP(hipStreamSynchronize(s));
        return 0.0;
    }
    double *loss = S.get<double>(1), *ploss = S.get<double>(GRAD_GROUPS);
    float *part = S.get<float>((size_t)GRAD_GROUPS * MLP_NPAR);
    grad_rows(theta, X, T, nullptr, n, part, ploss, s);
    grad_reduce(part, ploss, grad_groups(n), n, grad, loss, s);
    return read_scalar(loss, s);
}

void mlp_train(float *theta, const float *X, const float *T, long long n,
               int epochs, int batch, float lr, unsigned long long seed,
               double *epoch_loss, Scratch &S)
{
    hipStream_t s = S.stream();
    if (n <= 0 || epochs <= 0)
        return;
    if (batch <= 0)
        batch = 4096;
    float *g = S.get<float>(MLP_NPAR), *m = S.get<float>(MLP_NPAR),
          *v = S.get<float>(MLP_NPAR);
    fill(m, 0.f, MLP_NPAR, s);
    fill(v, 0.f, MLP_NPAR, s);
    double *loss = S.get<double>(1), *ploss = S.get<double>(GRAD_GROUPS);
    float *part = S.get<float>((size_t)GRAD_GROUPS * MLP_NPAR);
    uint32_t *k1 = S.get<uint32_t>(n), *v1 = S.get<uint32_t>(n);
    uint32_t *k2 = S.get<uint32_t>(n), *perm = S.get<uint32_t>(n);
    const float b1 = 0.9f, b2 = 0.999f, ae = 1e-8f;
    long long step = 0;
    for (int ep = 0; ep < epochs; ++ep) {
        FNN_LAUNCH(k_shuffle_keys, dim3(grid_for(n, 256)), dim3(256), 0, s, n,
                   seed + 0x1234567ull * (unsigned long long)(ep + 1), k1, v1);
        radix_sort_pairs(k1, v1, k2, perm, n, 32, S);
        fill(loss, 0.0, 1, s);
        for (long long b0 = 0; b0 < n; b0 += batch) {
            const long long B = std::min<long long>(batch, n - b0);
            grad_rows(theta, X, T, (const int32_t *)(perm + b0), B, part, ploss, s);
            grad_reduce(part, ploss, grad_groups(B), 0, g, loss, s);
            ++step;
            const float c1 = 1.f - powf(b1, (float)step);
            const float c2 = 1.f - powf(b2, (float)step);
            FNN_LAUNCH(k_adam, dim3(grid_for(MLP_NPAR, 256)), dim3(256), 0, s,
                       theta, g, m, v, MLP_NPAR, lr, b1, b2, ae, c1, c2);
        }
        if (epoch_loss)
            epoch_loss[ep] = read_scalar(loss, s) / (double)n;
    }
    FNN_HIP(hipStreamSynchronize(s));
}

// ------------------------------------------- allocation-free gradient --
//
// fnn_mlp_loss_grad_noalloc keeps its partial sums in a fixed device array
// instead of scratch memory from the pool: NA_GROUPS rows of per-work-group
// partial gradients, then NA_GROUPS partial losses (doubles).  Host code
// never passes `scratch` itself to a kernel (in host code the name is a
// stand-in, not a device address); it uses the address that
// hipGetSymbolAddress returns, looked up once per device.
constexpr int NA_GROUPS = GRAD_GROUPS;
constexpr size_t NA_GRAD_BYTES = sizeof(float) * (size_t)NA_GROUPS * MLP_NPAR;
constexpr size_t NA_BYTES = NA_GRAD_BYTES + sizeof(double) * NA_GROUPS;
static_assert(NA_GRAD_BYTES % alignof(double) == 0, "loss partials alignment");
static __device__ __align__(256) unsigned char scratch[NA_BYTES];

static std::mutex g_na_mu;
static void *g_na_ptr[64] = {nullptr};

static unsigned char *noalloc_scratch()
{
    int dev = 0;
    FNN_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64)
        fail(FNN_EUNSUPPORTED, "device id %d", dev);
    std::lock_guard<std::mutex> lk(g_na_mu);
    if (!g_na_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            fail(FNN_EHIP, "hipGetSymbolAddress(scratch) failed: %s",
                 hipGetErrorString(e));
        g_na_ptr[dev] = p;
    }
    return static_cast<unsigned char *>(g_na_ptr[dev]);
}

size_t mlp_noalloc_scratch_bytes() { return NA_BYTES; }

void mlp_loss_grad_noalloc(const float *theta, const float *X, const float *T,
                           long long n, float *grad, double *loss, hipStream_t s)
{
    unsigned char *base = noalloc_scratch();
    float *part = reinterpret_cast<float *>(base);
    double *ploss = reinterpret_cast<double *>(base + NA_GRAD_BYTES);
    // every work-group writes the whole of its own row, so no clear is needed
    // before the launch; the reduction reads exactly `groups` rows
    const int groups = grad_groups(n);
    if (groups < 1 || groups > NA_GROUPS)
        fail(FNN_EINTERNAL, "gradient work-groups out of range");
    if (n > 0)
        grad_rows(theta, X, T, nullptr, n, part, ploss, s);
    grad_reduce(part, ploss, n > 0 ? groups : 0, std::max<long long>(n, 1), grad, loss, s);
}

void tree_aux(fnn_tree *T, Scratch &S)
{
    hipStream_t s = S.stream();
    const int nn = (int)T->nnodes, n = (int)T->n;
    if (T->parent)
        return;
    T->parent = (int32_t *)T->own(sizeof(int32_t) * nn);
    T->depth_v = (int32_t *)T->own(sizeof(int32_t) * nn);
    T->leaf_of = (int32_t *)T->own(sizeof(int32_t) * n);
    T->pack_of = (int32_t *)T->own(sizeof(int32_t) * n);
    FNN_LAUNCH(k_parent, dim3(grid_for(nn, 256)), dim3(256), 0, s, T->child_begin,
               T->child_count, nn, T->parent);
    if (T->ncloud > 1)  // cloud roots are roots: the virtual vertex 0 is no parent
        fill(T->parent + 1, -1, T->ncloud, s);
    FNN_LAUNCH(k_depth, dim3(grid_for(nn, 256)), dim3(256), 0, s, T->parent, nn,
               T->depth_v);
    FNN_LAUNCH(k_owner, dim3(grid_for(nn, 4)), dim3(256), 0, s, T->pt_begin,
               T->pt_end, T->child_count, 0, nn, 1, T->leaf_of);
    FNN_LAUNCH(k_owner, dim3(grid_for(T->npacks, 4)), dim3(256), 0, s,
               T->q_pt_begin, T->q_pt_end, T->q_kcnt, (int)T->nnodes,
               (int)T->npacks, 0, T->pack_of);
}

void compute_features(const fnn_tree *T, const Pts &P, float eps,
                      const CloudThr *ct, float *feat, hipStream_t s)
{
    FeatArgs A;
    A.pack_of = T->pack_of;
    A.leaf_of = T->leaf_of;
    A.parent = T->parent;
    A.depth = T->depth_v;
    A.center_pos = T->center_pos;
    A.radius = T->radius;
    A.pb = T->pt_begin;
    A.pe = T->pt_end;
    A.ccnt = T->child_count;
    A.q_cpos = T->q_center_pos;
    A.q_rad = T->q_radius;
    A.q_pb = T->q_pt_begin;
    A.q_pe = T->q_pt_end;
    A.eps = eps;
    A.ct = ct;
    A.pcl = ct ? T->pcl : nullptr;
    A.first_pack = (int)T->nnodes;
    A.npacks = (int)T->npacks;
    const dim3 g(grid_for(T->n, 256));
    const bool vec = T->metric == M_L2 || T->metric == M_ANG;
    // vector rows of at most 128 floats: the pack sample from LDS; larger
    // packs (duplicates) are still taken by k_features, which then writes
    // every feature of their points
    const int local = vec && T->dp <= LOC_MAXD;
    switch (T->metric) {
    case M_L2:
        FNN_LAUNCH((k_features<M_L2>), g, dim3(256), 0, s, P, A, local, feat);
        break;
    case M_ANG:
        FNN_LAUNCH((k_features<M_ANG>), g, dim3(256), 0, s, P, A, local, feat);
        break;
    case M_HAM:
        FNN_LAUNCH((k_features<M_HAM>), g, dim3(256), 0, s, P, A, 0, feat);
        break;
    default:
        FNN_LAUNCH((k_features<M_LEV>), g, dim3(256), 0, s, P, A, 0, feat);
        break;
    }
    if (local) {
        const dim3 gp(grid_cap(T->npacks, 1, 16384));
        if (T->metric == M_L2)
            FNN_LAUNCH((k_pack_local<M_L2>), gp, dim3(256), 0, s, P, A, feat);
        else
            FNN_LAUNCH((k_pack_local<M_ANG>), gp, dim3(256), 0, s, P, A, feat);
    }
}

}  // namespace fnn
