// Kernels of the learned warm start: a 3D encoder-decoder CNN trained and run on the GPU.
//
// MFMA operands are BF16 (v_mfma_f32_16x16x16bf16_1k) or FP32 (v_mfma_f32_16x16x4f32), accumulation FP32,
// activations stored FP32. Lane layout (checked on gfx950): A(row = lane%16, k = KL*(lane/16) + e),
// B(k = KL*(lane/16) + e, col = lane%16), accumulator register r = D(row = 4*(lane/16) + r, col = lane%16),
// KL = 4 (bf16) or 1 (f32).
//   * 27-tap layers: direct convolution from LDS tiles (k_conv_direct; the data gradient is the same kernel
//     with mirrored, transposed weights) and a direct weight-gradient kernel (k_wgrad_direct);
//   * the 1x1x1 head: one MFMA per 16 voxels (k_head, both directions) and a reduction for its weight gradient
//     (k_wgrad_1x1).
// Also: bias add + ReLU in the epilogues, bias gradient, ReLU backward, 2x average pooling and nearest
// upsampling (both directions), MSE loss, Adam, the network input from the solver's arrays, and the trilinear
// or cubic prolongation of a coarse prediction to the solver's grid.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "helm_internal.h"

namespace helm {

namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

struct bf16 { unsigned short u; };

__device__ __forceinline__ unsigned short f2bf(float f) {   // round to nearest even
    unsigned u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (unsigned short)(u >> 16);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

template <typename T> struct MT;
template <> struct MT<float> {
    static constexpr int KL = 1;
    typedef float op;
    __device__ static float cvt(float f) { return f; }
    __device__ static v4f mma(op a, op b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};
template <> struct MT<bf16> {
    static constexpr int KL = 4;
    typedef v4s op;
    __device__ static bf16 cvt(float f) { bf16 r; r.u = f2bf(f); return r; }
    __device__ static v4f mma(op a, op b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0); }
};

template <typename T> __device__ __forceinline__ typename MT<T>::op load_op(const T *p);
template <> __device__ __forceinline__ float load_op<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ v4s load_op<bf16>(const bf16 *p) {
    v4s r;
    r[0] = (short)p[0].u; r[1] = (short)p[1].u; r[2] = (short)p[2].u; r[3] = (short)p[3].u;
    return r;
}

// The 1x1x1 head (Co, Ci <= 16), forward (bias) and data gradient (mask, with the output's strides: zero where it is not
// positive): out[o][v] = sum_i wt[o][i] in[i][v], one product per 16 voxels. Bound by its bytes. A wave takes 64 voxels; lane
// column j holds voxels 4j to 4j + 3 of its channels, so loads and stores are 16 bytes and product t takes voxel 4j + t
// of every column. V is a multiple of 256. At 4 x 64^3 18 us each way (67 MB at 4.1
// TB/s; as an implicit product staged through LDS 63 us).
template <typename T>
__global__ __launch_bounds__(256) void k_head(const float *__restrict__ in, long long in_bs, int Ci, int V,
                                              const T *__restrict__ wt, int Kp, const float *__restrict__ bias, int Co,
                                              float *__restrict__ out, long long out_bs, const float *__restrict__ mask) {
    constexpr int KL = MT<T>::KL, STEPS = 4 / KL;             // four channels per lane: one product of 16 or four of 4
    const int lane = threadIdx.x & 63, j = lane & 15, grp = lane >> 4;
    const int tiles = V / 256, b = blockIdx.x / tiles;
    const int v = (blockIdx.x - b * tiles) * 256 + (threadIdx.x >> 6) * 64 + 4 * j;
    const float *inb = in + b * in_bs + v;
    float x[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int c = (k / KL) * 4 * KL + KL * grp + k % KL;
        const float4 q = *reinterpret_cast<const float4 *>(inb + (long long)min(c, Ci - 1) * V);
        const float z = c < Ci ? 1.f : 0.f;
        x[k][0] = z != 0.f ? q.x : 0.f; x[k][1] = z != 0.f ? q.y : 0.f;
        x[k][2] = z != 0.f ? q.z : 0.f; x[k][3] = z != 0.f ? q.w : 0.f;
    }
    const long long at = b * out_bs + v;
    float4 mk[4];
    if (mask) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            mk[r] = *reinterpret_cast<const float4 *>(mask + at + (long long)min(4 * grp + r, Co - 1) * V);
    }
    v4f acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = v4f{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const typename MT<T>::op a = load_op<T>(wt + (long long)j * Kp + s * 4 * KL + KL * grp);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            T o[KL];
#pragma unroll
            for (int e = 0; e < KL; ++e) o[e] = MT<T>::cvt(x[s * KL + e][t]);
            acc[t] = MT<T>::mma(a, load_op<T>(o), acc[t]);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = 4 * grp + r;
        if (o >= Co) continue;
        const float bo = bias ? bias[o] : 0.f;
        float4 y = make_float4(acc[0][r] + bo, acc[1][r] + bo, acc[2][r] + bo, acc[3][r] + bo);
        if (mask) {
            y.x = mk[r].x > 0.f ? y.x : 0.f; y.y = mk[r].y > 0.f ? y.y : 0.f;
            y.z = mk[r].z > 0.f ? y.z : 0.f; y.w = mk[r].w > 0.f ? y.w : 0.f;
        }
        *reinterpret_cast<float4 *>(out + at + (long long)o * V) = y;
    }
}

// s + p[i0] + p[i0 + step] + ... (below n) in that order, K loads in flight
template <int K = 8, typename T> __device__ __forceinline__ T sum_strided(const T *__restrict__ p, long long i0, long long n, long long step) {
    T s = 0;
    long long i = i0;
    for (; i + (K - 1) * step < n; i += K * step) {
        T v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = p[i + k * step];
#pragma unroll
        for (int k = 0; k < K; ++k) s += v[k];
    }
    for (; i < n; i += step) s += p[i];
    return s;
}

// db[co] = sum_{b,v} g[b][co][v]: block (co, s) sums slice s of the B V voxels into part[co][s]; a second
// kernel adds the slices in order
constexpr int BG_SLICES = 64;
__global__ __launch_bounds__(256) void k_bias_part(const float *__restrict__ g, long long g_bs, int B, int V,
                                                   float *__restrict__ part) {
    __shared__ float sm[256];
    const int co = blockIdx.x / BG_SLICES, sl = blockIdx.x % BG_SLICES;
    const int NV = B * V;
    const int per = (NV + BG_SLICES - 1) / BG_SLICES;
    const int u0 = sl * per, u1 = u0 + per < NV ? u0 + per : NV;
    float s = 0.f;
    for (int u = u0 + threadIdx.x; u < u1; u += 8 * 256) {    // eight loads in flight, added in order
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int w = min(u + k * 256, u1 - 1), b = w / V;
            v[k] = g[(long long)b * g_bs + (long long)co * V + (w - b * V)];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (u + k * 256 < u1) s += v[k];
    }
    sm[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sm[0];
}
__global__ void k_bias_reduce(const float *__restrict__ part, int Co, float *__restrict__ db) {
    const int co = blockIdx.x * blockDim.x + threadIdx.x;
    if (co >= Co) return;
    db[co] = sum_strided(part + co * BG_SLICES, 0, BG_SLICES, 1);
}

// 2x average pooling and nearest upsampling between a volume of n^3 voxels (parents) and one of (2n)^3 (children), both
// directions; the backward kernels also apply the mask of the ReLU behind them (zero where y is not positive).
// A thread owns W parents along x (two where n is even) and their 8 W children, each row of which is one access: the
// bytes are what bounds them. Before, a thread took one output, its place from 64-bit divisions, and the mask was a pass
// of its own. At 4 x 64^3 in a training step: upsampling 172 -> 36 us, pooling backward 102 -> 50 us, the masks 150 us -> 13 us
// of longer epilogues; the step 2930 -> 2560 us, inference at 64^3 384 -> 352 us.
template <int N> struct FloatN;
template <> struct FloatN<1> { float v[1]; };
template <> struct __attribute__((aligned(8))) FloatN<2> { float v[2]; };
template <> struct __attribute__((aligned(16))) FloatN<4> { float v[4]; };
template <int N> __device__ __forceinline__ FloatN<N> ld(const float *p) { return *reinterpret_cast<const FloatN<N> *>(p); }
template <int N> __device__ __forceinline__ void st(float *p, const FloatN<N> &v) { *reinterpret_cast<FloatN<N> *>(p) = v; }

// this thread's parents: channel and sample, offset within the parents' channel and of the first child; false if none
template <int W> __device__ __forceinline__ bool parents(int n, int C, int &c, int &b, int &po, int &co) {
    const int nx = n / W, per = n * n * nx, nb = (per + 255) / 256;
    const int bc = blockIdx.x / nb, r = (blockIdx.x - bc * nb) * 256 + threadIdx.x;
    c = bc % C;
    b = bc / C;
    const int q = r / nx, x = (r - q * nx) * W, z = q / n, y = q - z * n;
    po = q * n + x;
    co = ((2 * z) * 2 * n + 2 * y) * 2 * n + 2 * x;
    return r < per;
}
// row k (0..3: z and y of the child) of a parent's children
__device__ __forceinline__ int child_row(int n, int k) { return ((k >> 1) * 2 * n + (k & 1)) * 2 * n; }

template <int W>
__global__ __launch_bounds__(256) void k_pool_fwd(const float *__restrict__ in, long long in_bs, float *__restrict__ out,
                                                  long long out_bs, int C, int n) {
    int c, b, po, co;
    if (!parents<W>(n, C, c, b, po, co)) return;
    const float *p = in + b * in_bs + 8LL * c * n * n * n + co;
    FloatN<2 * W> r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = ld<2 * W>(p + child_row(n, k));
    FloatN<W> o;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) { s += r[k].v[2 * w]; s += r[k].v[2 * w + 1]; }
        o.v[w] = 0.125f * s;
    }
    st<W>(out + b * out_bs + (long long)c * n * n * n + po, o);
}
// gin += gout / 8 on the children
template <int W>
__global__ __launch_bounds__(256) void k_pool_bwd(const float *__restrict__ gout, long long gout_bs, float *__restrict__ gin,
                                                  const float *__restrict__ y, long long gin_bs, int C, int n) {
    int c, b, po, co;
    if (!parents<W>(n, C, c, b, po, co)) return;
    const long long at = b * gin_bs + 8LL * c * n * n * n + co;
    const FloatN<W> g = ld<W>(gout + b * gout_bs + (long long)c * n * n * n + po);
    FloatN<2 * W> r[4], m[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        r[k] = ld<2 * W>(gin + at + child_row(n, k));
        m[k] = ld<2 * W>(y + at + child_row(n, k));
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int w = 0; w < 2 * W; ++w) r[k].v[w] = m[k].v[w] > 0.f ? r[k].v[w] + 0.125f * g.v[w / 2] : 0.f;
        st<2 * W>(gin + at + child_row(n, k), r[k]);
    }
}
template <int W>
__global__ __launch_bounds__(256) void k_up_fwd(const float *__restrict__ in, long long in_bs, float *__restrict__ out,
                                                long long out_bs, int C, int n) {
    int c, b, po, co;
    if (!parents<W>(n, C, c, b, po, co)) return;
    const FloatN<W> g = ld<W>(in + b * in_bs + (long long)c * n * n * n + po);
    FloatN<2 * W> r;
#pragma unroll
    for (int w = 0; w < 2 * W; ++w) r.v[w] = g.v[w / 2];
    float *o = out + b * out_bs + 8LL * c * n * n * n + co;
#pragma unroll
    for (int k = 0; k < 4; ++k) st<2 * W>(o + child_row(n, k), r);
}
template <int W>
__global__ __launch_bounds__(256) void k_up_bwd(const float *__restrict__ gout, long long gout_bs, float *__restrict__ gin,
                                                const float *__restrict__ y, long long gin_bs, int C, int n) {
    int c, b, po, co;
    if (!parents<W>(n, C, c, b, po, co)) return;
    const long long at = b * gin_bs + (long long)c * n * n * n + po;
    const float *p = gout + b * gout_bs + 8LL * c * n * n * n + co;
    const FloatN<W> m = ld<W>(y + at);
    FloatN<2 * W> r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = ld<2 * W>(p + child_row(n, k));
    FloatN<W> o;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) { s += r[k].v[2 * w]; s += r[k].v[2 * w + 1]; }
        o.v[w] = m.v[w] > 0.f ? s : 0.f;
    }
    st<W>(gin + at, o);
}

// MSE: partial sums of (y - t)^2 per block and the gradient 2 (y - t) / N
__global__ __launch_bounds__(256) void k_mse(const float *__restrict__ y, const float *__restrict__ t, long long n,
                                             float *__restrict__ g, double *__restrict__ part) {
    __shared__ double sm[256];
    long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    double s = 0.0;
    if (i < n) {
        float d = y[i] - t[i];
        g[i] = 2.f * d / (float)n;
        s = (double)d * d;
    }
    sm[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sm[0];
}
__global__ __launch_bounds__(256) void k_sum_d(const double *__restrict__ part, int np, double *__restrict__ out,
                                               double scale) {
    __shared__ double sm[256];
    sm[threadIdx.x] = sum_strided(part, threadIdx.x, np, 256);
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sm[0] * scale;
}

// Adam on the FP32 master parameters
__global__ void k_adam(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m, float *__restrict__ v,
                       long long n, float lr, float b1, float b2, float eps, float c1, float c2) {
    long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float gi = g[i];
    float mi = b1 * m[i] + (1.f - b1) * gi;
    float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// trilinear interpolation of a coarse prediction (channels Re, Im on nodes (i+1)/(nc+1)) to the fine nodes
// (I+1)/(nf+1), times `scale`, written as complex128. Beyond the outermost coarse nodes the values follow the
// ghost rule of the scheme on the coarse grid, U(-1) = gamma U(0) and U(nc) = gamma U(nc-1) per axis (gamma = 0
// gives zero extension).
__global__ void k_prolong(const float *__restrict__ coarse, int nc, double scale, double gre, double gim,
                          double2 *__restrict__ fine, int nf) {
    long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    long long nfn = (long long)nf * nf * nf;
    if (i >= nfn) return;
    const int F[3] = {(int)(i % nf), (int)((i / nf) % nf), (int)(i / ((long long)nf * nf))};
    int i0[3];
    double w1[3];
    for (int a = 0; a < 3; ++a) {                          // coarse index coordinate (F+1)(nc+1)/(nf+1) - 1
        long long num = (long long)(F[a] + 1) * (nc + 1);
        long long q = num / (nf + 1);
        i0[a] = (int)q - 1;
        w1[a] = (double)(num - q * (nf + 1)) / (nf + 1);
    }
    const long long V = (long long)nc * nc * nc;
    double re = 0.0, im = 0.0;
    for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
            for (int dx = 0; dx < 2; ++dx) {
                const int d[3] = {dx, dy, dz};
                double w = 1.0, fr = 1.0, fi = 0.0;          // weight and ghost factor gamma^(#clamped axes)
                int idx[3];
                for (int a = 0; a < 3; ++a) {
                    w *= d[a] ? w1[a] : 1.0 - w1[a];
                    int c = i0[a] + d[a];
                    if (c < 0 || c >= nc) {
                        c = c < 0 ? 0 : nc - 1;
                        const double nr = fr * gre - fi * gim, ni = fr * gim + fi * gre;
                        fr = nr;
                        fi = ni;
                    }
                    idx[a] = c;
                }
                if (w == 0.0) continue;
                const long long o = ((long long)idx[2] * nc + idx[1]) * nc + idx[0];
                const double ur = coarse[o], ui = coarse[V + o];
                re += w * (fr * ur - fi * ui);
                im += w * (fr * ui + fi * ur);
            }
    fine[i] = make_double2(scale * re, scale * im);
}

// the same prolongation with Keys' cubic convolution (a = -1/2) per axis: coarse indices i0-1 .. i0+2 around
// the fine node; ghost indices -m and nc-1+m (m = 1, 2) fold onto the boundary node with factor gamma^m
__global__ void k_prolong3(const float *__restrict__ coarse, int nc, double scale, double gre, double gim,
                           double2 *__restrict__ fine, int nf) {
    long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    long long nfn = (long long)nf * nf * nf;
    if (i >= nfn) return;
    const int F[3] = {(int)(i % nf), (int)((i / nf) % nf), (int)(i / ((long long)nf * nf))};
    double w[3][4];
    int idx[3][4], pw[3][4];
    for (int a = 0; a < 3; ++a) {
        long long num = (long long)(F[a] + 1) * (nc + 1);
        long long q = num / (nf + 1);
        const int i0 = (int)q - 1;
        const double t = (double)(num - q * (nf + 1)) / (nf + 1), t2 = t * t, t3 = t2 * t;
        w[a][0] = -0.5 * t3 + t2 - 0.5 * t;
        w[a][1] = 1.5 * t3 - 2.5 * t2 + 1.0;
        w[a][2] = -1.5 * t3 + 2.0 * t2 + 0.5 * t;
        w[a][3] = 0.5 * t3 - 0.5 * t2;
        for (int k = 0; k < 4; ++k) {
            int c = i0 - 1 + k, m = 0;
            if (c < 0) { m = -c; c = 0; }
            else if (c >= nc) { m = c - nc + 1; c = nc - 1; }
            idx[a][k] = c;
            pw[a][k] = m;
        }
    }
    double gr[7], gi[7];                                   // gamma^0 .. gamma^6
    gr[0] = 1.0; gi[0] = 0.0;
    for (int m = 1; m < 7; ++m) { gr[m] = gr[m - 1] * gre - gi[m - 1] * gim; gi[m] = gr[m - 1] * gim + gi[m - 1] * gre; }
    const long long V = (long long)nc * nc * nc;
    double re = 0.0, im = 0.0;
    for (int kz = 0; kz < 4; ++kz)
        for (int ky = 0; ky < 4; ++ky)
            for (int kx = 0; kx < 4; ++kx) {
                const double wt = w[0][kx] * w[1][ky] * w[2][kz];
                if (wt == 0.0) continue;
                const int m = pw[0][kx] + pw[1][ky] + pw[2][kz];
                const long long o = ((long long)idx[2][kz] * nc + idx[1][ky]) * nc + idx[0][kx];
                const double ur = coarse[o], ui = coarse[V + o];
                re += wt * (gr[m] * ur - gi[m] * ui);
                im += wt * (gr[m] * ui + gi[m] * ur);
            }
    fine[i] = make_double2(scale * re, scale * im);
}


// Separable form of the cubic prolongation (the 3-D operator is the product of three 1-D ones, ghost factors
// included): pass a interpolates along one axis, from an array [ch][n2][n1][nin] (innermost axis interpolated) to
// [ch][n2][n1][nout] with the output axis rotated to the front: out[ch][nout][n2][n1]. Three passes (x, y, z)
// give [ch][z][y][x] again. Complex data as (re, im) doubles; the first pass reads the FP32 prediction.
template <typename TIN>
__global__ void k_prolong3_pass(const TIN *__restrict__ src, int ncplx_in, int nin, int n1, int n2, int nout,
                                double gre, double gim, double scale, double2 *__restrict__ dst) {
    const long long total = (long long)nout * n1 * n2;
    const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    // output index: [o][a2][a1] (o slowest) so writes are contiguous along a1
    const int a1 = (int)(e % n1), a2 = (int)((e / n1) % n2), o = (int)(e / ((long long)n1 * n2));
    const long long num = (long long)(o + 1) * (nin + 1);
    const long long q = num / (nout + 1);
    const int i0 = (int)q - 1;
    const double t = (double)(num - q * (nout + 1)) / (nout + 1), t2 = t * t, t3 = t2 * t;
    const double w[4] = {-0.5 * t3 + t2 - 0.5 * t, 1.5 * t3 - 2.5 * t2 + 1.0, -1.5 * t3 + 2.0 * t2 + 0.5 * t,
                         0.5 * t3 - 0.5 * t2};
    double re = 0.0, im = 0.0;
    for (int k = 0; k < 4; ++k) {
        if (w[k] == 0.0) continue;
        int c = i0 - 1 + k, m = 0;
        if (c < 0) { m = -c; c = 0; }
        else if (c >= nin) { m = c - nin + 1; c = nin - 1; }
        double fr = 1.0, fi = 0.0;                     // gamma^m
        for (int r = 0; r < m; ++r) { const double nr = fr * gre - fi * gim; fi = fr * gim + fi * gre; fr = nr; }
        const long long si = ((long long)a2 * n1 + a1) * nin + c;
        double ur, ui;
        if (ncplx_in) { const double2 z = ((const double2 *)src)[si]; ur = z.x; ui = z.y; }
        else { ur = (double)((const float *)src)[si]; ui = (double)((const float *)src)[(long long)n1 * n2 * nin + si]; }
        re += w[k] * (fr * ur - fi * ui);
        im += w[k] * (fr * ui + fi * ur);
    }
    dst[e] = make_double2(scale * re, scale * im);
}

// network input from the solver's arrays: node (i, j, l) of the S^3 grid sits at ((i, j, l) + 1)/(S+1) in the unit
// cube, which is fine-grid index coordinate (i+1)(nf+1)/(S+1) - 1 per axis; k^2 and Re f are interpolated
// trilinearly there (weights from integer arithmetic, so nested grids inject exactly). Channel 0 =
// cs (k^2/k0^2 - 1), channel 1 = fs Re f. Arrays carry `halo` >= 1 cells; the upper neighbour index can be nf
// (a halo cell) only with weight zero.
__global__ void k_features(const double *__restrict__ k2h, const double2 *__restrict__ fh, int halo, int nf, int S,
                           double inv_k0sq, double cs, double fs, float *__restrict__ x) {
    long long v = (long long)blockIdx.x * 256 + threadIdx.x;
    const long long V = (long long)S * S * S;
    if (v >= V) return;
    const int c[3] = {(int)(v % S), (int)((v / S) % S), (int)(v / ((long long)S * S))};
    int i0[3];
    double w1[3];
    for (int a = 0; a < 3; ++a) {
        long long num = (long long)(c[a] + 1) * (nf + 1);
        i0[a] = (int)(num / (S + 1)) - 1;
        w1[a] = (double)(num % (S + 1)) / (S + 1);
    }
    const long long P = nf + 2 * halo;
    double k2 = 0.0, fr = 0.0;
    for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
            for (int dx = 0; dx < 2; ++dx) {
                double w = (dx ? w1[0] : 1.0 - w1[0]) * (dy ? w1[1] : 1.0 - w1[1]) * (dz ? w1[2] : 1.0 - w1[2]);
                if (w == 0.0) continue;
                long long o = ((long long)(i0[2] + dz + halo) * P + (i0[1] + dy + halo)) * P + (i0[0] + dx + halo);
                k2 += w * k2h[o];
                fr += w * fh[o].x;
            }
    x[v] = (float)(cs * (k2 * inv_k0sq - 1.0));
    x[V + v] = (float)(fs * fr);
}


// pair (a, b) of operand values as stored
__device__ __forceinline__ unsigned bf_pair(float a, float b) {
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    const v2bf r = {(__bf16)a, (__bf16)b};
    unsigned u;
    __builtin_memcpy(&u, &r, 4);
    return u;
}
__device__ __forceinline__ void st_two(float *p, float a, float b) { p[0] = a; p[1] = b; }
__device__ __forceinline__ void st_two(bf16 *p, float a, float b) { *reinterpret_cast<unsigned *>(p) = bf_pair(a, b); }
__device__ __forceinline__ void st_one(float *p, float a) { *p = a; }
__device__ __forceinline__ void st_one(bf16 *p, float a) { p->u = (unsigned short)bf_pair(a, 0.f); }

// Value, or four consecutive values, of a row of length S from x on, zero where `in` is false or outside the row. The
// loads are unconditional, from the row's start where the value is not wanted: under a branch each would wait for its
// own result before the next is issued. V4: S and x are multiples of 4.
__device__ __forceinline__ float row1(const float *row, int x, int S, bool in) {
    const bool ok = in && (unsigned)x < (unsigned)S;
    const float v = row[ok ? x : 0];
    return ok ? v : 0.f;
}
template <bool V4> __device__ __forceinline__ float4 row4(const float *row, int x, int S, bool in) {
    if constexpr (V4) {
        const bool ok = in && (unsigned)x < (unsigned)S;
        float4 v = *reinterpret_cast<const float4 *>(row + (ok ? x : 0));
        v.x = ok ? v.x : 0.f;
        v.y = ok ? v.y : 0.f;
        v.z = ok ? v.z : 0.f;
        v.w = ok ? v.w : 0.f;
        return v;
    } else {
        return make_float4(row1(row, x, S, in), row1(row, x + 1, S, in), row1(row, x + 2, S, in), row1(row, x + 3, S, in));
    }
}

// ---------------------------------------------------------------------------------------------- direct 3x3x3
// Direct convolution for the 27-tap layers. A workgroup owns a tile of TX x 4 x TZ voxels and FR blocks of 16 output
// channels. Per chunk of 16 input channels the tile with its one-voxel halo is staged once in LDS, channel-last in the
// operand type; a wave owns the four rows of 16-voxel column blocks of a plane and reads, per dz, the 18 operands of
// their six input rows and three shifts, which serve 36 products per row block. Weights are packed as
// wt[chunk][tap][COP][16] and read as A fragments from global memory (512 contiguous bytes that every wave shares).
// The tiles take whole rows (TX = 64, 32 or 16 by the volume's width), so that a 128-byte line is fetched for all of
// its voxels, and a thread stages four voxels of four channels with loads that are all in flight.
// At 4 x 64^3 in BF16: 16 -> 16 channels 73 us (before: 8 x 8 x 4 tiles staged element by element and every product's
// weights waited for, 110 us), 48 -> 16 at 168 us (319 us), 96 -> 32 at 32^3 62 us (168 us); bound by the staging's
// latency and its reads (1.8 TB/s of input at 16 -> 16), not by the products (12 us there).
// Every output's products are added in the order chunk, tap, channel.
constexpr int DCC = 16;                    // input channels per chunk
constexpr int CY = 4, CHY = CY + 2;        // tile height, rows with halo
// LDS place, in groups of four channels, of voxel v (halo at 3 and TX + 4, interior from 4) of a row, quarter q: eight
// bytes of padding after every four voxels spread the staging's stores over the banks
__host__ __device__ constexpr int c_at(int v, int q) { return 4 * v + (v >> 2) + q - 12; }
template <int TX, int TZ> struct ConvTile {
    static constexpr int ROWS = (TZ + 2) * CHY, PITCH = c_at(TX + 4, 3) + 1, QUADS = ROWS * PITCH;
};

// four channels of a voxel in the operand type. BF16: group q holds channels 4q .. 4q + 3, the operand of one product
// over 16 channels. FP32: group q holds channels q, 4 + q, 8 + q, 12 + q, the operands of four products of four.
template <typename T> struct Chan;
template <> struct Chan<bf16> {
    typedef uint2 t;
    __device__ __forceinline__ static int ch(int q, int j) { return 4 * q + j; }
    __device__ __forceinline__ static t make(float a, float b, float c, float d) { return make_uint2(bf_pair(a, b), bf_pair(c, d)); }
    __device__ __forceinline__ static v4f mul(const t &a, const t &b, v4f acc) {
        v4s x, y;
        __builtin_memcpy(&x, &a, 8);
        __builtin_memcpy(&y, &b, 8);
        return MT<bf16>::mma(x, y, acc);
    }
};
template <> struct Chan<float> {
    typedef float4 t;
    __device__ __forceinline__ static int ch(int q, int j) { return 4 * j + q; }
    __device__ __forceinline__ static t make(float a, float b, float c, float d) { return make_float4(a, b, c, d); }
    __device__ __forceinline__ static v4f mul(const t &a, const t &b, v4f acc) {
        acc = MT<float>::mma(a.x, b.x, acc);
        acc = MT<float>::mma(a.y, b.y, acc);
        acc = MT<float>::mma(a.z, b.z, acc);
        return MT<float>::mma(a.w, b.w, acc);
    }
};

// Stage one chunk of the tile at (x0, y0, z0), by NT threads (t = 0 .. NT - 1): units of four voxels and four channels
// of a row, then the halo ends of the rows. nc: channels of the chunk that exist. V4: rows are 16-byte aligned and
// a multiple of four voxels.
template <typename T, int TX, int TZ, int NT, bool V4>
__device__ __forceinline__ void conv_stage_rows(typename Chan<T>::t *sI, const float *in, int nc, int S, int V, int x0,
                                                int y0, int z0, int t) {
    typedef Chan<T> C;
    constexpr int ROWS = ConvTile<TX, TZ>::ROWS, PITCH = ConvTile<TX, TZ>::PITCH, NQ = TX / 4;
    constexpr int NI = ROWS * NQ * 4, NH = ROWS * 2 * 4;
#pragma unroll 3
    for (int p = 0; p < (NI + NT - 1) / NT; ++p) {
        const int u = t + NT * p;
        if (NI % NT && u >= NI) break;
        const int q = u & 3, xq = (u >> 2) % NQ, r = (u >> 2) / NQ;
        const int z = z0 + r / CHY - 1, y = y0 + r % CHY - 1, x = x0 + 4 * xq;
        const bool rin = (unsigned)z < (unsigned)S && (unsigned)y < (unsigned)S;
        const float *row = in + (rin ? ((long long)z * S + y) * S : 0);
        float4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = C::ch(q, j);
            const float *rc = row + (long long)(c < nc ? c : 0) * V;
            v[j] = row4<V4>(rc, x, S, rin && c < nc);
        }
        typename C::t *d = sI + r * PITCH + c_at(4 + 4 * xq, q);
        d[0] = C::make(v[0].x, v[1].x, v[2].x, v[3].x);
        d[4] = C::make(v[0].y, v[1].y, v[2].y, v[3].y);
        d[8] = C::make(v[0].z, v[1].z, v[2].z, v[3].z);
        d[12] = C::make(v[0].w, v[1].w, v[2].w, v[3].w);
    }
#pragma unroll 2
    for (int p = 0; p < (NH + NT - 1) / NT; ++p) {
        const int u = t + NT * p;
        if (NH % NT && u >= NH) break;
        const int q = u & 3, e = (u >> 2) & 1, r = u >> 3;
        const int z = z0 + r / CHY - 1, y = y0 + r % CHY - 1, x = e ? x0 + TX : x0 - 1;
        const bool rin = (unsigned)z < (unsigned)S && (unsigned)y < (unsigned)S;
        const float *row = in + (rin ? ((long long)z * S + y) * S : 0);
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = C::ch(q, j);
            v[j] = row1(row + (long long)(c < nc ? c : 0) * V, x, S, rin && c < nc);
        }
        sI[r * PITCH + c_at(e ? TX + 4 : 3, q)] = C::make(v[0], v[1], v[2], v[3]);
    }
}

template <typename T, int TX, int TZ, int NT>
__device__ __forceinline__ void conv_stage(typename Chan<T>::t *sI, const float *in, int nc, int S, int V, int x0, int y0,
                                           int z0, bool vec, int t) {
    if (vec) conv_stage_rows<T, TX, TZ, NT, true>(sI, in, nc, S, V, x0, y0, z0, t);
    else conv_stage_rows<T, TX, TZ, NT, false>(sI, in, nc, S, V, x0, y0, z0, t);
}

// the products of one dz for the four rows of a column block: b0 the lane's operands of the six input rows (PITCH
// apart) at the three shifts, a the weights of the nine taps
template <typename T, int FR, int PITCH>
__device__ __forceinline__ void conv_dz(v4f (&acc)[FR][4], const typename Chan<T>::t (&a)[9][FR],
                                        const typename Chan<T>::t *b0, const typename Chan<T>::t *b1,
                                        const typename Chan<T>::t *b2) {
    typename Chan<T>::t b[CHY][3];
#pragma unroll
    for (int y = 0; y < CHY; ++y) {
        b[y][0] = b0[y * PITCH];
        b[y][1] = b1[y * PITCH];
        b[y][2] = b2[y * PITCH];
    }
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int y = 0; y < CY; ++y)
#pragma unroll
                for (int f = 0; f < FR; ++f) acc[f][y] = Chan<T>::mul(a[dy * 3 + dx][f], b[y + dy][dx], acc[f][y]);
}

// All chunks by one workgroup of four waves: bias and ReLU in the epilogue, or the mask of a ReLU's backward pass (zero
// where mask, which has the output's strides, is not positive).
template <typename T, int FR, int TX, int TZ>
__global__ __launch_bounds__(256) void k_conv_direct(const float *__restrict__ in, long long in_bs, int Ci, int S,
                                                     const T *__restrict__ wt, int COP, const float *__restrict__ bias,
                                                     int Co, float *__restrict__ out, long long out_bs, int relu,
                                                     const float *__restrict__ mask, int rowgroups, int vec, int blocks) {
    typedef typename Chan<T>::t CT4;
    constexpr int PITCH = ConvTile<TX, TZ>::PITCH, NXB = TX / 16, NJ = NXB * TZ / 4;   // column blocks of a wave
    static_assert(NJ >= 1 && NJ * 4 == NXB * TZ, "four waves share the tile's column blocks");
    __shared__ __attribute__((aligned(16))) CT4 sI[ConvTile<TX, TZ>::QUADS];
    const int ntx = (S + TX - 1) / TX, nty = (S + CY - 1) / CY, ntz = (S + TZ - 1) / TZ;
    const int tiles = ntx * nty * ntz;
    const int per = (blocks + 7) / 8;
    int idx = (blockIdx.x % 8) * per + blockIdx.x / 8;        // neighbouring tiles on one XCD
    if (idx >= blocks) return;
    const int rg = idx % rowgroups;
    idx /= rowgroups;
    const int t = idx % tiles, b = idx / tiles;
    const int x0 = (t % ntx) * TX, y0 = ((t / ntx) % nty) * CY, z0 = (t / (ntx * nty)) * TZ;
    const int row0 = rg * FR * 16;
    const float *inb = in + (long long)b * in_bs;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int V = S * S * S;
    v4f acc[NJ][FR][4];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int f = 0; f < FR; ++f)
#pragma unroll
            for (int y = 0; y < 4; ++y) acc[j][f][y] = v4f{0, 0, 0, 0};
    const CT4 *lb[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) lb[dx] = sI + c_at(3 + (lane & 15) + dx, lane >> 4);
    const int nchunk = (Ci + DCC - 1) / DCC;
    for (int ch = 0; ch < nchunk; ++ch) {
        const CT4 *wc = reinterpret_cast<const CT4 *>(wt + ((long long)ch * 27 * COP + row0 + (lane & 15)) * DCC) + (lane >> 4);
        // the weights of a dz are loaded before the products of the one before (the first: before the tile)
        CT4 a[2][9][FR];
        auto weights = [&](CT4 (&w)[9][FR], int dz) {
#pragma unroll
            for (int k = 0; k < 9; ++k)
#pragma unroll
                for (int f = 0; f < FR; ++f) w[k][f] = wc[((long long)(dz * 9 + k) * COP + f * 16) * (DCC / 4)];
        };
        weights(a[0], 0);
        __syncthreads();
        conv_stage<T, TX, TZ, 256>(sI, inb + (long long)ch * DCC * V, min(DCC, Ci - ch * DCC), S, V, x0, y0, z0, vec != 0, tid);
        __syncthreads();
#pragma unroll
        for (int dz = 0; dz < 3; ++dz) {
            if (dz < 2) weights(a[(dz + 1) & 1], dz + 1);
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int cb = wave * NJ + j, o = (cb / NXB + dz) * CHY * PITCH + (cb % NXB) * (16 * 4 + 4);
                conv_dz<T, FR, PITCH>(acc[j], a[dz & 1], lb[0] + o, lb[1] + o, lb[2] + o);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int cb = wave * NJ + j;
        const int gz = z0 + cb / NXB, gx = x0 + (cb % NXB) * 16 + (lane & 15);
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            const int gy = y0 + y;
            const bool ok = gx < S && gy < S && gz < S;
            const long long at = (long long)b * out_bs + ((long long)gz * S + gy) * S + gx;
            float *o = out + at;
            float mk[FR][4];
            if (FR < 3 && mask) {                             // unconditional loads, all of a row in flight
                const float *m = mask + (ok ? at : 0);
#pragma unroll
                for (int f = 0; f < FR; ++f)
#pragma unroll
                    for (int r = 0; r < 4; ++r) mk[f][r] = m[(long long)min(row0 + f * 16 + 4 * (lane >> 4) + r, Co - 1) * V];
            }
#pragma unroll
            for (int f = 0; f < FR; ++f)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int co = row0 + f * 16 + 4 * (lane >> 4) + r;
                    if (!ok || co >= Co) continue;
                    float v = acc[j][f][y][r] + (bias ? bias[co] : 0.f);
                    if (relu) v = fmaxf(v, 0.f);
                    if (FR < 3 && mask && !(mk[f][r] > 0.f)) v = 0.f;
                    o[(long long)co * V] = v;
                }
        }
    }
}

// The chunks summed in parts, for the levels with few voxels (16 x 4 of one plane and 16 output channels per workgroup):
// part p takes chunks [p cpb, (p + 1) cpb), a wave one part (FP32 operands: two, for the LDS), and the parts are added in
// their order, bias first.
constexpr int PARTS_MAX = 8;
template <typename T> constexpr int deep_per() { return MT<T>::KL == 4 ? 1 : 2; }
template <typename T>
__global__ __launch_bounds__(64 * PARTS_MAX) void k_conv_deep(const float *__restrict__ in, long long in_bs, int Ci, int S,
                                                              const T *__restrict__ wt, int COP,
                                                              const float *__restrict__ bias, int Co,
                                                              float *__restrict__ out, long long out_bs, int relu,
                                                              const float *__restrict__ mask, int rowgroups, int vec, int nsplit, int cpb) {
    typedef typename Chan<T>::t CT4;
    constexpr int TX = 16, TZ = 1, PITCH = ConvTile<TX, TZ>::PITCH, QUADS = ConvTile<TX, TZ>::QUADS, PER = deep_per<T>();
    extern __shared__ __attribute__((aligned(16))) unsigned char dsm[];
    const int ntx = (S + TX - 1) / TX, nty = (S + CY - 1) / CY, tiles = ntx * nty * S;
    int idx = blockIdx.x;
    const int rg = idx % rowgroups;
    idx /= rowgroups;
    const int t = idx % tiles, b = idx / tiles;
    const int x0 = (t % ntx) * TX, y0 = ((t / ntx) % nty) * CY, z0 = t / (ntx * nty);
    const int row0 = rg * 16;
    const float *inb = in + (long long)b * in_bs;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int V = S * S * S;
    CT4 *sI = reinterpret_cast<CT4 *>(dsm) + wave * QUADS;
    v4f acc[PER][1][4];
#pragma unroll
    for (int i = 0; i < PER; ++i)
#pragma unroll
        for (int y = 0; y < 4; ++y) acc[i][0][y] = v4f{0, 0, 0, 0};
    const CT4 *lb[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) lb[dx] = sI + c_at(3 + (lane & 15) + dx, lane >> 4);
    const int nchunk = (Ci + DCC - 1) / DCC;
#pragma unroll
    for (int i = 0; i < PER; ++i)
        for (int k = 0; k < cpb; ++k) {
            const int part = wave * PER + i, ch = part * cpb + k;
            const bool have = part < nsplit && ch < nchunk;
            __syncthreads();
            if (have)
                conv_stage<T, TX, TZ, 64>(sI, inb + (long long)ch * DCC * V, min(DCC, Ci - ch * DCC), S, V, x0, y0, z0, vec != 0, lane);
            __syncthreads();
            if (!have) continue;
            const CT4 *wc = reinterpret_cast<const CT4 *>(wt + ((long long)ch * 27 * COP + row0 + (lane & 15)) * DCC) + (lane >> 4);
#pragma unroll
            for (int dz = 0; dz < 3; ++dz) {
                CT4 a[9][1];
#pragma unroll
                for (int q = 0; q < 9; ++q) a[q][0] = wc[(long long)(dz * 9 + q) * COP * (DCC / 4)];
                conv_dz<T, 1, PITCH>(acc[i], a, lb[0] + dz * CHY * PITCH, lb[1] + dz * CHY * PITCH, lb[2] + dz * CHY * PITCH);
            }
        }
    __syncthreads();
    float *red = reinterpret_cast<float *>(dsm);              // [part][row y][channel][x]
#pragma unroll
    for (int i = 0; i < PER; ++i)
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                red[(((wave * PER + i) * 4 + y) * 16 + 4 * (lane >> 4) + r) * 16 + (lane & 15)] = acc[i][0][y][r];
    __syncthreads();
    for (int e = tid; e < 1024; e += blockDim.x) {
        const int gx = x0 + (e & 15), co = row0 + ((e >> 4) & 15), gy = y0 + (e >> 8);
        if (gx >= S || gy >= S || co >= Co) continue;
        const long long at = (long long)b * out_bs + (long long)co * V + ((long long)z0 * S + gy) * S + gx;
        const float mk = mask ? mask[at] : 1.f;
        float v = bias ? bias[co] : 0.f;
        for (int k = 0; k < nsplit; ++k) v += red[k * 1024 + e];
        if (relu) v = fmaxf(v, 0.f);
        out[at] = mk > 0.f ? v : 0.f;
    }
}

// The operand forms of all layers in one launch (24 launches of 2.6 us took 90 us of a training step).
// 27 taps: direct format wt[chunk][tap][COP][16] (channels in the order of Chan<T>) of a conv with Co outputs and Ci inputs;
// transpose = 1 takes them from a layer W[Ci][Co][27] with the tap mirrored (the data-gradient convolution of that layer).
// 1 tap: wt[COP][Kp], row o, column i, zero-padded.
template <typename T> __global__ __launch_bounds__(256) void k_pack(CnnPackJobs p) {
    int k = 0;
    while (k + 1 < p.n && (int)blockIdx.x >= p.j[k + 1].block0) ++k;
    const CnnPackJob &q = p.j[k];
    const int e = ((int)blockIdx.x - q.block0) * 256 + threadIdx.x;
    if (e >= q.total) return;
    int o, i, tap = 0;
    if (q.taps == 27) {
        const int cc = e % DCC;
        int r = e / DCC;
        o = r % q.COP;
        r /= q.COP;
        tap = r % 27;
        i = r / 27 * DCC + Chan<T>::ch(cc / 4, cc % 4);
    } else {
        o = e / q.Kp;
        i = e % q.Kp;
    }
    float v = 0.f;
    if (o < q.Co && i < q.Ci) v = q.transpose ? q.W[(i * q.Co + o) * q.taps + (q.taps - 1 - tap)] : q.W[(o * q.Ci + i) * q.taps + tap];
    reinterpret_cast<T *>(q.wt)[e] = MT<T>::cvt(v);
}

// Weight gradient of a 27-tap layer, dW[o][i][tap] = sum_{b,v} g[b][o][v] in[b][i][v + off(tap)]. Per tap this is a
// product with M = output channels, N = 16 input channels and K = voxels. A workgroup (input-channel chunk ch, tile group
// tg) takes the 8 x 8 x 4 tiles tg, tg + G, ... of all samples and stages g and the input tile with its halo channel-first
// in LDS; a wave owns one block of 16 output rows and the nine taps of one dz, and its operands of the three dx of a dy
// come from one window of the input row: 22 LDS reads for 36 products.
// Every sum is made in the order that a training run has always had: a group's products tile by tile, two rows of eight
// voxels at a time (BF16: one product of 16; FP32: four products of four, half a row each), the groups j, j + 4, ... in
// four chains, and these one after another. Adam divides by the gradient's own size, so that an order which changes
// values near zero in their last bit changes the next step's gradients by 1e-3: the order is part of the result
// (tests/golden/cnn_training.npz).
// Bound: bringing g and the input to the CUs, and the latency of a tile's loads, which the other workgroups of a CU hide
// (five of them with 16 output channels, two with 64): neighbouring tiles run on one XCD, so that a 128-byte line comes
// from its L2 for all of its four tiles. At 4 x 64^3 in BF16, bias and final sum included: 48 -> 16 channels 220 us
// (whole-row tiles, with the sums in an order of their own, 232 us; four waves sharing the 27 taps of one tile, its
// neighbours on other XCDs, 720 us), 16 -> 16 at 92 us, 96 -> 32 at 32^3 97 us, all layers of a training step 0.69 ms.
constexpr int GX = 8, GY = 8, GZ = 4;                         // a tile
constexpr int GHY = GY + 2, GROWS = GHY * (GZ + 2), GROW = GX + 4;   // stored rows: halo at 1 and GX + 2, interior from 2
template <typename T> struct WgTile {
    // channel strides of 4 mod 8 (BF16) or 4 mod 16 (FP32) words: the 16 channels of a read share no bank
    static constexpr int PAD = sizeof(T) == 2 ? 8 : 4;
    static constexpr int XCH = GROWS * GROW + PAD, GCH = GX * GY * GZ + PAD;
};

// The nine taps of a dz over one plane of a tile: w the lane's channel of the input plane, a its output channel's row of g
template <typename T> struct WgPlane;
template <> struct WgPlane<bf16> {
    // four K steps of two rows; lane group k holds the four voxels 4 (k % 2) .. of row k / 2
    __device__ __forceinline__ static void run(const bf16 *w, const bf16 *a, int k, v4f *acc) {
        w += (k >> 1) * GROW + 4 * (k & 1);
        a += (k >> 1) * GX + 4 * (k & 1);
        uint2 lo[GHY - 1], hi[GHY - 1];                       // from two elements before the four voxels to two after
        v4s av[4];
#pragma unroll
        for (int y = 0; y < GHY - 1; ++y) {
            lo[y] = *reinterpret_cast<const uint2 *>(w + y * GROW);
            hi[y] = *reinterpret_cast<const uint2 *>(w + y * GROW + 4);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) __builtin_memcpy(&av[s], a + 2 * s * GX, 8);
#pragma unroll
        for (int y = 0; y < GHY - 1; ++y) {
            const unsigned m01 = __builtin_amdgcn_alignbit(lo[y].y, lo[y].x, 16);
            const unsigned m12 = __builtin_amdgcn_alignbit(hi[y].x, lo[y].y, 16);
            const unsigned m23 = __builtin_amdgcn_alignbit(hi[y].y, hi[y].x, 16);
            const uint2 b[3] = {make_uint2(m01, m12), make_uint2(lo[y].y, hi[y].x), make_uint2(m12, m23)};
            // row y is row 2 s + dy of step s; every tap meets the steps in their order
#pragma unroll
            for (int dy = 2; dy >= 0; --dy) {
                if ((y - dy) % 2 || y < dy || y - dy > 6) continue;
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) {
                    v4s b4;
                    __builtin_memcpy(&b4, &b[dx], 8);
                    acc[dy * 3 + dx] = MT<bf16>::mma(av[(y - dy) / 2], b4, acc[dy * 3 + dx]);
                }
            }
        }
    }
};
template <> struct WgPlane<float> {
    // sixteen K steps of half a row; lane group k holds voxel k of the half
    __device__ __forceinline__ static void run(const float *w, const float *a, int k, v4f *acc) {
#pragma unroll
        for (int y = 0; y < GHY; ++y) {
            float b[2][3];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) b[h][dx] = w[y * GROW + 1 + 4 * h + k + dx];
#pragma unroll
            for (int dy = 2; dy >= 0; --dy) {
                if (y < dy || y - dy >= GY) continue;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float av = a[(y - dy) * GX + 4 * h + k];
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx) acc[dy * 3 + dx] = MT<float>::mma(av, b[h][dx], acc[dy * 3 + dx]);
                }
            }
        }
    }
};

template <typename T, int FR, bool V4>
__global__ __launch_bounds__(192 * FR) void k_wgrad_direct(const float *__restrict__ g, long long g_bs, int Co,
                                                           const float *__restrict__ in, long long in_bs, int Ci, int S,
                                                           int B, int G, float *__restrict__ part) {
    constexpr int COP = FR * 16, NT = 192 * FR, XCH = WgTile<T>::XCH, GCH = WgTile<T>::GCH;
    __shared__ __attribute__((aligned(16))) T sm[DCC * XCH + COP * GCH];
    T *sX = sm, *sG = sm + DCC * XCH;
    const int nch = (Ci + DCC - 1) / DCC;
    const int per = (nch * G + 7) / 8;
    const int lin = (blockIdx.x % 8) * per + blockIdx.x / 8;  // neighbouring tile groups on one XCD
    if (lin >= nch * G) return;
    const int ch = lin % nch, tg = lin / nch;                 // the chunks of a tile group share its g
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int dz = wave % 3, rg = wave / 3;
    const int ntx = (S + GX - 1) / GX, nty = (S + GY - 1) / GY, ntz = (S + GZ - 1) / GZ;
    const int tiles = ntx * nty * ntz;
    const int V = S * S * S;
    const int nc = min(Ci - ch * DCC, DCC);
    v4f acc[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) acc[q] = v4f{0, 0, 0, 0};
    // staged in units of four channels, half a row and its halo end; channels from a unit's end on stay zero
    const int units = (nc + 3) / 4 * 2 * GROWS;
    for (int e = (nc + 3) / 4 * 4 * XCH + tid; e < DCC * XCH; e += NT) st_one(sX + e, 0.f);
    for (int tt = tg; tt < B * tiles; tt += G) {
        const int b = tt / tiles, t = tt % tiles;
        const int x0 = (t % ntx) * GX, y0 = ((t / ntx) % nty) * GY, z0 = (t / (ntx * nty)) * GZ;
        const float *ib = in + ((long long)b * in_bs + (long long)ch * DCC * V);
        const float *gb = g + (long long)b * g_bs;
        constexpr int GU = COP * GX * GY * GZ / 4, GP = (GU + NT - 1) / NT;   // quads of g; the last ones more than once
        float4 gv[GP];
#pragma unroll
        for (int p = 0; p < GP; ++p) {
            const int u = min(tid + NT * p, GU - 1), o = u >> 6, q = u & 63;
            const int z = z0 + (q >> 4), y = y0 + ((q >> 1) & 7);
            const bool rin = z < S && y < S && o < Co;
            gv[p] = row4<V4>(gb + (rin ? (long long)o * V + ((long long)z * S + y) * S : 0), x0 + 4 * (q & 1), S, rin);
        }
        __syncthreads();
        for (int u0 = 0; u0 < units; u0 += NT) {
            const int u = min(u0 + tid, units - 1), c0 = u / (2 * GROWS) * 4, r = u % (2 * GROWS) >> 1, e = u & 1;
            const int z = z0 + r / GHY - 1, y = y0 + r % GHY - 1;
            const bool rin = (unsigned)z < (unsigned)S && (unsigned)y < (unsigned)S;
            const float *row = ib + (rin ? ((long long)z * S + y) * S : 0);
            float4 v[4];
            float h[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool cin = c0 + j < nc;
                const float *rc = row + (long long)(cin ? c0 + j : 0) * V;
                v[j] = row4<V4>(rc, x0 + 4 * e, S, rin && cin);
                h[j] = row1(rc, e ? x0 + GX : x0 - 1, S, rin && cin);
            }
            T *d = sX + c0 * XCH + r * GROW;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                st_two(d + j * XCH + 2 + 4 * e, v[j].x, v[j].y);
                st_two(d + j * XCH + 4 + 4 * e, v[j].z, v[j].w);
                st_one(d + j * XCH + (e ? GX + 2 : 1), h[j]);
            }
        }
#pragma unroll
        for (int p = 0; p < GP; ++p) {
            const int u = min(tid + NT * p, GU - 1);
            T *d = sG + (u >> 6) * GCH + (u & 63) * 4;
            st_two(d, gv[p].x, gv[p].y);
            st_two(d + 2, gv[p].z, gv[p].w);
        }
        __syncthreads();
        const T *w = sX + (lane & 15) * XCH + dz * GHY * GROW, *a = sG + (rg * 16 + (lane & 15)) * GCH;
#pragma unroll
        for (int z = 0; z < GZ; ++z) WgPlane<T>::run(w + z * GHY * GROW, a + z * GX * GY, lane >> 4, acc);
    }
    // part[tg][ch][tap][row block][i][16 outputs], of the chunk's existing input channels (nci: of every chunk)
    const int nci = min(Ci, DCC), i = lane & 15;
    if (i >= nc) return;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        float *p = part + (((((long long)tg * nch + ch) * 27 + dz * 9 + q) * FR + rg) * nci + i) * 16 + 4 * (lane >> 4);
        *reinterpret_cast<float4 *>(p) = make_float4(acc[q][0], acc[q][1], acc[q][2], acc[q][3]);
    }
}

// dW from the tile groups' partial sums: thread (e, j) adds the groups j, j + 4, ... of value e, and the four sums are added
// in the order j = 0..3. The last block adds the slices of the bias (k_bias_part).
__global__ __launch_bounds__(256) void k_wgrad_sum(const float *__restrict__ part, const float *__restrict__ bpart, int G,
                                                   int n, int Co, int FR, int Ci, float *__restrict__ dW, float *__restrict__ db) {
    __shared__ float sm[4][64];
    const int el = threadIdx.x & 63, j = threadIdx.x >> 6;
    if (blockIdx.x == gridDim.x - 1) {
        if ((int)threadIdx.x < Co) db[threadIdx.x] = sum_strided(bpart + threadIdx.x * BG_SLICES, 0, BG_SLICES, 1);
        return;
    }
    const int e = blockIdx.x * 64 + el;
    sm[j][el] = e < n ? sum_strided<16>(part + e, (long long)j * n, (long long)G * n, 4LL * n) : 0.f;
    __syncthreads();
    if (j || e >= n) return;
    const int nci = min(Ci, DCC);
    int r = e / 16, o = e % 16;
    const int i = r % nci;
    r /= nci;
    o += r % FR * 16;
    r /= FR;
    const int tap = r % 27, c = r / 27 * DCC + i;
    if (o < Co && c < Ci) dW[((long long)o * Ci + c) * 27 + tap] = ((sm[0][el] + sm[1][el]) + sm[2][el]) + sm[3][el];
}

// dW[e] = sum_q part[q][e], q = 0..G-1: a block takes 64 consecutive e; thread (e, j) adds q = j, j + 4, ...
// (coalesced rows of 64 values), and the four partial sums are added in the order j = 0..3
__global__ __launch_bounds__(256) void k_wgrad_direct_sum(const float *__restrict__ part, int G, long long n,
                                                          float *__restrict__ dW) {
    __shared__ float sm[4][64];
    const int el = threadIdx.x & 63, j = threadIdx.x >> 6;
    const long long e = (long long)blockIdx.x * 64 + el;
    sm[j][el] = e < n ? sum_strided(part + e, j * n, G * n, 4 * n) : 0.f;
    __syncthreads();
    if (j == 0 && e < n) dW[e] = ((sm[0][el] + sm[1][el]) + sm[2][el]) + sm[3][el];
}

// weight gradient of the 1x1x1 head, dW[o][i] = sum_{b,v} g[b][o][v] in[b][i][v] (Co <= 2, Ci <= 16, V a multiple of 256):
// each thread accumulates all Co x Ci products over its voxels, blocks reduce in a fixed order into part[blk][o][i].
// Four voxels' loads are in flight at a time, and all outputs are reduced side by side; with a voxel's loads waited for and
// eight barriers per output it took 119 us at 4 x 64^3, now 16 us (76 MB at 4.8 TB/s).
constexpr int W1_CO = 2, W1_CI = 16, W1_VPT = 16;
__global__ __launch_bounds__(256) void k_wgrad_1x1(const float *__restrict__ g, long long g_bs, int Co,
                                                   const float *__restrict__ in, long long in_bs, int Ci, int V, int B,
                                                   float *__restrict__ part) {
    __shared__ float sm[W1_CO * W1_CI][256];
    const int tid = threadIdx.x;
    float acc[W1_CO][W1_CI];
#pragma unroll
    for (int o = 0; o < W1_CO; ++o)
#pragma unroll
        for (int i = 0; i < W1_CI; ++i) acc[o][i] = 0.f;
    const int rows = V / 256, total = rows * B;               // rows of 256 voxels, of one sample each
    for (int k0 = 0; k0 < W1_VPT; k0 += 4) {
        float gv[4][W1_CO], xv[4][W1_CI];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int q = min((int)blockIdx.x * W1_VPT + k0 + k, total - 1), b = q / rows;
            const int v = (q - b * rows) * 256 + tid;
#pragma unroll
            for (int o = 0; o < W1_CO; ++o) gv[k][o] = g[b * g_bs + (long long)min(o, Co - 1) * V + v];
#pragma unroll
            for (int i = 0; i < W1_CI; ++i) xv[k][i] = in[b * in_bs + (long long)min(i, Ci - 1) * V + v];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if ((int)blockIdx.x * W1_VPT + k0 + k >= total) break;
#pragma unroll
            for (int i = 0; i < W1_CI; ++i)
#pragma unroll
                for (int o = 0; o < W1_CO; ++o) acc[o][i] += gv[k][o] * xv[k][i];
        }
    }
#pragma unroll
    for (int o = 0; o < W1_CO; ++o)
#pragma unroll
        for (int i = 0; i < W1_CI; ++i) sm[o * W1_CI + i][tid] = acc[o][i];
    for (int w = 128; w > 0; w >>= 1) {
        __syncthreads();
        for (int e = tid; e < W1_CO * W1_CI * w; e += 256) sm[e / w][e % w] += sm[e / w][e % w + w];
    }
    __syncthreads();
    for (int e = tid; e < Co * Ci; e += 256) part[(long long)blockIdx.x * Co * Ci + e] = sm[e / Ci * W1_CI + e % Ci][0];
}

}  // namespace

// ---------------------------------------------------------------------------------------------- launchers
// Whether a layer's chunks are summed in parts (few 8 x 8 x 4 boxes of voxels times 16 output channels, several
// chunks) and by how many chunks each. It fixes the order of the sums, not the launch.
void cnn_direct_split(int Ci, int S, int COP, int B, int &nsplit, int &cpb) {
    const long long boxes = (long long)((S + 7) / 8) * ((S + 7) / 8) * ((S + 3) / 4) * B;
    const int nchunk = (Ci + DCC - 1) / DCC;
    const long long target = 1024, wg = boxes * (COP / 16);
    nsplit = 1;
    cpb = nchunk;
    if (boxes >= target || wg >= target || nchunk == 1) return;
    const int want = (int)std::min<long long>(nchunk, (target + wg - 1) / wg);
    cpb = (nchunk + want - 1) / want;
    nsplit = (nchunk + cpb - 1) / cpb;
}

struct ConvArgs {
    const float *in;
    long long in_bs;
    int Ci, S;
    const void *wt;
    int COP;
    const float *bias;
    int Co;
    float *out;
    long long out_bs;
    int relu;
    const float *mask;
    int B, vec;
};

template <typename T, int FR, int TX, int TZ> hipError_t conv_launch(const ConvArgs &a, hipStream_t s) {
    const int tiles = ((a.S + TX - 1) / TX) * ((a.S + CY - 1) / CY) * ((a.S + TZ - 1) / TZ);
    const int rowgroups = a.COP / 16 / FR, blocks = a.B * tiles * rowgroups;
    hipLaunchKernelGGL((k_conv_direct<T, FR, TX, TZ>), dim3((unsigned)((blocks + 7) / 8 * 8)), dim3(256), 0, s, a.in, a.in_bs,
                       a.Ci, a.S, (const T *)a.wt, a.COP, a.bias, a.Co, a.out, a.out_bs, a.relu, a.mask, rowgroups, a.vec,
                       blocks);
    return hipGetLastError();
}

// Output rows per workgroup and tile: as many row blocks as divide the layer's, up to three (they share the staged
// input), and 512 voxels; 256 voxels, then one row block, where that leaves fewer than 512 workgroups (two per CU)
template <typename T, int TX> hipError_t conv_shape(const ConvArgs &a, hipStream_t s) {
    constexpr int Z2 = 512 / 4 / TX, Z1 = Z2 / 2;
    const int fr = a.COP / 16;
    const long long vox = (long long)a.B * a.S * a.S * a.S;
    const int best = fr % 3 == 0 && !a.mask ? 3 : fr % 2 == 0 ? 2 : 1;   // (three leave no registers for a mask)
    const bool wide = vox / 512 * (fr / best) >= 512;
    const int take = wide || vox / 256 * (fr / best) >= 512 ? best : 1;
    if (wide) return take == 3 ? conv_launch<T, 3, TX, Z2>(a, s) : take == 2 ? conv_launch<T, 2, TX, Z2>(a, s) : conv_launch<T, 1, TX, Z2>(a, s);
    return take == 3 ? conv_launch<T, 3, TX, Z1>(a, s) : take == 2 ? conv_launch<T, 2, TX, Z1>(a, s) : conv_launch<T, 1, TX, Z1>(a, s);
}

template <typename T>
hipError_t cnn_conv_direct_t(const float *in, long long in_bs, int Ci, int S, const void *wt, int COP, const float *bias,
                             int Co, float *out, long long out_bs, int relu, const float *mask, int B, hipStream_t s) {
    const int vec = S % 4 == 0 && (uintptr_t)in % 16 == 0 && in_bs % 4 == 0;
    int nsplit, cpb;
    cnn_direct_split(Ci, S, COP, B, nsplit, cpb);
    if (nsplit > 1) {
        if (nsplit > PARTS_MAX) return hipErrorInvalidValue;
        constexpr int PER = deep_per<T>();
        const int rowgroups = COP / 16, tiles = ((S + 15) / 16) * ((S + CY - 1) / CY) * S, waves = (nsplit + PER - 1) / PER;
        const size_t lds = sizeof(typename Chan<T>::t) * ConvTile<16, 1>::QUADS * waves;
        static_assert(sizeof(typename Chan<T>::t) * ConvTile<16, 1>::QUADS >= 4096 * PER, "the parts fit the staging area");
        hipLaunchKernelGGL(k_conv_deep<T>, dim3((unsigned)((long long)B * tiles * rowgroups)), dim3(64 * waves), lds, s, in,
                           in_bs, Ci, S, (const T *)wt, COP, bias, Co, out, out_bs, relu, mask, rowgroups, vec, nsplit,
                           cpb);
        return hipGetLastError();
    }
    const ConvArgs a{in, in_bs, Ci, S, wt, COP, bias, Co, out, out_bs, relu, mask, B, vec};
    if (S > 32) return conv_shape<T, 64>(a, s);
    if (S > 16) return conv_shape<T, 32>(a, s);
    return conv_shape<T, 16>(a, s);
}

hipError_t cnn_conv_direct(int use_bf16, const float *in, long long in_bs, int Ci, int S, const void *wt, int COP,
                           const float *bias, int Co, float *out, long long out_bs, int relu, const float *mask, int B,
                           hipStream_t s) {
    return use_bf16 ? cnn_conv_direct_t<bf16>(in, in_bs, Ci, S, wt, COP, bias, Co, out, out_bs, relu, mask, B, s)
                    : cnn_conv_direct_t<float>(in, in_bs, Ci, S, wt, COP, bias, Co, out, out_bs, relu, mask, B, s);
}

// Tile groups: 1024 workgroups in all, or one tile each. The number fixes the order of the sums.
template <typename T, int FR>
hipError_t wgrad_launch(hipStream_t s, const float *g, long long g_bs, int Co, const float *in, long long in_bs, int Ci,
                        int S, int B, float *part, long long part_elems, float *bpart, float *dW, float *db) {
    const int nch = (Ci + DCC - 1) / DCC;
    if (nch > 1 && Ci % DCC) return hipErrorInvalidValue;     // every chunk has the same number of input channels
    const int tiles = ((S + GX - 1) / GX) * ((S + GY - 1) / GY) * ((S + GZ - 1) / GZ);
    const long long n = (long long)27 * FR * 16 * Ci;
    const int G = (int)std::min<long long>((long long)B * tiles, (1024 + nch - 1) / nch);
    if (G * n > part_elems) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_bias_part, dim3(Co * BG_SLICES), dim3(256), 0, s, g, g_bs, B, S * S * S, bpart);
    const unsigned grid = (unsigned)((nch * G + 7) / 8 * 8);
    // 16-byte loads need every row 16-byte aligned
    if (S % 4 == 0 && ((uintptr_t)g | (uintptr_t)in) % 16 == 0 && (g_bs | in_bs) % 4 == 0)
        hipLaunchKernelGGL((k_wgrad_direct<T, FR, true>), dim3(grid), dim3(192 * FR), 0, s, g, g_bs, Co, in, in_bs, Ci, S, B, G, part);
    else
        hipLaunchKernelGGL((k_wgrad_direct<T, FR, false>), dim3(grid), dim3(192 * FR), 0, s, g, g_bs, Co, in, in_bs, Ci, S, B, G, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_wgrad_sum, dim3((unsigned)((n + 63) / 64 + 1)), dim3(256), 0, s, part, bpart, G, (int)n, Co, FR, Ci, dW, db);
    return hipGetLastError();
}

template <typename T>
hipError_t cnn_wgrad_direct_t(const float *g, long long g_bs, int Co, const float *in, long long in_bs, int Ci, int S,
                              int B, float *part, long long part_elems, float *bpart, float *dW, float *db,
                              hipStream_t s) {
    switch ((Co + 15) / 16) {
    case 1: return wgrad_launch<T, 1>(s, g, g_bs, Co, in, in_bs, Ci, S, B, part, part_elems, bpart, dW, db);
    case 2: return wgrad_launch<T, 2>(s, g, g_bs, Co, in, in_bs, Ci, S, B, part, part_elems, bpart, dW, db);
    case 4: return wgrad_launch<T, 4>(s, g, g_bs, Co, in, in_bs, Ci, S, B, part, part_elems, bpart, dW, db);
    default: return hipErrorInvalidValue;
    }
}

hipError_t cnn_wgrad_1x1(const float *g, long long g_bs, int Co, const float *in, long long in_bs, int Ci, int V, int B,
                         float *part, long long part_elems, float *dW, hipStream_t s) {
    if (Co > W1_CO || Ci > W1_CI || V % 256) return hipErrorInvalidValue;
    const long long NV = (long long)V * B;
    const long long nblk = (NV + 256LL * W1_VPT - 1) / (256LL * W1_VPT);
    const long long per = (long long)Co * Ci;
    if (nblk * per > part_elems) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_wgrad_1x1, dim3((unsigned)nblk), dim3(256), 0, s, g, g_bs, Co, in, in_bs, Ci, V, B, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_wgrad_direct_sum, dim3((unsigned)((per + 63) / 64)), dim3(256), 0, s, part, (int)nblk, per, dW);
    return hipGetLastError();
}

hipError_t cnn_wgrad_direct(int use_bf16, const float *g, long long g_bs, int Co, const float *in, long long in_bs,
                            int Ci, int S, int B, float *part, long long part_elems, float *bpart, float *dW, float *db,
                            hipStream_t s) {
    return use_bf16 ? cnn_wgrad_direct_t<bf16>(g, g_bs, Co, in, in_bs, Ci, S, B, part, part_elems, bpart, dW, db, s)
                    : cnn_wgrad_direct_t<float>(g, g_bs, Co, in, in_bs, Ci, S, B, part, part_elems, bpart, dW, db, s);
}

long long cnn_direct_size(int Co, int Ci) { return (long long)((Ci + DCC - 1) / DCC) * 27 * ((Co + 15) / 16 * 16) * DCC; }

hipError_t cnn_pack(int use_bf16, CnnPackJobs &p, hipStream_t s) {
    int blocks = 0;
    for (int k = 0; k < p.n; ++k) {
        CnnPackJob &q = p.j[k];
        q.COP = (q.Co + 15) / 16 * 16;
        q.total = q.taps == 27 ? (int)cnn_direct_size(q.Co, q.Ci) : q.COP * q.Kp;
        q.block0 = blocks;
        blocks += (q.total + 255) / 256;
    }
    if (use_bf16) hipLaunchKernelGGL(k_pack<bf16>, dim3(blocks), dim3(256), 0, s, p);
    else hipLaunchKernelGGL(k_pack<float>, dim3(blocks), dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t cnn_head(int use_bf16, const float *in, long long in_bs, int Ci, int V, const void *wt, int Kp, const float *bias,
                    int Co, float *out, long long out_bs, const float *mask, int B, hipStream_t s) {
    if (Co > 16 || Ci > 16 || V % 256 || in_bs % 4 || out_bs % 4 || (uintptr_t)in % 16 || (uintptr_t)out % 16 || (uintptr_t)mask % 16)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)((long long)B * (V / 256)));
    if (use_bf16) hipLaunchKernelGGL(k_head<bf16>, grid, dim3(256), 0, s, in, in_bs, Ci, V, (const bf16 *)wt, Kp, bias, Co, out, out_bs, mask);
    else hipLaunchKernelGGL(k_head<float>, grid, dim3(256), 0, s, in, in_bs, Ci, V, (const float *)wt, Kp, bias, Co, out, out_bs, mask);
    return hipGetLastError();
}

hipError_t cnn_bias_grad(const float *g, long long g_bs, int B, long long V, int Co, float *part, float *db,
                         hipStream_t s) {
    hipLaunchKernelGGL(k_bias_part, dim3(Co * BG_SLICES), dim3(256), 0, s, g, g_bs, B, (int)V, part);
    hipLaunchKernelGGL(k_bias_reduce, dim3((Co + 63) / 64), dim3(64), 0, s, part, Co, db);
    return hipGetLastError();
}

// n: parents along an axis
#define PARENTS_LAUNCH(kernel, ...)                                                                                     \
    do {                                                                                                                \
        const long long per = (long long)n * n * n;                                                                     \
        if (n % 2 == 0) hipLaunchKernelGGL(kernel<2>, dim3((unsigned)((per / 2 + 255) / 256 * C * B)), dim3(256), 0, s, __VA_ARGS__); \
        else hipLaunchKernelGGL(kernel<1>, dim3((unsigned)((per + 255) / 256 * C * B)), dim3(256), 0, s, __VA_ARGS__);   \
        return hipGetLastError();                                                                                       \
    } while (0)
hipError_t cnn_pool_fwd(const float *in, long long in_bs, float *out, long long out_bs, int C, int n, int B, hipStream_t s) {
    PARENTS_LAUNCH(k_pool_fwd, in, in_bs, out, out_bs, C, n);
}
hipError_t cnn_pool_bwd(const float *gout, long long gout_bs, float *gin, const float *y, long long gin_bs, int C, int n, int B,
                        hipStream_t s) {
    PARENTS_LAUNCH(k_pool_bwd, gout, gout_bs, gin, y, gin_bs, C, n);
}
hipError_t cnn_up_fwd(const float *in, long long in_bs, float *out, long long out_bs, int C, int n, int B, hipStream_t s) {
    PARENTS_LAUNCH(k_up_fwd, in, in_bs, out, out_bs, C, n);
}
hipError_t cnn_up_bwd(const float *gout, long long gout_bs, float *gin, const float *y, long long gin_bs, int C, int n, int B,
                      hipStream_t s) {
    PARENTS_LAUNCH(k_up_bwd, gout, gout_bs, gin, y, gin_bs, C, n);
}
#undef PARENTS_LAUNCH
hipError_t cnn_mse(const float *y, const float *t, long long n, float *g, double *part, double *loss, hipStream_t s) {
    unsigned nb = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_mse, dim3(nb), dim3(256), 0, s, y, t, n, g, part);
    hipLaunchKernelGGL(k_sum_d, dim3(1), dim3(256), 0, s, part, (int)nb, loss, 1.0 / (double)n);
    return hipGetLastError();
}
hipError_t cnn_adam(float *w, const float *g, float *m, float *v, long long n, float lr, float b1, float b2, float eps,
                    float c1, float c2, hipStream_t s) {
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w, g, m, v, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}
hipError_t cnn_features(const double *k2h, const double2 *fh, int halo, int nf, int S, double k0sq, double cs,
                        double fs, float *x, hipStream_t s) {
    long long V = (long long)S * S * S;
    hipLaunchKernelGGL(k_features, dim3((unsigned)((V + 255) / 256)), dim3(256), 0, s, k2h, fh, halo, nf, S,
                       1.0 / k0sq, cs, fs, x);
    return hipGetLastError();
}
hipError_t cnn_prolong(const float *coarse, int nc, double scale, double gre, double gim, int cubic, double2 *fine,
                       int nf, double2 *work, hipStream_t s) {
    long long n = (long long)nf * nf * nf;
    if (cubic && work) {
        // x: [z][y][x] -> [x'][z][y]; y: [x'][z][y] -> [y'][x'][z]; z: [y'][x'][z] -> [z'][y'][x']
        double2 *t1 = work, *t2 = work + (long long)nf * nc * nc;
        const long long m1 = (long long)nf * nc * nc, m2 = (long long)nf * nf * nc;
        hipLaunchKernelGGL(k_prolong3_pass<float>, dim3((unsigned)((m1 + 255) / 256)), dim3(256), 0, s, coarse, 0, nc,
                           nc, nc, nf, gre, gim, 1.0, t1);
        hipLaunchKernelGGL(k_prolong3_pass<double2>, dim3((unsigned)((m2 + 255) / 256)), dim3(256), 0, s, t1, 1, nc,
                           nc, nf, nf, gre, gim, 1.0, t2);
        hipLaunchKernelGGL(k_prolong3_pass<double2>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, t2, 1, nc,
                           nf, nf, nf, gre, gim, scale, fine);
    } else if (cubic)
        hipLaunchKernelGGL(k_prolong3, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, coarse, nc, scale, gre, gim,
                           fine, nf);
    else
        hipLaunchKernelGGL(k_prolong, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, coarse, nc, scale, gre, gim,
                           fine, nf);
    return hipGetLastError();
}

}  // namespace helm
