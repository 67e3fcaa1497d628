// Krylov kernels of the (F)GMRES outer iteration: the block inner products V^H w together with ||w||^2 in
// one pass over the data (classical Gram-Schmidt with the norm taken from ||w||^2 - sum |h_i|^2), a fixed-
// order two-stage reduction (bitwise reproducible, no atomics), and the linear combination
// out = alpha * base + sum_i c_i V_i used for the orthogonalisation update, the end-of-cycle update
// x += Z y and the restart vector.
#include "krylov_dev.h"

namespace helm {

namespace {

constexpr int DOT_GROUP = 8;   // short vectors: basis vectors per block

// partials of output t are contiguous: part[t * gridDim.x + block], so the reduction reads them coalesced
template <int EPT>
__global__ __launch_bounds__(256) void k_dots(const double2 *__restrict__ V, long long ldv, int nv,
                                              const double2 *__restrict__ w, long long n, double2 *__restrict__ part) {
    const int t0 = blockIdx.y * DOT_GROUP, cnt = EPT == DOT_EPT ? nv : min(nv - t0, DOT_GROUP);
    dots_chunk<EPT>(V + t0 * ldv, ldv, cnt, w, n, part + (long long)t0 * gridDim.x, blockIdx.x, 1, gridDim.x,
                    t0 + cnt == nv);
}

// `host` (may be null): the values once more, in coherent host memory, for a caller that reads them after an event
// behind this kernel. A copy of them on a second stream came behind two more events and a copy, longer than the update that
// it was to hide behind: 32^3 solve 866 us, 128^3 7.28 ms; now (timers read behind the next launches) 670 us and 7.04 ms.
__global__ __launch_bounds__(256) void k_reduce(const double2 *__restrict__ part, int nblocks, int nout,
                                                double2 *__restrict__ out, double2 *__restrict__ host) {
    __shared__ double sr[256], si[256];
    const int t = blockIdx.x, tid = threadIdx.x;
    double re = 0.0, im = 0.0;
    for (int b = tid; b < nblocks; b += 256) {
        double2 v = part[(long long)t * nblocks + b];
        re += v.x;
        im += v.y;
    }
    sr[tid] = re;
    si[tid] = im;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) { sr[tid] += sr[tid + s]; si[tid] += si[tid + s]; }
        __syncthreads();
    }
    if (tid == 0) {
        out[t] = make_double2(sr[0], si[0]);
        if (host) host[t] = make_double2(sr[0], si[0]);
    }
}

constexpr int LC_MAX = 48;
struct LcCoef { double2 c[LC_MAX]; };
constexpr int LC_EPT = 4;   // elements per thread (independent loads in flight per vector)

__device__ __forceinline__ double2 wide(const double2 *p) { return ld_stream(p); }
__device__ __forceinline__ double2 wide(const float2 *p) { return ld_stream_wide(p); }

template <typename VT>
__global__ __launch_bounds__(256) void k_lincomb(double2 *out, const double2 *base, double2 alpha,
                                                 const VT *__restrict__ V, long long ldv, int nv, LcCoef co,
                                                 long long n) {
    const long long start = (long long)blockIdx.x * (256 * LC_EPT) + threadIdx.x;
    double2 acc[LC_EPT];
    bool ok[LC_EPT];
#pragma unroll
    for (int e = 0; e < LC_EPT; ++e) {
        const long long idx = start + (long long)e * 256;
        ok[e] = idx < n;
        acc[e] = make_double2(0.0, 0.0);
        if (base && ok[e]) {
            double2 b = ld_stream(base + idx);
            acc[e].x = alpha.x * b.x - alpha.y * b.y;
            acc[e].y = alpha.x * b.y + alpha.y * b.x;
        }
    }
    int i = 0;
    for (; i + 4 <= nv; i += 4) {            // four vectors per round: 16 loads in flight per thread
        double2 v[4][LC_EPT];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < LC_EPT; ++e) {
                const long long idx = start + (long long)e * 256;
                v[q][e] = ok[e] ? wide(V + (long long)(i + q) * ldv + idx) : make_double2(0.0, 0.0);
            }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double2 c = co.c[i + q];
#pragma unroll
            for (int e = 0; e < LC_EPT; ++e) {
                acc[e].x += c.x * v[q][e].x - c.y * v[q][e].y;
                acc[e].y += c.x * v[q][e].y + c.y * v[q][e].x;
            }
        }
    }
    for (; i < nv; ++i) {
        const VT *vi = V + (long long)i * ldv;
        const double2 c = co.c[i];
        double2 v[LC_EPT];
#pragma unroll
        for (int e = 0; e < LC_EPT; ++e) {
            const long long idx = start + (long long)e * 256;
            v[e] = ok[e] ? wide(vi + idx) : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int e = 0; e < LC_EPT; ++e) {
            acc[e].x += c.x * v[e].x - c.y * v[e].y;
            acc[e].y += c.x * v[e].y + c.y * v[e].x;
        }
    }
#pragma unroll
    for (int e = 0; e < LC_EPT; ++e) {
        const long long idx = start + (long long)e * 256;
        if (ok[e]) out[idx] = acc[e];
    }
}

// The orthogonalisation update of an Arnoldi step with its coefficients taken on the device from the reduced inner
// products red[0..nv-1] = V_i^H w and red[nv] = ||w||^2: eta^2 = ||w||^2 - sum |h_i|^2 and, when no severe
// cancellation happened (eta^2 > reorth ||w||^2), w <- -(w - V h) / eta; otherwise w <- -(w - V h) unscaled, for
// the host's second Gram-Schmidt pass. Every block recomputes the (uniform) coefficients, so no host round trip sits between the
// inner products and the update. Four elements per thread where that still gives a block per CU (128^3: bandwidth, 6.3 TB/s),
// one below (32^3: 32 blocks -> 128; dots and update together take a 32^3 solve from 884 to 848 us).
template <int EPT>
__global__ __launch_bounds__(256) void k_lincomb_cgs(double2 *w, const double2 *__restrict__ V, long long ldv, int nv,
                                                     const double2 *__restrict__ red, long long n, double reorth) {
    constexpr int NV = EPT == 1 ? 8 : 4;   // vectors per round
    const long long start = (long long)blockIdx.x * (256 * EPT) + threadIdx.x;
    long long idx[EPT];                    // past the end: the last element, read and not written
    double2 acc[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        idx[e] = start + (long long)e * 256 < n ? start + (long long)e * 256 : n - 1;
        acc[e] = ld_stream(w + idx[e]);
    }
    double hh = 0.0;
    int i = 0;
    for (; i + 8 <= nv; i += 8) {          // eight products in flight; summed one after another, as the host does
        double2 r[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) r[q] = red[i + q];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            hh = fma(r[q].x, r[q].x, hh);
            hh = fma(r[q].y, r[q].y, hh);
        }
    }
    for (; i < nv; ++i) {
        const double2 r = red[i];
        hh = fma(r.x, r.x, hh);
        hh = fma(r.y, r.y, hh);
    }
    const double ww = red[nv].x, eta2 = ww - hh;
    const double inv = eta2 > reorth * ww ? 1.0 / sqrt(eta2) : 1.0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) acc[e] = make_double2(-inv * acc[e].x, -inv * acc[e].y);
    i = 0;
    for (; i + NV <= nv; i += NV) {
        double2 v[NV][EPT];
#pragma unroll
        for (int q = 0; q < NV; ++q)
#pragma unroll
            for (int e = 0; e < EPT; ++e) v[q][e] = ld_stream(V + (long long)(i + q) * ldv + idx[e]);
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const double2 c = make_double2(red[i + q].x * inv, red[i + q].y * inv);
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                acc[e].x += c.x * v[q][e].x - c.y * v[q][e].y;
                acc[e].y += c.x * v[q][e].y + c.y * v[q][e].x;
            }
        }
    }
    for (; i < nv; ++i) {
        const double2 c = make_double2(red[i].x * inv, red[i].y * inv);
        double2 v[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) v[e] = ld_stream(V + (long long)i * ldv + idx[e]);
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            acc[e].x += c.x * v[e].x - c.y * v[e].y;
            acc[e].y += c.x * v[e].y + c.y * v[e].x;
        }
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e)
        if (start + (long long)e * 256 < n) w[start + (long long)e * 256] = acc[e];
}

__global__ void k_to_c64(const double2 *__restrict__ x, float2 *__restrict__ y, long long n) {
    long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx < n) y[idx] = make_float2((float)x[idx].x, (float)x[idx].y);
}

__global__ void k_zero(double2 *x, long long n) {
    long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx < n) x[idx] = make_double2(0.0, 0.0);
}

}  // namespace

// 16 elements per thread where that still gives a block per CU, else 4 or 1, with eight basis vectors per block: a short
// vector's pass is latency, and its blocks were few. 64^3: 64 blocks, 15.9 us -> 256 blocks of 4 elements per eight
// vectors, 9.3 us; 32^3: 8 blocks, 6.6 us -> 128 of one element, 4.1 us. At 127^3 (500 blocks) 4 elements per thread made a
// whole solve 0.4 % slower.
static int dots_ept(long long n) { return n >= 256LL * 256 * 16 ? 16 : n >= 256LL * 256 * 4 ? 4 : 1; }
int dots_blocks(long long n) {
    const int chunk = 256 * dots_ept(n);
    return (int)((n + chunk - 1) / chunk);
}
int batch_dots_blocks(long long n) { return (int)((n + 256 * DOT_EPT - 1) / (256 * DOT_EPT)); }

hipError_t launch_dots(const double2 *V, long long ldv, int nv, const double2 *w, long long n, double2 *partials,
                       int nblocks, double2 *red, double2 *host, hipStream_t s) {
    if (nv + 1 > MAXV) return hipErrorInvalidValue;
    if (nblocks != dots_blocks(n)) return hipErrorInvalidValue;
    const dim3 grid(nblocks, nv > DOT_GROUP ? (nv + DOT_GROUP - 1) / DOT_GROUP : 1);
    switch (dots_ept(n)) {
    case 16: hipLaunchKernelGGL(k_dots<16>, dim3(nblocks), dim3(256), 0, s, V, ldv, nv, w, n, partials); break;
    case 4: hipLaunchKernelGGL(k_dots<4>, grid, dim3(256), 0, s, V, ldv, nv, w, n, partials); break;
    default: hipLaunchKernelGGL(k_dots<1>, grid, dim3(256), 0, s, V, ldv, nv, w, n, partials); break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_reduce, dim3(nv + 1), dim3(256), 0, s, partials, nblocks, nv + 1, red, host);
    return hipGetLastError();
}

template <typename VT>
hipError_t lincomb_t(double2 *out, const double2 *base, double2 alpha, const VT *V, long long ldv, int nv,
                     const double2 *coef, long long n, hipStream_t s) {
    long long grid_ll = (n + 256 * LC_EPT - 1) / (256 * LC_EPT);
    int grid = (int)(grid_ll < 1 ? 1 : grid_ll);
    int done = 0;
    do {
        int cnt = nv - done < LC_MAX ? nv - done : LC_MAX;
        LcCoef co;
        for (int i = 0; i < cnt; ++i) co.c[i] = coef[done + i];
        const double2 *b = done == 0 ? base : out;
        double2 a = done == 0 ? alpha : make_double2(1.0, 0.0);
        hipLaunchKernelGGL(k_lincomb<VT>, dim3(grid), dim3(256), 0, s, out, b, a, V + (long long)done * ldv, ldv, cnt,
                           co, n);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        done += cnt;
    } while (done < nv);
    return hipSuccess;
}

hipError_t launch_lincomb(double2 *out, const double2 *base, double2 alpha, const double2 *V, long long ldv, int nv,
                          const double2 *coef, long long n, hipStream_t s) {
    return lincomb_t<double2>(out, base, alpha, V, ldv, nv, coef, n, s);
}

hipError_t launch_lincomb(double2 *out, const double2 *base, double2 alpha, const float2 *V, long long ldv, int nv,
                          const double2 *coef, long long n, hipStream_t s) {
    return lincomb_t<float2>(out, base, alpha, V, ldv, nv, coef, n, s);
}

hipError_t launch_lincomb_cgs(double2 *w, const double2 *V, long long ldv, int nv, const double2 *red, long long n,
                              double reorth, hipStream_t s) {
    if (n < 1) return hipErrorInvalidValue;
    if (n >= 256LL * 256 * LC_EPT)
        hipLaunchKernelGGL(k_lincomb_cgs<LC_EPT>, dim3((unsigned)((n + 256 * LC_EPT - 1) / (256 * LC_EPT))), dim3(256), 0, s,
                           w, V, ldv, nv, red, n, reorth);
    else
        hipLaunchKernelGGL(k_lincomb_cgs<1>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w, V, ldv, nv, red, n,
                           reorth);
    return hipGetLastError();
}

hipError_t launch_to_c64(const double2 *x, float2 *y, long long n, hipStream_t s) {
    hipLaunchKernelGGL(k_to_c64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, y, n);
    return hipGetLastError();
}

hipError_t launch_fill_zero(double2 *x, long long n, hipStream_t s) {
    hipLaunchKernelGGL(k_zero, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, n);
    return hipGetLastError();
}

}  // namespace helm
