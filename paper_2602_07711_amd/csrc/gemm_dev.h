// Device code of the complex MFMA GEMM, shared by the single-problem and the grouped (batched) kernels.
#pragma once
#include <type_traits>

#include "helm_internal.h"

namespace helm {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <typename T> struct cplx;
template <> struct cplx<double> { typedef double2 t; typedef v4d acc; };
template <> struct cplx<float> { typedef float2 t; typedef v4f acc; };

__device__ __forceinline__ v4d mfma(double a, double b, v4d c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma(float a, float b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <typename T, typename S> __device__ __forceinline__ typename cplx<T>::t cvt(S v) {
    typename cplx<T>::t r;
    r.x = (T)v.x;
    r.y = (T)v.y;
    return r;
}

template <typename TC, typename T> __device__ __forceinline__ TC pack(T re, T im) {
    TC r;
    r.x = re;
    r.y = im;
    return r;
}

// The MFMA products of one k-step of four: fragments fa (A, FM blocks of 16 rows) and fb (B, FN blocks of 16
// columns) into the accumulator sets t. RW = 1: A is real, RW = 2: B is real (the sine matrix of the PFFT
// transforms); then each complex MAC needs two real products. Otherwise 3M for FP32 (NS = 3) and 4M for FP64.
template <typename T, int RW, int NS, int FM, int FN>
__device__ __forceinline__ void mma_kstep(typename cplx<T>::acc (&t)[NS][FM][FN], const typename cplx<T>::t (&fa)[FM],
                                          const typename cplx<T>::t (&fb)[FN]) {
    if constexpr (RW == 1) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                t[0][i][j] = mfma(fa[i].x, fb[j].x, t[0][i][j]);
                t[1][i][j] = mfma(fa[i].x, fb[j].y, t[1][i][j]);
            }
    } else if constexpr (RW == 2) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                t[0][i][j] = mfma(fa[i].x, fb[j].x, t[0][i][j]);
                t[1][i][j] = mfma(fa[i].y, fb[j].x, t[1][i][j]);
            }
    } else if constexpr (NS == 3) {
        T sa[FM], sb[FN];
#pragma unroll
        for (int i = 0; i < FM; ++i) sa[i] = fa[i].x + fa[i].y;
#pragma unroll
        for (int j = 0; j < FN; ++j) sb[j] = fb[j].x + fb[j].y;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) t[0][i][j] = mfma(fa[i].x, fb[j].x, t[0][i][j]);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) t[1][i][j] = mfma(fa[i].y, fb[j].y, t[1][i][j]);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) t[2][i][j] = mfma(sa[i], sb[j], t[2][i][j]);
    } else {
        // t[0] = real part, t[1] = imaginary part
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                t[0][i][j] = mfma(fa[i].x, fb[j].x, t[0][i][j]);
                t[1][i][j] = mfma(fa[i].x, fb[j].y, t[1][i][j]);
            }
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                t[0][i][j] = mfma(-fa[i].y, fb[j].y, t[0][i][j]);
                t[1][i][j] = mfma(fa[i].y, fb[j].x, t[1][i][j]);
            }
    }
}

// The same for the first NX mode blocks only: along the columns (X) or the rows of the tile.
template <typename T, bool X, int NX, int RW, int NS, int FM, int FN>
__device__ __forceinline__ void fold_kstep(typename cplx<T>::acc (&t)[NS][FM][FN], const typename cplx<T>::t (&fa)[FM],
                                           const typename cplx<T>::t (&fb)[FN]) {
    typedef typename cplx<T>::t CT;
    typedef typename cplx<T>::acc ACC;
    constexpr int M = X ? FM : NX, N = X ? NX : FN;
    CT a[M], b[N];
    ACC u[NS][M][N];
#pragma unroll
    for (int i = 0; i < M; ++i) a[i] = fa[i];
#pragma unroll
    for (int j = 0; j < N; ++j) b[j] = fb[j];
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int i = 0; i < M; ++i)
#pragma unroll
            for (int j = 0; j < N; ++j) u[q][i][j] = t[q][i][j];
    mma_kstep<T, RW, NS>(u, a, b);
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int i = 0; i < M; ++i)
#pragma unroll
            for (int j = 0; j < N; ++j) t[q][i][j] = u[q][i][j];
}

// Complex value held in accumulator register r of block (i, j): 3M (T1, T2, T3) -> (T1 - T2, T3 - T1 - T2).
template <typename T, int NS, int FM, int FN>
__device__ __forceinline__ void acc_value(const typename cplx<T>::acc (&t)[NS][FM][FN], int i, int j, int r, T &re,
                                          T &im) {
    if constexpr (NS == 3) {
        re = t[0][i][j][r] - t[1][i][j][r];
        im = t[2][i][j][r] - t[0][i][j][r] - t[1][i][j][r];
    } else {
        re = t[0][i][j][r];
        im = t[1][i][j][r];
    }
}

// Row of accumulator register r within a 16x16 block: f64 holds rows 4r + lane/16, f32 rows 4(lane/16) + r.
template <typename T> __device__ __forceinline__ int acc_row(int lane, int r) {
    return sizeof(T) == 8 ? 4 * r + (lane >> 4) : 4 * (lane >> 4) + r;
}

// One BM x BN output tile of C[b] = A[b] B[b]; `tile` enumerates (batch, m-tile, n-tile) with n fastest.
template <typename TA, typename TB, typename TC, typename T, int BM, int BN, int BK, int RW>
__device__ __forceinline__ void gemm_tile(const TA *__restrict__ A, const TB *__restrict__ B, TC *__restrict__ C,
                                          const GemmDesc &d, long long tile) {
    typedef typename cplx<T>::t CT;
    typedef typename cplx<T>::acc ACC;
    constexpr int FM = BM / 32;           // 16x16 blocks per wave along M (2 waves along M)
    constexpr int FN = BN / 32;           // along N (2 waves along N)
    constexpr int EA = BM * BK / 256;     // A elements per thread per chunk
    constexpr int EB = BK * BN / 256;
    __shared__ CT sA[BK][BM + 1];
    __shared__ CT sB[BK][BN];

    const int tm = (d.M + BM - 1) / BM, tn = (d.N + BN - 1) / BN;
    const int b = (int)(tile / ((long long)tm * tn));
    const int rem = (int)(tile % ((long long)tm * tn));
    const int mt = rem / tn, nt = rem % tn;
    const int m0 = mt * BM, n0 = nt * BN;
    A += (long long)b * d.sA;
    B += (long long)b * d.sB;
    C += (long long)b * d.sC;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // RW = 1: A is real, RW = 2: B is real (the sine matrix of the PFFT transforms); then each complex MAC
    // needs two real products. Otherwise 3M for FP32 and 4M for FP64.
    constexpr bool G3 = sizeof(T) == 4 && RW == 0;
    constexpr int NS = G3 ? 3 : 2;
    ACC t[NS][FM][FN];
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) t[q][i][j] = ACC{0, 0, 0, 0};

    CT ra[EA], rb[EB];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int e = 0; e < EA; ++e) {
            int idx = tid + e * 256;
            int mm = idx / BK, kk = idx % BK;          // consecutive threads walk k (contiguous in A rows)
            int gm = m0 + mm, gk = k0 + kk;
            ra[e] = (gm < d.M && gk < d.K) ? cvt<T>(A[(long long)gm * d.lda + gk]) : CT{0, 0};
        }
#pragma unroll
        for (int e = 0; e < EB; ++e) {
            int idx = tid + e * 256;
            int kk = idx / BN, nn = idx % BN;          // consecutive threads walk n (contiguous in B rows)
            int gk = k0 + kk, gn = n0 + nn;
            rb[e] = (gk < d.K && gn < d.N) ? cvt<T>(B[(long long)gk * d.ldb + gn]) : CT{0, 0};
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int e = 0; e < EA; ++e) {
            int idx = tid + e * 256;
            sA[idx % BK][idx / BK] = ra[e];
        }
#pragma unroll
        for (int e = 0; e < EB; ++e) {
            int idx = tid + e * 256;
            sB[idx / BN][idx % BN] = rb[e];
        }
    };

    const int rowA = wm * (BM / 2) + (lane & 15);
    const int colB = wn * (BN / 2) + (lane & 15);
    const int kl = lane >> 4;

    fetch(0);
    for (int k0 = 0; k0 < d.K; k0 += BK) {
        __syncthreads();
        stash();
        __syncthreads();
        if (k0 + BK < d.K) fetch(k0 + BK);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 4) {
            CT fa[FM], fb[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) fa[i] = sA[kk + kl][rowA + i * 16];
#pragma unroll
            for (int j = 0; j < FN; ++j) fb[j] = sB[kk + kl][colB + j * 16];
            mma_kstep<T, RW, NS>(t, fa, fb);
        }
    }

#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int gn = n0 + wn * (BN / 2) + j * 16 + (lane & 15);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gm = m0 + wm * (BM / 2) + i * 16 + acc_row<T>(lane, r);
                if (gm < d.M && gn < d.N) {
                    T re, im;
                    acc_value<T>(t, i, j, r, re, im);
                    C[(long long)gm * d.ldc + gn] = pack<TC, T>(re, im);
                }
            }
        }
}

// ---------------------------------------------------------------------------------------------------------
// Folded EigT transforms. Lambda-bar has the same closure at both ends, so it is centrosymmetric and its
// eigenvectors are symmetric or skew about the middle of the axis: V = Q diag(Vs, Va), V^{-1} = diag(Vs^{-1},
// Va^{-1}) Q^T with Q the butterfly (e_i +- e_{n-1-i})/sqrt(2) (plus e_m alone for odd n). A length-n transform
// is then two products with the half blocks, n^2/2 complex MACs instead of n^2; the butterfly is fused into
// the operand load (forward: the data enters as D[i] +- D[n-1-i]) or the epilogue (inverse: the two half
// products P, M are written as P + M at i and P - M at n-1-i). The 1/sqrt(2) factors (1/2 and 1 for the
// middle of an odd axis) live in the block matrices. Modes are ordered [symmetric (ms) | skew (ma)].
//   FOLD_XF  x forward:  C[c][o_p + k] = sum_{i < K_p} (D[c][i] +- D[c][n-1-i]) M_p[i][k]
//   FOLD_YF  y forward:  C[o_p + k][x] = sum_{i < K_p} M_p[k][i] (D[i][x] +- D[n-1-i][x])
//   FOLD_XI  x inverse:  P = sum_{k < ms} D[c][k] M_s[k][i],  M = sum_{k < ma} D[c][ms + k] M_a[k][i]
//   FOLD_YI  y inverse:  P = sum_{k < ms} M_s[j][k] D[k][x],  M = sum_{k < ma} M_a[j][k] D[ms + k][x]
// with p = s (sign +, K_s = ms, o_s = 0) or a (sign -, K_a = ma, o_a = ms); in the inverse, i (j) < ms and the
// middle of an odd axis (i = ma, no skew partner: M = 0 there) is written once.
//
// Tiles. The long dimension of a transform is its lines (x) or the columns of all its slices in a row (y); the short one
// its modes (inverse: positions). A workgroup of four waves takes BL lines by BX modes (BM x BN for x, BN x BM for y), a
// wave BL / 4 lines by all of the tile's modes, so every wave has the same work whatever the number of modes, and a
// tile computes 64, 48 or 32 modes (BX = 64; 128, 96 or 64 for BX = 128), whichever its half still needs (with waves of
// 32 x 32 a 200-long axis took 128 modes for its 100, now 112; columns took whole tiles per slice, 256 for its 200).
// Bound by the matrix cores where they are many (FP64 MFMAs busy 70% of the time at 200^3), by latency where few.
// One transform, before and after: FP64 200^3 x 168 -> 163 us, y 203 -> 163, y inverse 215 -> 161 (four and a z-solve of 71
// are an application of 711; under a profiler they take 175 to 182); 256^3 x 317 -> 304;
// 32^3 5.2 -> 3.8, inverse 9.1 -> 6.3; FP32 256^3 x 159 -> 152, y inverse 136 -> 130, 64^3 inverse 10.3 -> 7.3.
// The block matrices are zero-padded (fold_pad_sum, fold_pad_out), which makes their loads unconditional and lets the
// data's run past the end of the half: they are clamped to the line's own values, which then meet zeros. A tile of 128
// modes may reach past the padding of its block: there it reads the last padded mode, for results that are not stored.

template <int MODE, int BM, int BN> __host__ __device__ inline long long fold_tiles(const FoldDesc &f) {
    return fold_tile_count(MODE, f, BM, BN);
}

// Occupancy the register allocator is asked for: without it, the FP64 kernels keep their accumulators in
// AGPRs on top of the VGPRs the operand staging needs and drop to two waves per SIMD. The x-forward transforms
// with FP64 data hold two raw FP64 values per operand element across a chunk (the butterfly is formed when the
// chunk is written to LDS) and get one wave less. The FP32 inverse transforms on 64 x 64 x 16 tiles park P in LDS
// (fold_tile), 48 KiB per block in all, which fits three blocks per CU.
template <typename T, typename TD, int MODE, int BM, int BN, int BK> constexpr int fold_waves() {
    if (sizeof(T) == 4 && (MODE == FOLD_XI || MODE == FOLD_YI) && BM * BN * BK <= 64 * 64 * 16) return 3;
    return (sizeof(T) == 8 ? (BM * BN * BK <= 64 * 64 * 16 ? 3 : 1) : (BM * BN * BK <= 64 * 64 * 16 ? 4 : 2)) -
           ((MODE == FOLD_XF && sizeof(TD) == 16 && BM * BN * BK <= 64 * 64 * 16) ? 1 : 0);
}

// a +- b in the precision the data is stored in, then converted to the arithmetic type
template <typename T, typename S> __device__ __forceinline__ typename cplx<T>::t fold2(S a, S b, bool minus) {
    S r;
    r.x = minus ? a.x - b.x : a.x + b.x;
    r.y = minus ? a.y - b.y : a.y + b.y;
    return cvt<T>(r);
}

template <typename S> struct Pair { S a, b; };

// The K loop of one tile: raw operands of chunk k0 come from fetchA(k0, e) and fetchB(k0, e), element e of this thread
// (e * 256 + thread, A: consecutive threads walk k, B: consecutive threads walk the columns), and are staged through LDS
// double buffered in registers, as in gemm_tile. finA / finB turn a raw operand into the arithmetic type (conversion, the
// butterfly's sum or difference) only when it is written to LDS, one chunk later: doing it at load time would make
// every chunk wait for its own loads before the MFMAs that should hide them. X: the modes are the columns (else the
// rows); NX: the 16-wide mode blocks that are computed, fixed for the loop (a branch around each block's MFMAs would
// move accumulators between registers, and the compiler then read some before they were written).
template <typename T, bool X, int NX, int BM, int BN, int BK, int NS, int RW, int FM, int FN, typename LA, typename LB,
          typename FA, typename FB>
__device__ __forceinline__ void fold_kloop(typename cplx<T>::acc (&t)[NS][FM][FN], int K, LA fetchA, LB fetchB, FA finA,
                                           FB finB, typename cplx<T>::t (*sA)[BM + 1],
                                           typename cplx<T>::t (*sB)[BN], int tid) {
    typedef typename cplx<T>::t CT;
    constexpr int EA = BM * BK / 256, EB = BK * BN / 256;
    const int lane = tid & 63, wave = tid >> 6;
    decltype(fetchA(0, 0)) ra[EA];
    decltype(fetchB(0, 0)) rb[EB];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int e = 0; e < EA; ++e) ra[e] = fetchA(k0, e);
#pragma unroll
        for (int e = 0; e < EB; ++e) rb[e] = fetchB(k0, e);
    };
    const int rowA = (X ? wave * FM * 16 : 0) + (lane & 15);
    const int colB = (X ? 0 : wave * FN * 16) + (lane & 15);
    const int kl = lane >> 4;
    fetch(0);
    for (int k0 = 0; k0 < K; k0 += BK) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < EA; ++e) {
            const int idx = tid + e * 256;
            sA[idx % BK][idx / BK] = finA(ra[e]);
        }
#pragma unroll
        for (int e = 0; e < EB; ++e) {
            const int idx = tid + e * 256;
            sB[idx / BN][idx % BN] = finB(rb[e]);
        }
        __syncthreads();
        if (k0 + BK < K) fetch(k0 + BK);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 4) {
            CT fa[FM], fb[FN];
#pragma unroll
            for (int i = 0; i < (X ? FM : NX); ++i) fa[i] = sA[kk + kl][rowA + i * 16];
#pragma unroll
            for (int j = 0; j < (X ? NX : FN); ++j) fb[j] = sB[kk + kl][colB + j * 16];
            fold_kstep<T, X, NX, RW, NS>(t, fa, fb);
        }
    }
}

// One tile (`tile` < fold_tiles) of a folded transform.
template <int MODE, typename TD, typename TM, typename TC, typename T, int BM, int BN, int BK, int RW = 0>
__device__ __forceinline__ void fold_tile(const TD *__restrict__ D, const TM *__restrict__ Ms, const TM *__restrict__ Ma,
                                          TC *__restrict__ C, const FoldDesc &f, long long tile) {
    typedef typename cplx<T>::t CT;
    typedef typename cplx<T>::acc ACC;
    constexpr bool X = MODE == FOLD_XF || MODE == FOLD_XI, FWD = MODE == FOLD_XF || MODE == FOLD_YF;
    constexpr int BL = X ? BM : BN, BX = X ? BN : BM;         // lines and modes of a tile
    constexpr int FM = X ? BM / 64 : BM / 16, FN = X ? BN / 16 : BN / 64;
    constexpr int NS = (sizeof(T) == 4 && RW == 0) ? 3 : 2;
    __shared__ CT sA[BK][BM + 1];
    __shared__ CT sB[BK][BN];

    const int n = f.n, ms = f.ms, ma = f.ma;
    const int lines = f.rows * f.batch;                       // x: lines (batch = 1); y: columns of all slices
    const long long ld = f.ld;
    const int hs = (ms + BX - 1) / BX, ha = FWD ? (ma + BX - 1) / BX : 0;
    const int lt = (int)(tile / (hs + ha)), r = (int)(tile % (hs + ha));   // the tiles of the same lines are neighbours
    const int l0 = lt * BL;

    ACC t[NS][FM][FN];
    auto zero = [&]() {
#pragma unroll
        for (int q = 0; q < NS; ++q)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) t[q][i][j] = ACC{0, 0, 0, 0};
    };
    // the product of half `skew`, mode block x0: the data of the forward transforms is folded, that of the inverse ones
    // starts at mode `off`, stride mst
    auto product = [&](bool skew, int x0) {
        // an opaque copy of the thread index: the index arithmetic of two K loops in one kernel (the inverse
        // transforms) is then not shared between them and held in registers across the first
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int K = skew ? ma : ms, outs = fold_pad_out(K), P = X ? outs : fold_pad_sum(K);
        const int off = skew ? f.moff : 0, mst = f.mstep;
        const int nblk = (min(K, x0 + BX) - x0 + 15) / 16;
        const TM *Mp = (skew ? Ma : Ms) + (X ? x0 : (long long)x0 * P);
        const int last = FWD ? n - 1 : K - 1;
        auto run = [&](auto loop) {
            constexpr int FX = BX / 16;
            if (nblk > FX * 3 / 4) loop(std::integral_constant<int, FX>());
            else if (nblk > FX / 2) loop(std::integral_constant<int, FX * 3 / 4>());
            else loop(std::integral_constant<int, FX / 2>());
        };
        auto fmat = [](const TM &v) { return cvt<T>(v); };
        auto fdat = [&](const auto &v) {
            if constexpr (FWD) return fold2<T>(v.a, v.b, skew);
            else return cvt<T>(v);
        };
        if constexpr (X) {
            const TD *base = D + l0 * ld;
            auto la = [&](int k0, int e) {
                const int idx = tid + e * 256, gk = min(k0 + idx % BK, last);
                const int line = min(idx / BK, lines - 1 - l0);
                const unsigned row = (unsigned)line * (unsigned)ld;
                if constexpr (FWD) return Pair<TD>{base[row + gk], base[row + (n - 1 - gk)]};
                else return base[row + off + mst * gk];
            };
            const int mode = BX > 64 ? min(tid % BN, outs - 1 - x0) : tid % BN;
            auto lb = [&](int k0, int e) { return (Mp + (long long)k0 * P)[(unsigned)((tid + e * 256) / BN * P + mode)]; };
            run([&](auto nx) { fold_kloop<T, X, decltype(nx)::value, BM, BN, BK, NS, RW>(t, K, la, lb, fdat, fmat, sA, sB, tid); });
        } else {
            const int col = min(l0 + tid % BN, lines - 1);
            const TD *base = D + (long long)(col / f.rows) * f.sD + col % f.rows + (FWD ? 0 : off * ld);
            // positions as 32-bit offsets (an axis times its stride is at most the vector's 2^31 entries)
            const unsigned uld = (unsigned)ld, top = (unsigned)(n - 1) * uld, end = (unsigned)last * uld;
            const unsigned first = (unsigned)(tid / BN) * uld;
            auto la = [&](int k0, int e) {
                const int idx = tid + e * 256, mode = BX > 64 ? min(idx / BK, outs - 1 - x0) : idx / BK;
                return (Mp + k0)[(unsigned)(mode * P + idx % BK)];
            };
            auto lb = [&](int k0, int e) {
                const unsigned o = min(first + (unsigned)(k0 + e * (256 / BN)) * uld, end);
                if constexpr (FWD) return Pair<TD>{base[o], base[top - o]};
                else return base[mst == 1 ? o : 2 * o];
            };
            run([&](auto nx) { fold_kloop<T, X, decltype(nx)::value, BM, BN, BK, NS, RW>(t, K, la, lb, fmat, fdat, sA, sB, tid); });
        }
    };
    // line and mode (position) of accumulator register r of block (i, j), and the line's offset
    const int lane0 = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto place = [&](int lane, int i, int j, int r, int &line, int &x) {
        const int row = i * 16 + acc_row<T>(lane, r), col = j * 16 + (lane & 15);
        line = l0 + (X ? wave * FM * 16 + row : wave * FN * 16 + col);
        x = X ? col : row;
    };
    auto at = [&](int line) -> long long {                    // x: start of the line; y: the column's first element
        if constexpr (X) return line * ld;
        else return (long long)(line / f.rows) * f.sD + line % f.rows;
    };
    const long long step = X ? 1 : ld;                        // between modes (positions) of a line

    if constexpr (FWD) {
        const bool skew = r >= hs;
        const int x0 = (skew ? r - hs : r) * BX;
        const int K = skew ? ma : ms, off = skew ? f.moff : 0, mst = f.mstep;
        zero();
        product(skew, x0);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    int line, x;
                    place(lane0, i, j, q, line, x);
                    T re, im;
                    acc_value<T>(t, i, j, q, re, im);
                    if (line < lines && x0 + x < K) C[at(line) + (off + mst * (x0 + x)) * step] = pack<TC, T>(re, im);
                }
    } else {
        // FP32 64 x 64 tiles park P in LDS (32 KiB per block, read back only by the thread that wrote it)
        constexpr bool PLDS = sizeof(T) == 4 && FM * FN * 4 * 256 * sizeof(CT) <= 32768;
        __shared__ CT sP[PLDS ? FM * FN * 4 * 256 : 1];
        const int x0 = r * BX;
        zero();
        product(false, x0);
        // park P in this thread's own output slots (first half of the axis; the skew results go to the disjoint second
        // half), or for the FP32 64 x 64 tile in a per-thread LDS area, instead of holding a second accumulator set in
        // registers
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    int line, x;
                    place(lane0, i, j, q, line, x);
                    T re, im;
                    acc_value<T>(t, i, j, q, re, im);
                    if constexpr (PLDS) sP[((i * FN + j) * 4 + q) * 256 + threadIdx.x] = pack<CT, T>(re, im);
                    else if (line < lines && x0 + x < ms) C[at(line) + (x0 + x) * step] = pack<TC, T>(re, im);
                }
        zero();
        // a compiler memory barrier: the epilogue reloads P instead of the stored values being forwarded to it in
        // registers through the second K loop
        asm volatile("" ::: "memory");
        if (x0 < ma) product(true, x0);
        // the epilogue recomputes the slot addresses (an opaque copy of the lane index) rather than keeping the
        // park step's addresses alive through the second K loop
        int lane_e = lane0;
        asm volatile("" : "+v"(lane_e));
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    int line, x;
                    place(lane_e, i, j, q, line, x);
                    const int pos = x0 + x;                   // position along the transformed axis
                    if (line >= lines || pos >= ms) continue;
                    T re, im;
                    acc_value<T>(t, i, j, q, re, im);
                    const long long o = at(line);
                    TC *c = C + o + pos * step;
                    T p0, p1;
                    if constexpr (PLDS) {
                        const CT pv = sP[((i * FN + j) * 4 + q) * 256 + threadIdx.x];
                        p0 = pv.x;
                        p1 = pv.y;
                    } else {
                        const TC pv = *c;
                        p0 = (T)pv.x;
                        p1 = (T)pv.y;
                    }
                    if (pos < ma) {
                        *c = pack<TC, T>(p0 + re, p1 + im);
                        C[o + (n - 1 - pos) * step] = pack<TC, T>(p0 - re, p1 - im);
                    } else if constexpr (PLDS) {
                        *c = pack<TC, T>(p0, p1);             // the middle of an odd axis: P alone
                    }
                }
    }
}

}  // namespace
}  // namespace helm
