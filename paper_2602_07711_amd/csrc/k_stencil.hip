// Compact-stencil kernels: derived k^2 fields, the modified right-hand side, and the matrix-vector product
// y = A x of the 2nd/4th/6th-order schemes with the ghost-eliminated absorbing closure.
//
// Operator (per node p, neighbour offsets o in {-1,0,1}^3, U_o the neighbour value, k_o^2 its k^2):
//   order 4 (Sec. 2.2 eq. scheme4):  sum_o c_o U_o + k_p^2 U_p / 2 + sum_faces k_o^2 U_o / 12, with the
//     grid-only coefficients c_o of Delta + sum (h_nu^2+h_mu^2)/12 T_nu T_mu (19 points).
//   order 6 (Sec. 2.3 eq. scheme6, uniform h): collecting the scheme by neighbour class,
//     y = dg U_p + (S3 + 3 S2 + 14 S1)/(30 h^2) + (SW2 - SW1)/90 + sum_nu g_nu (2 D_nu U + D_nu E + h^2 D_nu W)
//     with S1/S2/S3 the sums of U over faces/edges/corners, SW1/SW2 the sums of k^2 U over faces/edges,
//     D_nu U = U(+nu) - U(-nu), D_nu W the same for k^2 U, D_nu E the difference of the edge sums on the
//     +nu and -nu sides, g_nu = h (k^2)_nu / 120 and dg = -64/(15 h^2) + 14/15 k^2 + h^2/20 (lap k^2 - k^4).
// Ghost rule (Sec. 2.3 eq. D_bc): a neighbour outside the grid along an axis takes the boundary node's value
// times gamma of that axis (per clamped axis), and k^2 there is the boundary node's k^2, so the products
// k^2 U obey the same rule.
//
// The matvec (stencil_dev.h) streams z-planes of U and k^2 (with a one-node halo) through LDS, one thread per
// output column. Per node it streams x (16 B), k^2 (8 B), the order-6 field block (32 B), F in the residual form
// (16 B) and writes y (16 B).
#include "stencil_dev.h"

namespace helm {

namespace {

// --------------------------------------------------------------------------- derived fields
// k2 (interior copy) and, for order 6, fld = (dg, g_x, g_y, g_z). k2_halo has `halo` cells per side.
__global__ void k_derived(const double *__restrict__ k2h, int halo, double *__restrict__ k2, double4 *__restrict__ fld,
                          int nx, int ny, int nz, int order, double h, int *__restrict__ bad) {
    long long n = (long long)nx * ny * nz;
    long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    int i = (int)(p % nx);
    int j = (int)((p / nx) % ny);
    int l = (int)(p / ((long long)nx * ny));
    const int px = nx + 2 * halo, py = ny + 2 * halo;
    auto at = [&](int di, int dj, int dl) -> double {
        return k2h[((long long)(l + halo + dl) * py + (j + halo + dj)) * px + (i + halo + di)];
    };
    double c = at(0, 0, 0);
    if (!isfinite(c)) atomicOr(bad, 1);
    k2[p] = c;
    if (order != 6) return;
    double g[3], lap = 0.0;
    for (int a = 0; a < 3; ++a) {
        int dx = (a == 0), dy = (a == 1), dz = (a == 2);
        double p1 = at(dx, dy, dz), m1 = at(-dx, -dy, -dz), p2 = at(2 * dx, 2 * dy, 2 * dz), m2 = at(-2 * dx, -2 * dy, -2 * dz);
        if (!isfinite(p1) || !isfinite(m1) || !isfinite(p2) || !isfinite(m2)) atomicOr(bad, 1);
        g[a] = (-p2 + 8.0 * p1 - 8.0 * m1 + m2) / (12.0 * h);
        lap += (-p2 + 16.0 * p1 - 30.0 * c + 16.0 * m1 - m2) / (12.0 * h * h);
    }
    double h2 = h * h;
    double dg = -64.0 / (15.0 * h2) + 14.0 / 15.0 * c + h2 / 20.0 * (lap - c * c);
    fld[p] = make_double4(dg, h * g[0] / 120.0, h * g[1] / 120.0, h * g[2] / 120.0);
}

// complex k^2: the same differences on complex samples, real and imaginary parts stored separately
__global__ void k_derived_c(const double2 *__restrict__ k2h, int halo, double *__restrict__ k2,
                            double *__restrict__ k2i, double4 *__restrict__ fld, double4 *__restrict__ fldi, int nx,
                            int ny, int nz, int order, double h, int *__restrict__ bad) {
    long long n = (long long)nx * ny * nz;
    long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    int i = (int)(p % nx);
    int j = (int)((p / nx) % ny);
    int l = (int)(p / ((long long)nx * ny));
    const int px = nx + 2 * halo, py = ny + 2 * halo;
    auto at = [&](int di, int dj, int dl) -> double2 {
        return k2h[((long long)(l + halo + dl) * py + (j + halo + dj)) * px + (i + halo + di)];
    };
    const double2 c = at(0, 0, 0);
    if (!isfinite(c.x) || !isfinite(c.y)) atomicOr(bad, 1);
    k2[p] = c.x;
    k2i[p] = c.y;
    if (order != 6) return;
    double2 g[3], lap = make_double2(0.0, 0.0);
    for (int a = 0; a < 3; ++a) {
        int dx = (a == 0), dy = (a == 1), dz = (a == 2);
        double2 p1 = at(dx, dy, dz), m1 = at(-dx, -dy, -dz), p2 = at(2 * dx, 2 * dy, 2 * dz), m2 = at(-2 * dx, -2 * dy, -2 * dz);
        if (!isfinite(p1.x + p1.y + m1.x + m1.y + p2.x + p2.y + m2.x + m2.y)) atomicOr(bad, 1);
        g[a] = cscale(cadd(csub(m2, p2), cscale(csub(p1, m1), 8.0)), 1.0 / (12.0 * h));
        lap = cadd(lap, cscale(cadd(cadd(cscale(cadd(p1, m1), 16.0), cscale(c, -30.0)), cscale(cadd(p2, m2), -1.0)),
                               1.0 / (12.0 * h * h)));
    }
    const double h2 = h * h;
    const double2 dg = cadd(make_double2(-64.0 / (15.0 * h2) + 14.0 / 15.0 * c.x, 14.0 / 15.0 * c.y),
                            cscale(csub(lap, cmul(c, c)), h2 / 20.0));
    fld[p] = make_double4(dg.x, h * g[0].x / 120.0, h * g[1].x / 120.0, h * g[2].x / 120.0);
    fldi[p] = make_double4(dg.y, h * g[0].y / 120.0, h * g[1].y / 120.0, h * g[2].y / 120.0);
}

// --------------------------------------------------------------------------- right-hand side
// F = R_h f. order 4: f + sum_a h_a^2/12 T_a f. order 6, uniform h: f + h^2/12 Lap_h f - h^4/240 sum delta^4 f +
// h^4/90 P_h f - h^2/20 k^2 f + h^4/60 sum (k^2)_nu delta_nu f, the last with (k^2)_nu = 120 g_nu / h.
// A thread owns a column of outputs over ZC planes and carries the centre values of five planes and the sums of the
// x and y neighbours of three, so a node costs 13 reads of f (5 at order 4), which the rows of a block share through
// L1, instead of 25. Bound by those reads through the caches (f, k^2 and the field block read, F written: 72 B):
// 250 x 190 x 217, order 6, 227 us (3.3 TB/s; one thread per node with 25 reads 349 us), 64^3 6.2 (8.9), 128^3 34 (56),
// 256^3 330 (526).
// order 2: the samples themselves, without the halo
__global__ void k_rhs2(const double2 *__restrict__ f, double2 *__restrict__ F, int nx, int ny, long long n) {
    const long long p = (long long)blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    const int i = (int)(p % nx), j = (int)((p / nx) % ny);
    const long long l = p / ((long long)nx * ny);
    F[p] = f[((l + 2) * (ny + 4) + (j + 2)) * (nx + 4) + (i + 2)];
}
template <int ORDER, bool KC, int ZC, int RX>
__global__ __launch_bounds__(256) void k_rhs(const double2 *__restrict__ f, const double *__restrict__ k2,
                                                    const double4 *__restrict__ fld, const double *__restrict__ k2i,
                                                    const double4 *__restrict__ fldi, double2 *__restrict__ F, int nx,
                                                    int ny, int nz, double h) {
    constexpr int RY = 256 / RX;
    const int tx = (nx + RX - 1) / RX, ty = (ny + RY - 1) / RY;
    const int T = tx * ty * ((nz + ZC - 1) / ZC);
    const int per = (T + 7) / 8;
    const int tile = (int)(blockIdx.x % 8) * per + blockIdx.x / 8;   // consecutive tiles on one XCD
    if (tile >= T) return;
    const int io = tile % tx * RX + threadIdx.x, jo = (tile / tx) % ty * RY + threadIdx.y;
    const int z0 = tile / (tx * ty) * ZC, z1 = min(z0 + ZC, nz);
    const bool ok = io < nx && jo < ny;
    const int i = min(io, nx - 1), j = min(jo, ny - 1);
    const long long px = nx + 4, pp = px * (ny + 4), plane = (long long)nx * ny;
    const double2 *c = f + (long long)(z0 + 2) * pp + (long long)(j + 2) * px + (i + 2);   // centre of plane z0
    long long o = (long long)z0 * plane + (long long)j * nx + i;
    double2 cm2, cm, c0 = c[0], cp = c[pp], Fxm, Fym, xm = c[-1], xp = c[1], ym = c[-px], yp = c[px];
    if (ORDER == 6) {
        cm2 = c[-2 * pp];
        Fxm = cadd(c[-pp - 1], c[-pp + 1]);
        Fym = cadd(c[-pp - px], c[-pp + px]);
    }
    cm = c[-pp];
    const double h2 = h * h;
    for (int l = z0; l < z1; ++l, c += pp, o += plane) {
        // plane l + 1: the neighbours; plane l + 2: the centre (order 4: both of plane l + 1)
        const double2 xmn = c[pp - 1], xpn = c[pp + 1], ymn = c[pp - px], ypn = c[pp + px];
        const double2 Fx = cadd(xm, xp), Fy = cadd(ym, yp), Fz = cadd(cm, cp);
        double2 out, cn = c[2 * pp];
        if (ORDER == 4) {
            out = cfma(1.0 / 12.0, csub(cadd(cadd(Fx, Fy), Fz), cscale(c0, 6.0)), c0);
        } else {
            const double2 x2 = cadd(c[-2], c[2]), y2 = cadd(c[-2 * px], c[2 * px]), z2 = cadd(cm2, cn);
            const double2 dg = cadd(cadd(c[-px - 1], c[-px + 1]), cadd(c[px - 1], c[px + 1]));
            const double4 fl = fld[o], fli = KC ? fldi[o] : make_double4(0, 0, 0, 0);
            const double2 kk = make_double2(k2[o], KC ? k2i[o] : 0.0);
            const double2 Fxp = cadd(xmn, xpn), Fyp = cadd(ymn, ypn);
            const double2 E = cadd(cadd(Fx, Fy), Fz);
            out = cfma(1.0 / 12.0, csub(E, cscale(c0, 6.0)), c0);
            out = cfma(-1.0 / 240.0, cadd(csub(cadd(cadd(x2, y2), z2), cscale(E, 4.0)), cscale(c0, 18.0)), out);
            // P: the xy, xz and yz products of second differences; every face enters two of them with -2
            const double2 P = cadd(cadd(dg, cadd(cadd(Fxm, Fxp), cadd(Fym, Fyp))), csub(cscale(c0, 12.0), cscale(E, 4.0)));
            out = cfma(1.0 / 90.0, P, out);
            double2 gd;
            if (KC) {
                gd = cadd(cmul(make_double2(fl.y, fli.y), csub(xp, xm)), cmul(make_double2(fl.z, fli.z), csub(yp, ym)));
                gd = cadd(gd, cmul(make_double2(fl.w, fli.w), csub(cp, cm)));
                gd = csub(gd, cscale(cmul(kk, c0), 1.0 / 20.0));
            } else {
                gd = cfma(fl.w, csub(cp, cm), cfma(fl.z, csub(yp, ym), cscale(csub(xp, xm), fl.y)));
                gd = cfma(-kk.x / 20.0, c0, gd);
            }
            out = cfma(h2, gd, out);
            cm2 = cm;
            Fxm = Fx;
            Fym = Fy;
        }
        if (ok) F[o] = out;
        cm = c0;
        c0 = cp;
        cp = cn;
        xm = xmn; xp = xpn; ym = ymn; yp = ypn;
    }
}

template <int ORDER, bool RESID, typename XT, bool KC>
__global__ __launch_bounds__(NT) void k_matvec(const XT *__restrict__ x, const double *__restrict__ k2,
                                                 const double4 *__restrict__ fld, const double2 *__restrict__ F,
                                                 double2 *__restrict__ y, StencilParams p) {
    matvec_tile<ORDER, RESID, XT, KC>(x, k2, fld, F, y, p, blockIdx.x);
}

template <typename XT, bool KC>
hipError_t launch_matvec_k(StencilParams p, const XT *x, const double *k2, const double4 *fld, const double2 *F, double2 *y,
                           hipStream_t s) {
    if (!F) { p.zchunk = p.zchunk_plain; p.zchunks = p.zchunks_plain; }
    int T = p.tiles_x * p.tiles_y * p.zchunks;
    int grid = 8 * ((T + 7) / 8);
    dim3 blk(64, TY);
    if (p.order == 6) {
        if (F) hipLaunchKernelGGL((k_matvec<6, true, XT, KC>), dim3(grid), blk, 0, s, x, k2, fld, F, y, p);
        else hipLaunchKernelGGL((k_matvec<6, false, XT, KC>), dim3(grid), blk, 0, s, x, k2, fld, F, y, p);
    } else if (p.order == 4) {
        if (F) hipLaunchKernelGGL((k_matvec<4, true, XT, KC>), dim3(grid), blk, 0, s, x, k2, fld, F, y, p);
        else hipLaunchKernelGGL((k_matvec<4, false, XT, KC>), dim3(grid), blk, 0, s, x, k2, fld, F, y, p);
    } else {
        if (F) hipLaunchKernelGGL((k_matvec<2, true, XT, KC>), dim3(grid), blk, 0, s, x, k2, fld, F, y, p);
        else hipLaunchKernelGGL((k_matvec<2, false, XT, KC>), dim3(grid), blk, 0, s, x, k2, fld, F, y, p);
    }
    return hipGetLastError();
}

template <typename XT>
hipError_t launch_matvec_t(const StencilParams &p, const XT *x, const double *k2, const double4 *fld,
                           const double2 *F, double2 *y, hipStream_t s) {
    if (p.k2i) return launch_matvec_k<XT, true>(p, x, k2, fld, F, y, s);
    return launch_matvec_k<XT, false>(p, x, k2, fld, F, y, s);
}

}  // namespace

hipError_t launch_derived_fields(const double *k2_halo, int halo, double *k2, double4 *fld, const StencilParams &p,
                                 double h, hipStream_t s) {
    long long n = (long long)p.nx * p.ny * p.nz;
    int *bad = nullptr;
    hipError_t e = hipMalloc(&bad, sizeof(int));
    if (e != hipSuccess) return e;
    e = hipMemsetAsync(bad, 0, sizeof(int), s);
    if (e != hipSuccess) { hipFree(bad); return e; }
    int blocks = (int)((n + 255) / 256);
    hipLaunchKernelGGL(k_derived, dim3(blocks), dim3(256), 0, s, k2_halo, halo, k2, fld, p.nx, p.ny, p.nz, p.order, h,
                       bad);
    e = hipGetLastError();
    int hbad = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    hipFree(bad);
    if (e != hipSuccess) return e;
    return hbad ? hipErrorInvalidValue : hipSuccess;
}

hipError_t launch_derived_fields_c(const double2 *k2_halo, int halo, double *k2, double *k2i, double4 *fld,
                                   double4 *fldi, const StencilParams &p, double h, hipStream_t s) {
    long long n = (long long)p.nx * p.ny * p.nz;
    int *bad = nullptr;
    hipError_t e = hipMalloc(&bad, sizeof(int));
    if (e != hipSuccess) return e;
    e = hipMemsetAsync(bad, 0, sizeof(int), s);
    if (e != hipSuccess) { hipFree(bad); return e; }
    int blocks = (int)((n + 255) / 256);
    hipLaunchKernelGGL(k_derived_c, dim3(blocks), dim3(256), 0, s, k2_halo, halo, k2, k2i, fld, fldi, p.nx, p.ny, p.nz,
                       p.order, h, bad);
    e = hipGetLastError();
    int hbad = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    hipFree(bad);
    if (e != hipSuccess) return e;
    return hbad ? hipErrorInvalidValue : hipSuccess;
}

// Blocks of a matvec that run at once (one per CU at order 6: 200 VGPRs, eight waves; two in the products y = A x of orders
// 2 and 4) and CUs
struct Resident { int blocks, cus; };
template <int ORDER, bool KC, bool RESID> Resident matvec_resident() {
    static const Resident r = [] {
        int dev = 0, cus = 0, nb = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_matvec<ORDER, RESID, double2, KC>, NT, 0) != hipSuccess || nb * cus <= 0)
            return Resident{256, 256};
        return Resident{nb * cus, cus};
    }();
    return r;
}
template <bool RESID> Resident matvec_resident(int order, bool kc) {
    return order == 6 ? (kc ? matvec_resident<6, true, RESID>() : matvec_resident<6, false, RESID>())
         : order == 4 ? (kc ? matvec_resident<4, true, RESID>() : matvec_resident<4, false, RESID>())
                      : (kc ? matvec_resident<2, true, RESID>() : matvec_resident<2, false, RESID>());
}

// A block of zc planes streams zc + 2 of them and costs about two more to start, and blocks run in rounds of the
// resident ones, so the length that makes rounds (zc + 4) least is taken, plus zc / 3 for the last round, which
// finishes unevenly. Measured (order 6, one product): 32^3 11.7 -> 5.6 us (1 plane per block instead of 8), 64^3 12.3 ->
// 6.9 (2), 128^3 33.0 -> 30.8 (16), 200^3 174 -> 152 (40 instead of 19), 250 x 190 x 217 194 -> 170 (28 instead of 20),
// 256^3 unchanged (32; 64 planes: 270 against 253). Two blocks on a CU take half as long again as one and start more
// slowly (seven planes): over twenty boxes that choice is the best length within 1 %, order 4, one product: 64^3 8.6 -> 5.5
// us, 128^3 17.2 -> 17.0, 200^3 92.6 -> 77.2, 310 x 300 x 31 25.1 -> 23.2 (16 planes; counted as one block each, 7: 26.7).
int matvec_chunk(StencilParams *const *ps, int count, const Resident &r) {
    const bool shared = r.blocks > r.cus;
    const double start = shared ? 7.0 : 4.0, slow = shared ? 1.5 : 1.0;
    int nzmax = 1, best = 1;
    for (int i = 0; i < count; ++i) nzmax = ps[i]->nz > nzmax ? ps[i]->nz : nzmax;
    double cost = 1e300;
    for (int zc = 1; zc <= nzmax; ++zc) {
        long long blocks = 0;
        for (int i = 0; i < count; ++i)
            blocks += (long long)ps[i]->tiles_x * ps[i]->tiles_y * ((ps[i]->nz + zc - 1) / zc);
        const long long last = blocks % r.blocks;
        const double rounds = (double)(blocks / r.blocks) * slow + (last > r.cus ? slow : last ? 1.0 : 0.0);
        const double c = rounds * (zc + start) + zc / 3.0;
        if (c < cost) { cost = c; best = zc; }
    }
    return best;
}

void stencil_split(StencilParams *const *ps, int count) {
    const int order = ps[0]->order;
    const bool kc = ps[0]->k2i != nullptr;
    const int resid = matvec_chunk(ps, count, matvec_resident<true>(order, kc));
    const int plain = matvec_chunk(ps, count, matvec_resident<false>(order, kc));
    for (int i = 0; i < count; ++i) {
        StencilParams &p = *ps[i];
        p.zchunk = resid < p.nz ? resid : p.nz;
        p.zchunks = (p.nz + p.zchunk - 1) / p.zchunk;
        p.zchunk_plain = plain < p.nz ? plain : p.nz;
        p.zchunks_plain = (p.nz + p.zchunk_plain - 1) / p.zchunk_plain;
    }
}

hipError_t launch_matvec(const StencilParams &p, const double2 *x, const double *k2, const double4 *fld,
                         const double2 *F, double2 *y, hipStream_t s) {
    return launch_matvec_t<double2>(p, x, k2, fld, F, y, s);
}

hipError_t launch_matvec(const StencilParams &p, const float2 *x, const double *k2, const double4 *fld,
                         const double2 *F, double2 *y, hipStream_t s) {
    return launch_matvec_t<float2>(p, x, k2, fld, F, y, s);
}

namespace {
template <int ORDER, bool KC, int ZC, int RX>
hipError_t rhs_launch(const StencilParams &p, const double2 *f, const double *k2, const double4 *fld, double h, double2 *F,
                      hipStream_t s) {
    constexpr int RY = 256 / RX;
    const long long T = (long long)((p.nx + RX - 1) / RX) * ((p.ny + RY - 1) / RY) * ((p.nz + ZC - 1) / ZC);
    hipLaunchKernelGGL((k_rhs<ORDER, KC, ZC, RX>), dim3((unsigned)(8 * ((T + 7) / 8))), dim3(RX, RY), 0, s, f, k2, fld, p.k2i,
                       p.fldi, F, p.nx, p.ny, p.nz, h);
    return hipGetLastError();
}
// Blocks of 32 x 8 nodes where a row's last 64 would be at most half used (24 nodes wide, 150 x 200, order 4: 10.5 -> 7.3 us,
// one thread per node 9.9; 160^3, order 6: 126 -> 86). The planes of a column follow one another at about 1 us each: four
// where 512 blocks remain (80^3, order 6: 17.3 -> 13.1 us; below, 64^3, one: 6.4 against 6.8), sixteen where 1024 do and at
// order 6 4096, whose longer columns need the more to even out (200^3, complex k^2: 240 us with four, 287 with sixteen, one
// thread per node 311; 256^3 464 and 451).
template <int ORDER, bool KC, int RX>
hipError_t rhs_columns(const StencilParams &p, const double2 *f, const double *k2, const double4 *fld, double h, double2 *F,
                       hipStream_t s) {
    constexpr int RY = 256 / RX;
    const long long planes = (long long)((p.nx + RX - 1) / RX) * ((p.ny + RY - 1) / RY) * p.nz;
    if (planes >= 16 * (ORDER == 6 ? 4096 : 1024)) return rhs_launch<ORDER, KC, 16, RX>(p, f, k2, fld, h, F, s);
    if (planes >= 4 * 512) return rhs_launch<ORDER, KC, 4, RX>(p, f, k2, fld, h, F, s);
    return rhs_launch<ORDER, KC, 1, RX>(p, f, k2, fld, h, F, s);
}
template <int ORDER, bool KC>
hipError_t rhs_width(const StencilParams &p, const double2 *f, const double *k2, const double4 *fld, double h, double2 *F,
                     hipStream_t s) {
    return (p.nx - 1) % 64 < 32 ? rhs_columns<ORDER, KC, 32>(p, f, k2, fld, h, F, s) : rhs_columns<ORDER, KC, 64>(p, f, k2, fld, h, F, s);
}
}  // namespace

hipError_t launch_rhs(const StencilParams &p, const double2 *f, const double *k2, const double4 *fld, double h, double2 *F,
                      hipStream_t s) {
    if (p.order == 2) {
        const long long n = (long long)p.nx * p.ny * p.nz;
        hipLaunchKernelGGL(k_rhs2, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, f, F, p.nx, p.ny, n);
        return hipGetLastError();
    }
    if (p.order == 4) return rhs_width<4, false>(p, f, k2, fld, h, F, s);
    return p.k2i ? rhs_width<6, true>(p, f, k2, fld, h, F, s) : rhs_width<6, false>(p, f, k2, fld, h, F, s);
}

}  // namespace helm
