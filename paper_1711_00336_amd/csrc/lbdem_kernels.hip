// HIP kernels (gfx950) of one coupled LBM-DEM time step, following Alg. 1
// of Rettinger & Ruede (arXiv 1711.00336, Sec. 3.3).
//
// Layout: cell fields are structure-of-arrays [ncomp][nc] with x fastest, so
// a 64-lane wavefront touches 64 consecutive cells of one component. PDFs
// are stored as deviations f_q - w_q (rho_0 = 1) in float or double.
// Particles are SoA [3][cap] doubles in slots that stay put between two list
// rebuilds; every subcycle sorts only their slot indices by (cell, insertion
// index). Particle -> cell transfers are gathers: every cell sums the particles
// of its 3x3x3 neighbouring 1-cell bins (contiguous ranges of the sorted
// indices), so the result is deterministic and needs no floating-point atomics.
#include "lbdem_internal.h"

#include <mutex>

#include <cmath>

namespace lbdem {

// ---------------------------------------------------------------------------
// D3Q19 velocity set: 0 rest; 1..6 +x,-x,+y,-y,+z,-z; 7..18 face diagonals
// (1,1,0),(-1,-1,0),(1,-1,0),(-1,1,0),(1,0,1),(-1,0,-1),(1,0,-1),(-1,0,1),
// (0,1,1),(0,-1,-1),(0,1,-1),(0,-1,1). Weights 1/3, 1/18, 1/36.
// Written as constexpr selectors so that unrolled loops fold to immediates.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int CX(int q)
{
    return (q == 1 || q == 7 || q == 9 || q == 11 || q == 13) ? 1
         : (q == 2 || q == 8 || q == 10 || q == 12 || q == 14) ? -1 : 0;
}
__host__ __device__ constexpr int CY(int q)
{
    return (q == 3 || q == 7 || q == 10 || q == 15 || q == 17) ? 1
         : (q == 4 || q == 8 || q == 9 || q == 16 || q == 18) ? -1 : 0;
}
__host__ __device__ constexpr int CZ(int q)
{
    return (q == 5 || q == 11 || q == 14 || q == 15 || q == 18) ? 1
         : (q == 6 || q == 12 || q == 13 || q == 16 || q == 17) ? -1 : 0;
}
__host__ __device__ constexpr int CC(int q, int a) { return a == 0 ? CX(q) : a == 1 ? CY(q) : CZ(q); }
__host__ __device__ constexpr double WQ(int q) { return q == 0 ? 1.0 / 3.0 : q <= 6 ? 1.0 / 18.0 : 1.0 / 36.0; }
__host__ __device__ constexpr int OPP(int q) { return q == 0 ? 0 : ((q & 1) ? q + 1 : q - 1); }

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2. Remap the hardware block id so that every XCD walks one contiguous
// range of logical blocks (a slab of cells or a run of cell-sorted
// particles): stencil neighbours then hit the same L2. A bijection on
// [0, nblocks) for any dispatch order, so only performance depends on it.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t nb)
{
    const uint32_t per = nb >> 3, rem = nb & 7u, x = b & 7u, idx = b >> 3;
    return x < rem ? x * (per + 1) + idx : rem * (per + 1) + (x - rem) * per + idx;
}

__device__ __forceinline__ int64_t gidx(int64_t per_block = kBlock)
{
    return (int64_t)xcd_remap(blockIdx.x, gridDim.x) * per_block + threadIdx.x;
}

// wrap a coordinate that is at most one period outside [0, n)
__device__ __forceinline__ int wrap1(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

__device__ __forceinline__ uint32_t fdiv(uint32_t c, uint32_t m, uint32_t s)
{
    return (__umulhi(c, m) + c) >> s;
}

__device__ __forceinline__ void cell_coords(const Geo &g, int64_t c64, int &i, int &j, int &k)
{
    const uint32_t c = (uint32_t)c64;
    const uint32_t kk = fdiv(c, g.mxy, g.sxy);
    const uint32_t rem = c - kk * (uint32_t)(g.n[0] * g.n[1]);
    const uint32_t jj = fdiv(rem, g.mx, g.sx);
    i = (int)(rem - jj * (uint32_t)g.n[0]);
    j = (int)jj;
    k = (int)kk;
}

__device__ __forceinline__ int64_t cidx(const Geo &g, int i, int j, int k)
{
    return (int64_t)i + (int64_t)g.n[0] * ((int64_t)j + (int64_t)g.n[1] * k);
}

// ---------------------------------------------------------------------------
// Roma et al. three-point kernel (Sec. 3.1.2, Eq. filter_def), applied per
// axis; the 3-D weight is the product over axes. Walled axes drop cells
// outside the domain and renormalise the rest to unit sum.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double roma(double r)
{
    r = fabs(r);
    if (r < 0.5) return (1.0 + sqrt(1.0 - 3.0 * r * r)) / 3.0;
    if (r < 1.5) return (5.0 - 3.0 * r - sqrt(1.0 - 3.0 * (1.0 - r) * (1.0 - r))) / 6.0;
    return 0.0;
}

// per-axis kernel weights of a particle at xp: cells b-1, b, b+1 with
// b = floor(xp); out-of-domain cells on walled axes get weight 0 and the
// others are divided by their sum.
__device__ __forceinline__ void axis_weights(double xp, int n, int per, int &b, double w[3])
{
    b = (int)floor(xp);
    if (per) b = b < 0 ? 0 : (b >= n ? n - 1 : b);
    double sum = 0.0;
#pragma unroll
    for (int o = -1; o <= 1; ++o) {
        const int i = b + o;
        const double wo = roma((double)i + 0.5 - xp);
        if (per || (i >= 0 && i < n)) {
            w[o + 1] = wo;
            sum += wo;
        } else {
            w[o + 1] = 0.0;
        }
    }
    if (!per) {
#pragma unroll
        for (int o = 0; o < 3; ++o) w[o] /= sum;
    }
}

// cell coordinate of stencil offset o (clamped on walled axes, where the
// weight of an out-of-domain offset is zero)
__device__ __forceinline__ int stencil_coord(int b, int o, int n, int per)
{
    int i = b + o;
    if (per) return wrap1(i, n);
    return i < 0 ? 0 : (i >= n ? n - 1 : i);
}

// distinct wrapped coordinates c-r..c+r on one axis, in this order also where
// they are all cells of it, as the gather tiles take them (walled: in range only)
__device__ __forceinline__ int axis_range(int c, int r, int n, int per, int *out, int cap)
{
    int m = 0;
    if (per) {
        if (2 * r + 1 > n) {
            for (int i = 0; i < n && m < cap; ++i) out[m++] = i;
        } else {
            for (int o = -r; o <= r; ++o) out[m++] = wrap1(c + o, n);
        }
    } else {
        for (int o = -r; o <= r; ++o) {
            const int i = c + o;
            if (i >= 0 && i < n) out[m++] = i;
        }
    }
    return m;
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

__device__ __forceinline__ int64_t particle_cell(const Geo &g, double x, double y, double z)
{
    const int i = clampi((int)floor(x), 0, g.n[0] - 1);
    const int j = clampi((int)floor(y), 0, g.n[1] - 1);
    const int k = clampi((int)floor(z), 0, g.n[2] - 1);
    return cidx(g, i, j, k);
}

__device__ __forceinline__ double sphere_volume(double d) { return M_PI * d * d * d / 6.0; }

// 4-vector cell fields ([nc][4], a vector and a scalar that is read with it, or
// 0): one 16- or 32-byte access per cell instead of three or four scattered ones
__device__ __forceinline__ void store_vec4(float *p, float a, float b, float c, float d = 0.0f)
{
    *reinterpret_cast<float4 *>(p) = make_float4(a, b, c, d);
}
__device__ __forceinline__ void store_vec4(double *p, double a, double b, double c, double d = 0.0)
{
    reinterpret_cast<double2 *>(p)[0] = make_double2(a, b);
    reinterpret_cast<double2 *>(p)[1] = make_double2(c, d);
}
__device__ __forceinline__ void load_vec4(const float *p, float v[4])
{
    const float4 t = *reinterpret_cast<const float4 *>(p);
    v[0] = t.x;
    v[1] = t.y;
    v[2] = t.z;
    v[3] = t.w;
}
__device__ __forceinline__ void load_vec4(const double *p, double v[4])
{
    const double2 a = reinterpret_cast<const double2 *>(p)[0], b = reinterpret_cast<const double2 *>(p)[1];
    v[0] = a.x;
    v[1] = a.y;
    v[2] = b.x;
    v[3] = b.y;
}

// u_f of a cell with its eps_p: 4-vectors in the FP32 form, [3][nc] beside eps_p
// in the FP64 form. There a 4-vector is two 16-byte stores 32 bytes apart, which
// cost the gathers that write u_f in every subcycle more than the drag pass gains
// by reading it whole: 128^3 cells with 64 thousand spheres, per subcycle, gathers
// 118 us as [3][nc] and 128 as 4-vectors, drag 99 and 93 us; with lift gathers 159
// and 174 us.
__device__ __forceinline__ void store_uf(const Cells<float> &C, int64_t, int64_t c, const float u[3], float ep)
{
    store_vec4(C.uf + 4 * c, u[0], u[1], u[2], ep);
}
__device__ __forceinline__ void store_uf(const Cells<double> &C, int64_t nc, int64_t c, const double u[3], double)
{
#pragma unroll
    for (int b = 0; b < 3; ++b) C.uf[b * nc + c] = u[b];
}
__device__ __forceinline__ void load_uf(const Cells<float> &C, int64_t, int64_t c, float v[4])
{
    load_vec4(C.uf + 4 * c, v);
}
__device__ __forceinline__ void load_uf(const Cells<double> &C, int64_t nc, int64_t c, double v[4])
{
#pragma unroll
    for (int b = 0; b < 3; ++b) v[b] = C.uf[b * nc + c];
    v[3] = C.epsp[c];
}

// ---------------------------------------------------------------------------
// a1: moments of the post-stream PDFs (Eq. MacVel): rho - 1 = sum df,
// j = sum c df (exact with deviations since sum_q w_q c_q = 0).
// ---------------------------------------------------------------------------
template <typename R>
__global__ __launch_bounds__(kBlock) void k_moments(Desc D, Cells<R> C)
{
    const int64_t nc = D.g.nc;
    const int64_t c = gidx();
    if (c >= nc) return;
    R r = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        const R f = C.df_src[q * nc + c];
        r += f;
        if (CX(q) > 0) jx += f; else if (CX(q) < 0) jx -= f;
        if (CY(q) > 0) jy += f; else if (CY(q) < 0) jy -= f;
        if (CZ(q) > 0) jz += f; else if (CZ(q) < 0) jz -= f;
    }
    store_vec4(C.j + 4 * c, jx, jy, jz, r);
    // fluid-phase velocity with the body force only (Eq. MacVel, u_f = u_bar/eps_f);
    // with lift also the first subcycle's u_f, from which its curl is taken
    const double e = 1.0 - (double)C.epsp[c];
    const double rho = 1.0 + (double)r;
    const R u0 = (R)(((double)jx + 0.5 * e * D.p.fb[0]) / (rho * e));
    const R u1 = (R)(((double)jy + 0.5 * e * D.p.fb[1]) / (rho * e));
    const R u2 = (R)(((double)jz + 0.5 * e * D.p.fb[2]) / (rho * e));
    store_vec4(C.un + 4 * c, u0, u1, u2, r);
    if (D.p.use_lift) {
        const R uf[3] = {u0, u1, u2};
        store_uf(C, nc, c, uf, C.epsp[c]);
    }
}

// Neighbours x + c_q with the wall ghost rule: the mirrored in-domain cell;
// a velocity flips sign once per mirrored axis (no-slip at the half-way
// plane), a scalar keeps its value. Resolved once per cell and axis: o[a][d+1]
// is the flat-index term of coordinate (i_a + d) (times 1, nx or nx*ny;
// 32-bit, since a domain has fewer than 2^31 cells) and s[a][d+1] the sign a
// velocity takes there.
struct Nbh {
    int o[3][3];
    double s[3][3];
};

__device__ __forceinline__ void neighbourhood(const Geo &g, int i, int j, int k, Nbh &h)
{
    const int c[3] = {i, j, k};
    const int stride[3] = {1, g.n[0], g.n[0] * g.n[1]};
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int d = -1; d <= 1; ++d) {
            int t = c[a] + d;
            double sg = 1.0;
            if (t < 0 || t >= g.n[a]) {
                if (g.per[a]) t = wrap1(t, g.n[a]);
                else {
                    t = c[a];
                    sg = -1.0;
                }
            }
            h.o[a][d + 1] = t * stride[a];
            h.s[a][d + 1] = sg;
        }
}

// flat index and velocity sign of neighbour x + c_q (q a compile-time constant
// in unrolled loops, so the table lookups are register selects)
__device__ __forceinline__ int ghost(const Nbh &h, int q, double &sign)
{
    sign = h.s[0][CX(q) + 1] * h.s[1][CY(q) + 1] * h.s[2][CZ(q) + 1];
    return h.o[0][CX(q) + 1] + h.o[1][CY(q) + 1] + h.o[2][CZ(q) + 1];
}

// ---------------------------------------------------------------------------
// a2/a3: per-step cell fields (Alg. 1, the step before the subcycle loop,
// which keeps the material derivative fixed for the whole LBM step):
//   u_f^n = (j + eps_f f_b / 2) / (rho eps_f)      (Eq. MacVel, u_f = u_bar/eps_f)
//   Du_f/Dt = (u_f^n - u_prev) + (u_f^n . grad_L) u_f^n (0 time part at step 0)
//   grad P = (1/c_s^2) sum_q w_q c_q P(x+c_q) = sum_q w_q c_q (rho-1)(x+c_q)
// with the lattice gradient of Sec. 3.2.3. Also resets f_acc.
// ---------------------------------------------------------------------------
template <typename R>
__global__ __launch_bounds__(kBlock) void k_cellfields(Desc D, Cells<R> C)
{
    const int64_t nc = D.g.nc;
    const int64_t c = gidx();
    if (c >= nc) return;
    int i, j, k;
    cell_coords(D.g, c, i, j, k);
    Nbh h;
    neighbourhood(D.g, i, j, k, h);
    double G[3][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
    double gp[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        double sg;
        const int64_t nb = ghost(h, q, sg);
        R v[4];
        load_vec4(C.un + 4 * nb, v);
        const double u0 = (double)v[0], u1 = (double)v[1], u2 = (double)v[2], dr = (double)v[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (CC(q, a) == 0) continue;
            const double wc = CC(q, a) > 0 ? WQ(q) : -WQ(q);
            G[a][0] += wc * (sg * u0);
            G[a][1] += wc * (sg * u1);
            G[a][2] += wc * (sg * u2);
            gp[a] += wc * dr;
        }
    }
    R un0[4];
    load_vec4(C.un + 4 * c, un0);
    const double un[3] = {(double)un0[0], (double)un0[1], (double)un0[2]};
    const bool have_prev = *D.stepc > 0;
    R du[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        double conv = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) conv += un[a] * (3.0 * G[a][b]);
        const double dtu = have_prev ? (un[b] - (double)C.uprev[b * nc + c]) : 0.0;
        du[b] = (R)(dtu + conv);
        C.uprev[b * nc + c] = (R)un[b];
        C.facc[b * nc + c] = (R)0;
    }
    store_vec4(C.gradp + 4 * c, (R)gp[0], (R)gp[1], (R)gp[2]);
    store_vec4(C.dudt + 4 * c, du[0], du[1], du[2]);
}

// ---------------------------------------------------------------------------
// Lift only, at every subcycle start (Alg. 1, the first step inside the
// subcycle loop, which also needs u_f; grad P depends on rho alone and comes
// from the per-step pass): the lattice curl of Sec. 3.2.3,
//   curl u_f(x) = (1/c_s^2) sum_q w_q c_q x u_f(x + c_q),
// of the subcycle-start u_f = (j + eps_f f_b / 2) / (rho eps_f) that the
// moments pass (first subcycle) or the volume-fraction gather (later ones)
// leaves in uf; neighbours beyond a wall by the velocity ghost rule above.
// ---------------------------------------------------------------------------
template <typename R>
__global__ __launch_bounds__(kBlock) void k_curl(Desc D, Cells<R> C)
{
    const int64_t nc = D.g.nc;
    const int64_t c = gidx();
    if (c >= nc) return;
    int i, j, k;
    cell_coords(D.g, c, i, j, k);
    Nbh h;
    neighbourhood(D.g, i, j, k, h);
    double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 1; q < 19; ++q) {
        double sg;
        const int64_t nb = ghost(h, q, sg);
        R v[4];
        load_uf(C, nc, nb, v);
        const double u0 = sg * (double)v[0], u1 = sg * (double)v[1], u2 = sg * (double)v[2];
        s[0] += WQ(q) * (CY(q) * u2 - CZ(q) * u1);
        s[1] += WQ(q) * (CZ(q) * u0 - CX(q) * u2);
        s[2] += WQ(q) * (CX(q) * u1 - CY(q) * u0);
    }
    store_vec4(C.curl + 4 * c, (R)(3.0 * s[0]), (R)(3.0 * s[1]), (R)(3.0 * s[2]));
}

// ---------------------------------------------------------------------------
// a4: added mass (Table 1): F_am = C_am rho_f V (Du_f/Dt|_p - du_p/dt), the
// fluid derivative interpolated with Eq. interpolation. Also records the
// subcycle-start velocity and position.
// ---------------------------------------------------------------------------
struct Stencil {
    int b[3];
    double w[3][3];
};

// stored kernel weight u (= 3*axis + o+1) of slot p, in the storage precision
template <typename R> __device__ __forceinline__ R stencil_weight(const Parts &P, int u, int64_t p);
template <> __device__ __forceinline__ float stencil_weight<float>(const Parts &P, int u, int64_t p)
{
    return P.swf[u * P.cap + p];
}
template <> __device__ __forceinline__ double stencil_weight<double>(const Parts &P, int u, int64_t p)
{
    return P.sw[u * P.cap + p];
}

template <typename R> __device__ __forceinline__ void load_stencil(const Parts &P, int64_t i, Stencil &st)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        st.b[a] = P.sb[a * P.cap + i];
#pragma unroll
        for (int o = 0; o < 3; ++o) st.w[a][o] = (double)stencil_weight<R>(P, 3 * a + o, i);
    }
}

// kernel stencil of a particle at x, stored for slot s; the weights left in st
// are the stored ones (rounded to FP32 in the FP32 form)
__device__ __forceinline__ void store_stencil(const Desc &D, int64_t s, const double x[3], Stencil &st)
{
    const Parts &P = D.pt;
    const int64_t cap = P.cap;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        int b;
        double wt[3];
        axis_weights(x[a], D.g.n[a], D.g.per[a], b, wt);
        P.sb[a * cap + s] = b;
        st.b[a] = b;
#pragma unroll
        for (int o = 0; o < 3; ++o) {
            if (P.swf) {
                const float f = (float)wt[o];
                P.swf[(3 * a + o) * cap + s] = f;
                st.w[a][o] = (double)f;
            } else {
                P.sw[(3 * a + o) * cap + s] = wt[o];
                st.w[a][o] = wt[o];
            }
        }
    }
}

// st.w[a][o] for a runtime o without indexing a register array
__device__ __forceinline__ double sel3(const double w[3], int o) { return o == 0 ? w[0] : (o == 1 ? w[1] : w[2]); }

// F_am = C_am rho_f V (Du/Dt|p - a_p) (Table 1) of slot i from the particle's
// diameter, du_p/dt, velocity and position; records the subcycle-start
// velocity and position (a single substep has them at hand)
template <typename R>
__device__ __forceinline__ void am_store(const Desc &D, int64_t i, const R Du[3], double d, const double a[3],
                                         const double u[3], const double x[3])
{
    const Parts &P = D.pt;
    const int64_t cap = P.cap;
    const R V = (R)sphere_volume(d);
    const R cam = (R)(D.p.c_am * D.p.rho_f);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const R F = D.p.use_am ? cam * V * (Du[b] - (R)a[b]) : (R)0;
        P.Fam[b * cap + i] = (double)F;
        if (D.p.n_dem > 1) {
            P.ustart[b * cap + i] = u[b];
            P.xstart[b * cap + i] = x[b];
        }
    }
}

// the same for the particle in slot i (subcycle start state)
template <typename R> __device__ __forceinline__ void am_force(const Desc &D, int64_t i, const R Du[3])
{
    const Parts &P = D.pt;
    const int64_t cap = P.cap;
    double a[3], u[3] = {0.0, 0.0, 0.0}, x[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        a[b] = P.a[b * cap + i];
        if (D.p.n_dem > 1) {
            u[b] = P.u[b * cap + i];
            x[b] = P.x[b * cap + i];
        }
    }
    am_store<R>(D, i, Du, P.d[i], a, u, x);
}

// Du_f/Dt|p = sum of the 27 stencil cells' Du_f/Dt with the stored weights
// (Eq. interpolation), summed in R in the order (z, y, x)
template <typename R>
__device__ __forceinline__ void interp_dudt(const Desc &D, const Cells<R> &C, const Stencil &st, R Du[3])
{
#pragma unroll 1
    for (int oz = 0; oz < 3; ++oz) {
        const int cz = stencil_coord(st.b[2], oz - 1, D.g.n[2], D.g.per[2]);
#pragma unroll
        for (int oy = 0; oy < 3; ++oy) {
            const int cy = stencil_coord(st.b[1], oy - 1, D.g.n[1], D.g.per[1]);
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
                const int cx = stencil_coord(st.b[0], ox - 1, D.g.n[0], D.g.per[0]);
                const int64_t cell = cidx(D.g, cx, cy, cz);
                const R w = (R)(st.w[0][ox] * st.w[1][oy] * sel3(st.w[2], oz));
                R v[4];
                load_vec4(C.dudt + 4 * cell, v);
#pragma unroll
                for (int b = 0; b < 3; ++b) Du[b] += w * v[b];
            }
        }
    }
}

// F_l = 1.61 d^2 sqrt(mu rho_f / |w_f|) ((u_f|p - u_p) x w_f) (Table 1, lift),
// w_f = (curl u_f)|p; zero where w_f = 0 (the formula's limit). u_p and u_f
// are those of the subcycle start.
template <typename R> __device__ __forceinline__ void lift_force(const Desc &D, int64_t i, const R uf[3], const R om[3])
{
    const Parts &P = D.pt;
    const int64_t cap = P.cap;
    const R on = sqrt(om[0] * om[0] + om[1] * om[1] + om[2] * om[2]);
    R F[3] = {(R)0, (R)0, (R)0};
    if (on > (R)0) {
        R w[3];
#pragma unroll
        for (int b = 0; b < 3; ++b) w[b] = uf[b] - (R)P.u[b * cap + i];
        const R d = (R)P.d[i];
        const R s = (R)1.61 * d * d * sqrt((R)D.p.mu * (R)D.p.rho_f / on);
        F[0] = s * (w[1] * om[2] - w[2] * om[1]);
        F[1] = s * (w[2] * om[0] - w[0] * om[2]);
        F[2] = s * (w[0] * om[1] - w[1] * om[0]);
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) P.Fl[b * cap + i] = (double)F[b];
}

// interpolation sums and the added-mass force (and with LIFT the lift from
// the interpolated u_f and curl u_f) in the cell precision R (FP32 in the
// FP32-deviation form); the forces are stored FP64
template <typename R, bool LIFT>
__global__ __launch_bounds__(kBlock) void k_part_am(Desc D, Cells<R> C)
{
    const int64_t i = gidx();
    const Parts &P = D.pt;
    if (i >= P.np) return;
    Stencil st;
    load_stencil<R>(P, i, st);
    R Du[3] = {(R)0, (R)0, (R)0};
    R U[3] = {(R)0, (R)0, (R)0}, Om[3] = {(R)0, (R)0, (R)0};
    if (!LIFT) {
        interp_dudt<R>(D, C, st, Du);
        am_force<R>(D, i, Du);
        return;
    }
#pragma unroll 1
    for (int oz = 0; oz < 3; ++oz) {
        const int cz = stencil_coord(st.b[2], oz - 1, D.g.n[2], D.g.per[2]);
#pragma unroll
        for (int oy = 0; oy < 3; ++oy) {
            const int cy = stencil_coord(st.b[1], oy - 1, D.g.n[1], D.g.per[1]);
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
                const int cx = stencil_coord(st.b[0], ox - 1, D.g.n[0], D.g.per[0]);
                const int64_t cell = cidx(D.g, cx, cy, cz);
                const R w = (R)(st.w[0][ox] * st.w[1][oy] * sel3(st.w[2], oz));
                R v[4];
                load_vec4(C.dudt + 4 * cell, v);
#pragma unroll
                for (int b = 0; b < 3; ++b) Du[b] += w * v[b];
                if (LIFT) {
                    R o[4], uf[4];
                    load_vec4(C.curl + 4 * cell, o);
                    load_uf(C, D.g.nc, cell, uf);
#pragma unroll
                    for (int b = 0; b < 3; ++b) {
                        U[b] += w * uf[b];
                        Om[b] += w * o[b];
                    }
                }
            }
        }
    }
    am_force<R>(D, i, Du);
    if (LIFT) lift_force<R>(D, i, U, Om);
}

// ---------------------------------------------------------------------------
// Gather of a particle quantity to one cell (Eq. distribution_filter with
// D = I): s = sum_p D(x, x_p) v_p over the particles of the 3x3x3
// neighbouring bins. The slot list is sorted by cell, so each x-row of three
// bins is one contiguous range of it.
// ---------------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ double stencil_w(const Parts &P, int64_t p, int axis, int ic, int n, int per)
{
    const int b = P.sb[axis * P.cap + p];
    int o = ic - b;
    if (per) {
        if (n < 3) {  // several stencil offsets land on the same cell
            double w = 0.0;
#pragma unroll
            for (int t = -1; t <= 1; ++t)
                if (wrap1(b + t, n) == ic) w += (double)stencil_weight<R>(P, 3 * axis + t + 1, p);
            return w;
        }
        o = o > 1 ? o - n : (o < -1 ? o + n : o);
    }
    return (o >= -1 && o <= 1) ? (double)stencil_weight<R>(P, 3 * axis + o + 1, p) : 0.0;
}

// weights and values in the storage precision R, products accumulated in
// FP64 (the same arithmetic as the LDS tiles, so all variants agree)
template <typename R, int NV, typename F>
__device__ __forceinline__ void gather_range(const Desc &D, int i, int j, int k, int p0, int p1, const F &val,
                                             double *s)
{
    for (int q0 = p0; q0 < p1; ++q0) {
        const int p = D.b.list[q0];
        const R wx = (R)stencil_w<R>(D.pt, p, 0, i, D.g.n[0], D.g.per[0]);
        const R wy = (R)stencil_w<R>(D.pt, p, 1, j, D.g.n[1], D.g.per[1]);
        const R wz = (R)stencil_w<R>(D.pt, p, 2, k, D.g.n[2], D.g.per[2]);
        const R w = wx * wy * wz;
        if (w == (R)0) continue;
        double v[NV];
        val(p, v);
#pragma unroll
        for (int q = 0; q < NV; ++q) s[q] += (double)w * (double)(R)v[q];
    }
}

template <typename R, int NV, typename F>
__device__ __forceinline__ void gather_cell(const Desc &D, int i, int j, int k, const F &val, double *s)
{
    int cx[3], cy[3], cz[3];
    const int mx = axis_range(i, 1, D.g.n[0], D.g.per[0], cx, 3);
    const int my = axis_range(j, 1, D.g.n[1], D.g.per[1], cy, 3);
    const int mz = axis_range(k, 1, D.g.n[2], D.g.per[2], cz, 3);
    // one contiguous x-run of bins when the row does not wrap
    const bool run = mx == 3 && cx[0] + 2 == cx[2];
#pragma unroll
    for (int t = 0; t < NV; ++t) s[t] = 0.0;
    for (int a = 0; a < mz; ++a)
        for (int b = 0; b < my; ++b) {
            if (run) {
                const int64_t b0 = cidx(D.g, cx[0], cy[b], cz[a]);
                gather_range<R, NV>(D, i, j, k, D.b.start[b0], D.b.start[b0 + 3], val, s);
            } else {
                for (int c = 0; c < mx; ++c) {
                    const int64_t bin = cidx(D.g, cx[c], cy[b], cz[a]);
                    gather_range<R, NV>(D, i, j, k, D.b.start[bin], D.b.start[bin + 1], val, s);
                }
            }
        }
}

// ---------------------------------------------------------------------------
// LDS-tiled gather. A workgroup owns a TX x TY x (TZ*CZ) tile of cells, each
// thread CZ consecutive cells along z. It counts the particles of the tile's
// halo bins (the tile widened by one cell, wrapped on periodic axes), notes
// their places in the sorted slot list in LDS (a bin is one contiguous range of
// that list, noted by the thread that owns the bin), stages their stencils and
// values into LDS one entry per thread (gathers through the list, independent
// of each other; slots are close to list order), and then every cell sums the
// particles of its own 3x3x3 bins from LDS, in the order (dz, dy, dx, insertion
// index) whatever the tile shape and the slots. Tiles whose halo holds more
// than KMAX particles are staged in runs of halo planes; only where one plane
// exceeds KMAX does the tile fall back to the per-cell global gather. (Half-cell
// spheres at solid fraction 0.3, 4.6 per cell, 16^3 cells, FP64: 47 us
// for the volume fraction with the added mass, 425 us per cell, which reads
// every particle's 13 values once per cell of its stencil.)
//   MODE_AM : fam  = -sum_p D (F_am + F_l)            (Eq. forces_pf, added mass, lift)
//   MODE_FD : facc += (eps_f f_b + fam - sum_p D F_d) / n_int   (mean f_ext)
//   MODE_EPS: epsp = sum_p D V_p                      (Eq. fluid_volume_fraction)
//   MODE_EPS_AM: both of the new positions: the volume fraction at the end of
//            one subcycle and the added-mass spreading of the next one
//   MODE_EPS_UF: the volume fraction and, for the lift's curl, the next
//            subcycle's starting u_f = (j + eps_f f_b/2) / (rho eps_f)
// MODE_AM and MODE_EPS_AM also store the re-evaluated fluid-phase velocity
// u_f = (j + (eps_f f_b + fam)/2) / (rho eps_f) (Sec. 3.2.3, Alg. 1).
// ---------------------------------------------------------------------------
enum { MODE_AM = 0, MODE_FD = 1, MODE_EPS = 2, MODE_EPS_AM = 3, MODE_EPS_UF = 4 };

template <int MODE> struct GatherNV {
    static constexpr int v = (MODE == MODE_EPS || MODE == MODE_EPS_UF) ? 1 : (MODE == MODE_EPS_AM ? 4 : 3);
};

template <int MODE>
__device__ __forceinline__ void gather_value(const Parts &P, int p, double *v)
{
    if (MODE == MODE_EPS || MODE == MODE_EPS_UF) {
        v[0] = sphere_volume(P.d[p]);
    } else if (MODE == MODE_EPS_AM) {
        v[0] = sphere_volume(P.d[p]);
        v[1] = P.Fam[p];
        v[2] = P.Fam[P.cap + p];
        v[3] = P.Fam[2 * P.cap + p];
    } else {
        const double *F = MODE == MODE_AM ? P.Fam : P.Fd;
        v[0] = F[p];
        v[1] = F[P.cap + p];
        v[2] = F[2 * P.cap + p];
        if (MODE == MODE_AM && P.Fl) {  // lift, spread together with the added mass
            v[0] += P.Fl[p];
            v[1] += P.Fl[P.cap + p];
            v[2] += P.Fl[2 * P.cap + p];
        }
    }
}

// fam = -sam and u_f = (j + (eps_f f_b + fam)/2) / (rho eps_f) of cell c with the
// solid fraction ep, which u_f keeps for the drag pass
template <typename R>
__device__ __forceinline__ void store_fam_uf(const Desc &D, const Cells<R> &C, int64_t c, R ep, const double *sam)
{
    const int64_t nc = D.g.nc;
    R j[4], uf[3];
    load_vec4(C.j + 4 * c, j);
    const double e = 1.0 - (double)ep;
    const double rho = 1.0 + (double)j[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const R fam = (R)(-sam[b]);
        C.fam[b * nc + c] = fam;
        const double fext = e * D.p.fb[b] + (double)fam;
        uf[b] = (R)(((double)j[b] + 0.5 * fext) / (rho * e));
    }
    store_uf(C, nc, c, uf, ep);
}

template <typename R, int MODE>
__device__ __forceinline__ void gather_store(const Desc &D, const Cells<R> &C, int64_t c, const double *s)
{
    if (MODE == MODE_AM) {
        store_fam_uf<R>(D, C, c, C.epsp[c], s);
    } else if (MODE == MODE_EPS_AM) {
        const double e = 1.0 - s[0];
        if (!(e > 0.0) || !isfinite(e)) atomicOr(D.flags, FLAG_EPS);
        C.epsp[c] = (R)s[0];
        store_fam_uf<R>(D, C, c, (R)s[0], s + 1);
    } else if (MODE == MODE_FD) {
        const int64_t nc = D.g.nc;
        const double e = 1.0 - (double)C.epsp[c];
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const double fext = e * D.p.fb[b] + (double)C.fam[b * nc + c] - s[b];
            C.facc[b * nc + c] = (R)((double)C.facc[b * nc + c] + fext * D.p.dt_int);
        }
        if (c == 0) {  // requests that have been served, before this subcycle's substeps make new ones
#pragma unroll
            for (int t = 0; t < 2; ++t)
                if (D.clear & (1 << t)) D.pt.need[t] = 0;
        }
    } else {
        const double e = 1.0 - s[0];
        if (!(e > 0.0) || !isfinite(e)) atomicOr(D.flags, FLAG_EPS);
        C.epsp[c] = (R)s[0];
        if (MODE == MODE_EPS_UF) {
            R j[4], uf[3];
            load_vec4(C.j + 4 * c, j);
            const double ef = 1.0 - (double)(R)s[0];
            const double rho = 1.0 + (double)j[3];
#pragma unroll
            for (int b = 0; b < 3; ++b) uf[b] = (R)(((double)j[b] + 0.5 * ef * D.p.fb[b]) / (rho * ef));
            store_uf(C, D.g.nc, c, uf, (R)s[0]);
        }
    }
}

template <typename R, int MODE, int TX, int TY, int TZ, int CZ, int KMAX>
__global__ __launch_bounds__(TX *TY *TZ) void k_gather_tile(Desc D, Cells<R> C)
{
    constexpr int NT = TX * TY * TZ, HX = TX + 2, HY = TY + 2, HZ = TZ * CZ + 2, NHB = HX * HY * HZ;
    constexpr int NV = GatherNV<MODE>::v;
    constexpr int PER = (NHB + NT - 1) / NT;
    constexpr int NW = NT / 64;
    static_assert(NT % 64 == 0, "whole wavefronts");
    __shared__ int hoff[NHB + 1];
    __shared__ int wsum[NW];
    // staged weights and values in the storage precision R (halves LDS in the
    // FP32 form); products are accumulated in FP64
    __shared__ R sw_l[9][KMAX];
    __shared__ R sv_l[NV][KMAX];
    __shared__ int sslot[KMAX];  // position in the sorted slot list of each staged entry

    const int tid = threadIdx.x;
    const int n0 = D.g.n[0], n1 = D.g.n[1], n2 = D.g.n[2];
    const uint32_t lin = xcd_remap(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z),
                                   gridDim.x * gridDim.y * gridDim.z);
    const int bx = (int)(lin % gridDim.x), by = (int)((lin / gridDim.x) % gridDim.y),
              bz = (int)(lin / (gridDim.x * gridDim.y));
    const int x0 = bx * TX, y0 = by * TY, z0 = bz * TZ * CZ;
    // halo bins beyond the last cell of a partial tile (+1) are not needed
    const int lx = min(x0 + TX, n0) - x0 + 1, ly = min(y0 + TY, n1) - y0 + 1,
              lz = min(z0 + TZ * CZ, n2) - z0 + 1;

    // each thread owns PER consecutive halo bins
    int src[PER], cnt[PER];
    int sum = 0;
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const int hb = tid * PER + t;
        src[t] = 0;
        cnt[t] = 0;
        if (hb < NHB) {
            const int hx = hb % HX, hy = (hb / HX) % HY, hz = hb / (HX * HY);
            int g[3] = {x0 - 1 + hx, y0 - 1 + hy, z0 - 1 + hz};
            bool ok = hx <= lx && hy <= ly && hz <= lz;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                if (g[a] < 0 || g[a] >= D.g.n[a]) {
                    if (D.g.per[a]) g[a] = wrap1(g[a], D.g.n[a]);
                    else ok = false;
                }
            }
            if (ok) {
                const int64_t bin = cidx(D.g, g[0], g[1], g[2]);
                src[t] = D.b.start[bin];
                cnt[t] = D.b.start[bin + 1] - src[t];
            }
        }
        sum += cnt[t];
    }
    // exclusive scan of the per-thread counts: wavefront shuffles, then the
    // wavefront totals through LDS (one barrier)
    const int lane = tid & 63, wv = tid >> 6;
    int incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int run = incl - sum, K = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int ws = wsum[w];
        if (w < wv) run += ws;
        K += ws;
    }
    // offsets of the halo bins
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        const int hb = tid * PER + t;
        if (hb < NHB) hoff[hb] = run;
        run += cnt[t];
    }
    if (tid == NT - 1) hoff[NHB] = K;
    __syncthreads();
    const Parts &P = D.pt;

    const int tx = tid % TX, ty = (tid / TX) % TY, tz = tid / (TX * TY);
    const int i = x0 + tx, j = y0 + ty, kb = z0 + tz * CZ;
    const bool own = i < n0 && j < n1;
    double s[CZ][NV];

    // a halo plane that alone exceeds the staging buffer: per-cell gather from
    // global memory
    bool crowded = false;
    if (K > KMAX)
        for (int h = 0; h < HZ; ++h) crowded |= hoff[(h + 1) * HX * HY] - hoff[h * HX * HY] > KMAX;
    if (crowded) {
        if (!own) return;
#pragma unroll
        for (int c = 0; c < CZ; ++c) {
            if (kb + c >= n2) break;
            gather_cell<R, NV>(D, i, j, kb + c, [&](int p, double *v) { gather_value<MODE>(D.pt, p, v); }, s[c]);
            gather_store<R, MODE>(D, C, cidx(D.g, i, j, kb + c), s[c]);
        }
        return;
    }

#pragma unroll
    for (int c = 0; c < CZ; ++c)
#pragma unroll
        for (int t = 0; t < NV; ++t) s[c][t] = 0.0;
    // The halo is staged in runs of whole z-planes, as many as fit the buffer:
    // all of them at once in all but crowded tiles. A cell takes its three
    // planes in ascending order whatever the runs, so the order of its sum
    // does not depend on them.
    for (int h0 = K > 0 ? 0 : HZ, h1; h0 < HZ; h0 = h1) {  // (empty tiles have nothing to sum)
        const int base = hoff[h0 * HX * HY];
        // (the usual tile fits whole: searching for its last plane, a chain of LDS
        // reads, would take longer than the rest of an empty one)
        h1 = K - base <= KMAX ? HZ : h0 + 1;
        while (h1 < HZ && hoff[(h1 + 1) * HX * HY] - base <= KMAX) ++h1;
        const int nk = hoff[h1 * HX * HY] - base;
        if (h0 > 0) __syncthreads();
        // the list position of every staged entry (written by the thread that
        // owns the bin: LDS stores only) ...
#pragma unroll
        for (int t = 0; t < PER; ++t) {
            const int hb = tid * PER + t;
            if (hb >= h0 * HX * HY && hb < h1 * HX * HY)
                for (int q = 0; q < cnt[t]; ++q) sslot[hoff[hb] - base + q] = src[t] + q;
        }
        __syncthreads();
        // ... then the staging of weights and values, one entry per thread, so
        // that a wavefront's loads are independent (same entries, same order)
        for (int kk = tid; kk < nk; kk += NT) {
            const int p = D.b.list[sslot[kk]];
#pragma unroll
            for (int u = 0; u < 9; ++u) sw_l[u][kk] = stencil_weight<R>(P, u, p);
            double v[NV];
            gather_value<MODE>(P, p, v);
#pragma unroll
            for (int u = 0; u < NV; ++u) sv_l[u][kk] = (R)v[u];
        }
        __syncthreads();
        if (!own) continue;
        // The bin of a staged particle fixes its stencil offset relative to a
        // cell: a particle in bin (i-1+dx, j-1+dy, k-1+dz) sees the cell at offset
        // (1-dx, 1-dy, 1-dz), i.e. weight slots 2-dx, 2-dy, 2-dz of its axes.
        // Halo row r (z = kb - 1 + r) feeds the thread's cells c with dz = r - c.
#pragma unroll
        for (int r = 0; r < CZ + 2; ++r) {
            const int hz = tz * CZ + r;
            if (hz < h0 || hz >= h1) continue;
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                const int hb0 = (hz * HY + (ty + dy)) * HX + tx;
                const int k0 = hoff[hb0] - base, k1 = hoff[hb0 + 1] - base, k2 = hoff[hb0 + 2] - base,
                          k3 = hoff[hb0 + 3] - base;
                for (int kk = k0; kk < k3; ++kk) {
                    const int sx = kk < k1 ? 2 : (kk < k2 ? 1 : 0);
                    const R wxy = sw_l[sx][kk] * sw_l[3 + 2 - dy][kk];
                    R v[NV];
#pragma unroll
                    for (int t = 0; t < NV; ++t) v[t] = sv_l[t][kk];
#pragma unroll
                    for (int c = 0; c < CZ; ++c) {
                        const int dz = r - c;
                        if (dz < 0 || dz > 2) continue;
                        const R w = wxy * sw_l[6 + 2 - dz][kk];
#pragma unroll
                        for (int t = 0; t < NV; ++t) s[c][t] += (double)w * (double)v[t];
                    }
                }
            }
        }
    }
    if (!own) return;
#pragma unroll
    for (int c = 0; c < CZ; ++c)
        if (kb + c < n2) gather_store<R, MODE>(D, C, cidx(D.g, i, j, kb + c), s[c]);
}

// per-cell global gather (thin periodic axes, where a cell's neighbour bins coincide)
template <typename R, int MODE>
__global__ __launch_bounds__(kBlock) void k_gather_cells(Desc D, Cells<R> C)
{
    const int64_t nc = D.g.nc;
    const int64_t c = gidx();
    if (c >= nc) return;
    int i, j, k;
    cell_coords(D.g, c, i, j, k);
    constexpr int NV = GatherNV<MODE>::v;
    double s[NV];
    gather_cell<R, NV>(D, i, j, k, [&](int p, double *v) { gather_value<MODE>(D.pt, p, v); }, s);
    gather_store<R, MODE>(D, C, c, s);
}

// ---------------------------------------------------------------------------
// a6: pressure-gradient force, drag, gravity + buoyancy (Table 1, Sec. 3.1.2)
// with u_f re-evaluated from f_ext = eps_f f_b + f_am (Sec. 3.2.3 stability
// measures; Alg. 1, the u_f update between the two particle loops).
// ---------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ T drag_factor(T Re, T ep)
{
    const T e1 = (T)1 - ep;
    const T cd0 = (T)1 + (T)0.15 * (Re > (T)0 ? pow(Re, (T)0.687) : (T)0);
    const T A = (T)5.81 * ep / (e1 * e1 * e1) + (T)0.48 * (ep > (T)0 ? cbrt(ep) : (T)0) / (e1 * e1 * e1 * e1);
    const T B = ep * ep * ep * Re * ((T)0.95 + (T)0.61 * ep * ep * ep / (e1 * e1));
    const T cd = e1 * (cd0 / (e1 * e1 * e1) + A + B);
    return e1 * cd;
}

// F_pr = -V grad P|p, F_d (Tenneti closure as the paper prints it, Table 1),
// gravity and buoyancy; F_const for the DEM substeps
template <typename R>
__device__ __forceinline__ void drag_forces(const Desc &D, int64_t i, const R uf[3], const R gp[3], R ep, int record)
{
    const Parts &P = D.pt;
    const int64_t cap = P.cap;
    const double dd = P.d[i];
    const R d = (R)dd;
    const R V = (R)sphere_volume(dd);
    const R mu = (R)D.p.mu, rho_f = (R)D.p.rho_f;
    R wv[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) wv[b] = uf[b] - (R)P.u[b * cap + i];
    const R wn = sqrt(wv[0] * wv[0] + wv[1] * wv[1] + wv[2] * wv[2]);
    const R Re = ((R)1 - ep) * rho_f * d * wn / mu;
    const R fac = (R)3 * (R)M_PI * d * mu * drag_factor(Re, ep);
    const R rp = (R)P.rho[i];
    const int pid = record ? P.id[i] : 0;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const R Fpr = -V * gp[b];
        const R Fd = fac * wv[b];
        const R fgb = (rp - rho_f) * V * (R)D.p.g[b];
        const R Fam = (R)P.Fam[b * cap + i];
        const R Fl = P.Fl ? (R)P.Fl[b * cap + i] : (R)0;
        const R Fc = Fd + Fpr + Fam + Fl + fgb;
        P.Fd[b * cap + i] = (double)Fd;
        P.Fc[b * cap + i] = (double)Fc;
        if (record) {
            P.Fam_id[b * cap + pid] = (double)Fam;
            P.Fd_id[b * cap + pid] = (double)Fd;
            P.Fpr_id[b * cap + pid] = (double)Fpr;
            P.Fc_id[b * cap + pid] = (double)Fc;
            if (P.Fl_id) P.Fl_id[b * cap + pid] = (double)Fl;
        }
    }
}

// interpolation sums and the closures in the cell precision R (FP32 in the
// FP32-deviation form); the forces are stored FP64
template <typename R>
__global__ __launch_bounds__(kBlock) void k_part_drag(Desc D, Cells<R> C, int record)
{
    const int64_t i = gidx();
    const Parts &P = D.pt;
    if (i >= P.np) return;
    Stencil st;
    load_stencil<R>(P, i, st);
    R uf[3] = {(R)0, (R)0, (R)0}, gp[3] = {(R)0, (R)0, (R)0}, ep = (R)0;
#pragma unroll 1
    for (int oz = 0; oz < 3; ++oz) {
        const int cz = stencil_coord(st.b[2], oz - 1, D.g.n[2], D.g.per[2]);
#pragma unroll
        for (int oy = 0; oy < 3; ++oy) {
            const int cy = stencil_coord(st.b[1], oy - 1, D.g.n[1], D.g.per[1]);
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
                const int cx = stencil_coord(st.b[0], ox - 1, D.g.n[0], D.g.per[0]);
                const int64_t cell = cidx(D.g, cx, cy, cz);
                const R w = (R)(st.w[0][ox] * st.w[1][oy] * sel3(st.w[2], oz));
                R u4[4], g4[4];
                load_uf(C, D.g.nc, cell, u4);
                load_vec4(C.gradp + 4 * cell, g4);
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    uf[b] += w * u4[b];
                    gp[b] += w * g4[b];
                }
                ep += w * u4[3];
            }
        }
    }
    drag_forces<R>(D, i, uf, gp, ep, record);
}

// ---------------------------------------------------------------------------
// LDS-tiled particle pass (a6 drag/pressure/gravity, and a4's added mass
// with lift; without lift the added mass runs per particle). A workgroup owns
// the particles whose bins lie in a TX x TY x TZ tile of cells (one contiguous
// range of the sorted slot list per x-row of bins). It loads the cell fields of
// the tile widened by one cell (wrapped on periodic axes, clamped on walled
// ones, as the per-particle stencil does) into LDS with coalesced loads, and
// every particle interpolates from LDS. The arithmetic and its order are
// those of k_part_am / k_part_drag, so the results are bit-identical.
// ---------------------------------------------------------------------------
//
// The cell fields come as 4-vectors, (u_f, eps_p) and grad P for the drag, Du/Dt,
// u_f and the curl for the added mass with lift: two or three 16-byte accesses
// per cell instead of seven or nine 4-byte ones (but see store_uf). In LDS the
// drag keeps all four components; the added mass the three that it reads, which
// lets three workgroups of the FP64 form share a CU, not two (128^3 cells, 64
// thousand spheres: 117 us against 136).
enum { PASS_DRAG = 1, PASS_AML = 2 };

template <typename R, int PASS, int TX, int TY, int TZ, int NT>
__global__ __launch_bounds__(NT) void k_part_tile(Desc D, Cells<R> C, int record)
{
    constexpr int HX = TX + 2, HY = TY + 2, HZ = TZ + 2, NHC = HX * HY * HZ;
    constexpr int NF = PASS == PASS_DRAG ? 2 : 3;  // 4-vectors per cell
    constexpr int NR = TY * TZ;
    static_assert(NR <= 64, "rows of one tile are scanned by one wavefront");
    constexpr int NC = PASS == PASS_DRAG ? 4 : 3;  // components kept
    __shared__ __align__(16) R cv[NF][NHC][NC];
    __shared__ int rp[NR + 1], rsrc[NR];

    const int tid = threadIdx.x;
    const int n0 = D.g.n[0], n1 = D.g.n[1], n2 = D.g.n[2];
    const uint32_t lin = xcd_remap(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z),
                                   gridDim.x * gridDim.y * gridDim.z);
    const int bx = (int)(lin % gridDim.x), by = (int)((lin / gridDim.x) % gridDim.y),
              bz = (int)(lin / (gridDim.x * gridDim.y));
    const int x0 = bx * TX, y0 = by * TY, z0 = bz * TZ;
    const int xe = min(x0 + TX, n0);
    const int lx = xe - x0 + 1, ly = min(y0 + TY, n1) - y0 + 1, lz = min(z0 + TZ, n2) - z0 + 1;

    // own particles: one range of the slot list per row of bins
    if (tid < 64) {
        int cnt = 0, src = 0;
        if (tid < NR) {
            const int y = y0 + tid % TY, z = z0 + tid / TY;
            if (y < n1 && z < n2) {
                src = D.b.start[cidx(D.g, x0, y, z)];
                cnt = D.b.start[cidx(D.g, xe - 1, y, z) + 1] - src;
            }
            rsrc[tid] = src;
        }
        int incl = cnt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(incl, off, 64);
            if ((tid & 63) >= off) incl += y;
        }
        if (tid < NR) rp[tid] = incl - cnt;
        if (tid == NR - 1) rp[NR] = incl;
    }
    // where most tiles are empty, they end before reading their cells
    if (D.pt.np < (int64_t)gridDim.x * gridDim.y * gridDim.z) {
        __syncthreads();
        if (rp[NR] == 0) return;
    }
    // halo cell fields
    constexpr int FU = PASS == PASS_DRAG ? 0 : 1;  // place of u_f
    const R *field[3] = {C.dudt, C.gradp, C.curl};
    for (int hc = tid; hc < NHC; hc += NT) {
        const int hx = hc % HX, hy = (hc / HX) % HY, hz = hc / (HX * HY);
        R v[NF][4];
        if (hx <= lx && hy <= ly && hz <= lz) {
            const int gx = stencil_coord(x0, hx - 1, n0, D.g.per[0]);
            const int gy = stencil_coord(y0, hy - 1, n1, D.g.per[1]);
            const int gz = stencil_coord(z0, hz - 1, n2, D.g.per[2]);
            const int64_t cell = cidx(D.g, gx, gy, gz);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                if (f == FU) load_uf(C, D.g.nc, cell, v[f]);
                else load_vec4(field[f] + 4 * cell, v[f]);
            }
        } else {
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int t = 0; t < 4; ++t) v[f][t] = (R)0;
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if constexpr (NC == 4) store_vec4(cv[f][hc], v[f][0], v[f][1], v[f][2], v[f][3]);
            else
#pragma unroll
                for (int t = 0; t < 3; ++t) cv[f][hc][t] = v[f][t];
        }
    }
    __syncthreads();

    const Parts &P = D.pt;
    const int K = rp[NR];
    for (int k = tid; k < K; k += NT) {
        int lo = 0, hi = NR - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (rp[mid] <= k) lo = mid;
            else hi = mid - 1;
        }
        const int64_t i = D.b.list[rsrc[lo] + (k - rp[lo])];
        Stencil st;
        load_stencil<R>(P, i, st);
        // the stencil base is the particle's bin, inside this tile; the clamp
        // only keeps LDS indices in range for a particle already flagged as
        // having left the domain
        const int hx0 = min(max(st.b[0] - x0, 0), TX - 1), hy0 = min(max(st.b[1] - y0, 0), TY - 1),
                  hz0 = min(max(st.b[2] - z0, 0), TZ - 1);
        R acc[NF][4];
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[f][t] = (R)0;
#pragma unroll 1
        for (int oz = 0; oz < 3; ++oz) {
#pragma unroll
            for (int oy = 0; oy < 3; ++oy) {
#pragma unroll
                for (int ox = 0; ox < 3; ++ox) {
                    const int hc = ((hz0 + oz) * HY + (hy0 + oy)) * HX + (hx0 + ox);
                    const R w = (R)(st.w[0][ox] * st.w[1][oy] * sel3(st.w[2], oz));
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        R v[4];
                        if constexpr (NC == 4) load_vec4(cv[f][hc], v);
                        else
#pragma unroll
                            for (int t = 0; t < 3; ++t) v[t] = cv[f][hc][t];
#pragma unroll
                        for (int t = 0; t < (PASS == PASS_DRAG && f == 0 ? 4 : 3); ++t) acc[f][t] += w * v[t];
                    }
                }
            }
        }
        if (PASS == PASS_AML) {
            am_force<R>(D, i, acc[0]);
            lift_force<R>(D, i, acc[1], acc[NF - 1]);
        } else {
            drag_forces<R>(D, i, acc[0], acc[1], acc[0][3], record);
        }
    }
}

// ---------------------------------------------------------------------------
// a8: DEM (Sec. 3.1.1) + lubrication (Sec. 3.1.3) forces of one substep.
// ---------------------------------------------------------------------------
// Pair and wall forces are evaluated in FP64 in both storage forms: FP32 pair
// arithmetic was measured to cost ~5e-5 relative error per step in dense,
// lubrication-dominated packings. In the FP32-deviation form the velocities,
// spins and masses come from the packed records, rounded to FP32.
struct PV {
    double x[3], d, m;          // position, diameter, mass
    double u[3];
};

template <typename T> __device__ __forceinline__ void cross3(const T a[3], const T b[3], T c[3])
{
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}
template <typename T> __device__ __forceinline__ T dot3(const T a[3], const T b[3])
{
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// 1/x in FP64 from the hardware reciprocal estimate refined by two Newton
// steps (error below one ulp of the correctly rounded quotient for the
// positive, normal arguments used here): a third of the instructions of a
// full IEEE division
__device__ __forceinline__ double rcp64(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}

// max(a, b) in one instruction: fmax also quiets signalling NaNs, which costs an
// instruction per operand (no signalling NaN arises here; with a quiet one both
// return the other operand)
__device__ __forceinline__ double max_f64(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// fma in its three-operand form: with the coefficients of a series kept in
// registers the compiler otherwise copies each one and accumulates onto the copy
__device__ __forceinline__ double fma_keep(double a, double b, double c)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Square root of a non-negative double that is not huge (below 1e300): one
// coupled Newton step from the hardware's inverse root, then two residual
// corrections, correctly rounded as the library's root is, whose range scaling
// and special cases cost as many instructions again. The clamp keeps the root
// of 0 (coinciding centres, which the reciprocal then turns into a flagged
// non-finite force) at 0.
__device__ __forceinline__ double sqrt_pos(double x)
{
    const double y = __builtin_amdgcn_rsq(max_f64(x, 1e-280));
    double g = x * y, h = 0.5 * y;
    double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    e = fma(-g, g, x);
    g = fma(e, h, g);
    e = fma(-g, g, x);
    return fma(e, h, g);
}

// Natural logarithm of a positive normal double: x = 2^k m with m in
// [1/sqrt 2, sqrt 2) and ln m = 2 atanh(s), s = (m - 1)/(m + 1), so that
// |s| <= 3 - 2 sqrt 2 = 0.1716, summed as the Taylor series of atanh through
// s^19 (the first omitted term is below 3e-17 of the sum). Within 2 ulp of
// the correctly rounded logarithm; about a third of the instructions of the
// general library logarithm, which also handles zero, negative, subnormal
// and non-finite arguments (the lubrication logarithm ln(<d>/2h) only sees
// gaps h >= h_min > 0).
__device__ __forceinline__ double log_pos(double x)
{
    double m = __builtin_amdgcn_frexp_mant(x);  // x = m 2^k, m in [1/2, 1)
    int k = __builtin_amdgcn_frexp_exp(x);
    if (m < M_SQRT1_2) {
        m += m;
        --k;
    }
    const double s = (m - 1.0) * rcp64(m + 1.0);
    const double z = s * s;
    double q = 1.0 / 19.0;
    q = fma_keep(q, z, 1.0 / 17.0);
    q = fma_keep(q, z, 1.0 / 15.0);
    q = fma_keep(q, z, 1.0 / 13.0);
    q = fma_keep(q, z, 1.0 / 11.0);
    q = fma_keep(q, z, 1.0 / 9.0);
    q = fma_keep(q, z, 1.0 / 7.0);
    q = fma_keep(q, z, 1.0 / 5.0);
    q = fma_keep(q, z, 1.0 / 3.0);
    const double t = s + s;
    return fma((double)k, M_LN2, fma(t * z, q, t));
}

// spring-dashpot normal force and Coulomb-limited tangential force Fc = F^n + F^t
// and n x F^t; the torque about the centre is (d_i/2) n x F^t (the moment of F^t
// at the contact point)
__device__ __forceinline__ void contact(const Phys &p, double delta, const double n[3], const double ur[3], double mij,
                                        double Fc[3], double tq[3])
{
    const double kn = mij * p.kn_per_m;
    const double xi = mij * p.xi_per_m;
    const double urn_s = dot3(ur, n);
    double urn[3], urt[3], Fn[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        urn[a] = urn_s * n[a];
        urt[a] = ur[a] - urn[a];
        Fn[a] = -kn * delta * n[a] - xi * urn[a];
    }
    const double urt_n = sqrt(dot3(urt, urt));
    double Ft[3] = {0.0, 0.0, 0.0};
    if (urt_n > 0.0) {
        const double fn_n = sqrt(dot3(Fn, Fn));
        const double mag = fmin(p.mu_c * fn_n, xi * urt_n) * rcp64(urt_n);
#pragma unroll
        for (int a = 0; a < 3; ++a) Ft[a] = -mag * urt[a];
    }
    cross3(n, Ft, tq);
#pragma unroll
    for (int a = 0; a < 3; ++a) Fc[a] = Fn[a] + Ft[a];
}

// Eq. lubrication_force, applied for h < h_c with h := max(h, h_min) and,
// when lub_stab is set, h >= 3 pi mu <d>^2 dt_DEM / (8 r m_ij) with r = 1/4:
// the leading squeeze term then relaxes one pair by at most a quarter of
// its relative velocity per substep, so a sphere with a full shell of
// partners at the floor (up to (12 + 1)/2 times one pair's rate) stays
// below the explicit limit 2 - 2 C_am rho_f/rho_p; inv_dm = 1/<d>.
// With lub_contact = 0 only on the open gap (h > 0). The reduced mass is
// passed as m_ij = m_prod / m_sum.
__device__ __forceinline__ void lubrication(const Phys &p, double h, double dm, double inv_dm, double m_prod,
                                            double m_sum, const double n[3], const double upr[3], double F[3])
{
    if (!(h < p.h_c)) return;
    if (!p.lub_contact && !(h > 0.0)) return;  // open gap only
    const double mu = p.mu;
    const double pi = M_PI;
    double he = max_f64(h, p.h_min);
    if (p.lub_stab) {
        // he = max(he, c / (2 m_ij)) with m_ij = m_prod / m_sum, compared
        // without the division, which only the few pairs at the floor need
        const double c = 3.0 * pi * mu * dm * dm * p.dt_dem * m_sum;
        if (he * (2.0 * m_prod) < c) he = c * rcp64(2.0 * m_prod);
    }
    // 1/he and 1/(he + <d>) from one reciprocal
    const double q = rcp64(he * (he + dm));
    const double inv_he = (he + dm) * q;
    const double s = 2.0 * he * q;
    const double Lg = log_pos(dm * 0.5 * inv_he);
    const double asq = 1.5 * pi * mu * dm * (dm * 0.25 * inv_he + (18.0 / 40.0) * Lg + (9.0 / 84.0) * (he * inv_dm) * Lg);
    const double ash = 0.5 * pi * mu * dm * Lg * (dm + he) * (dm + he) / 4.0;
    const double un = dot3(upr, n);
#pragma unroll
    for (int a = 0; a < 3; ++a) F[a] += -asq * un * n[a] - ash * s * s * (upr[a] - un * n[a]);
}

// contact of the pair (i, j) with spins wi, wj at centre offset dx = x_j - x_i;
// false, and nothing done, if the spheres do not overlap
__device__ __forceinline__ bool pair_contact(const Phys &p, const PV &pi, const double wi[3], const PV &pj,
                                             const double wj[3], const double dx[3], double Fc[3], double tq[3])
{
    const double ri = 0.5 * pi.d, rj = 0.5 * pj.d;
    const double dist = sqrt_pos(dot3(dx, dx));
    const double delta = ri + rj - dist;
    if (!(delta > 0.0)) return false;
    const double inv = rcp64(dist);
    const double n[3] = {dx[0] * inv, dx[1] * inv, dx[2] * inv};
    const double mij = pi.m * pj.m * rcp64(pi.m + pj.m);
    double s[3], ur[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) s[a] = ri * wi[a] + rj * wj[a];
    cross3(s, n, ur);
#pragma unroll
    for (int a = 0; a < 3; ++a) ur[a] += pi.u[a] - pj.u[a];
    contact(p, delta, n, ur, mij, Fc, tq);
    return true;
}

// lubrication of the pair (i, j) at the unit normal n and the overlap delta =
// r_i + r_j - dist
__device__ __forceinline__ void pair_lubrication(const Phys &p, const PV &pi, const PV &pj, const double n[3],
                                                 double delta, double F[3])
{
    // <d> = 2 d_i d_j / (d_i + d_j) and its inverse from one reciprocal
    const double sd = pi.d + pj.d, pd = pi.d * pj.d;
    const double q = rcp64(sd * pd);
    const double dm = 2.0 * pd * pd * q;
    const double inv_dm = 0.5 * sd * sd * q;
    const double upr[3] = {pi.u[0] - pj.u[0], pi.u[1] - pj.u[1], pi.u[2] - pj.u[2]};
    lubrication(p, -delta, dm, inv_dm, pi.m * pj.m, pi.m + pj.m, n, upr, F);
}

__device__ __forceinline__ void wall_interaction(const Phys &p, const Geo &g, const PV &pi, const double w[3],
                                                 double F[3], double Tq[3])
{
    const double r = 0.5 * pi.d;
    for (int a = 0; a < 3; ++a) {
        if (g.per[a]) continue;
        for (int side = 0; side < 2; ++side) {
            const double dist = side == 0 ? pi.x[a] : (double)g.n[a] - pi.x[a];
            double n[3] = {0.0, 0.0, 0.0};
            n[a] = side == 0 ? -1.0 : 1.0;
            const double delta = r - dist;
            if (delta > 0.0) {
                double s[3], ur[3];
#pragma unroll
                for (int b = 0; b < 3; ++b) s[b] = r * w[b];
                cross3(s, n, ur);
#pragma unroll
                for (int b = 0; b < 3; ++b) ur[b] += pi.u[b];
                double Fc[3], tq[3];
                contact(p, delta, n, ur, pi.m, Fc, tq);
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    F[b] += Fc[b];
                    Tq[b] += r * tq[b];
                }
            }
            if (p.use_lub) lubrication(p, -delta, 2.0 * pi.d, 0.5 * rcp64(pi.d), pi.m, 1.0, n, pi.u, F);
        }
    }
}

// 16-byte pieces of a particle's DEM record
template <int N> __device__ __forceinline__ void copy_quads(const void *src, void *dst)
{
    const uint4 *s = reinterpret_cast<const uint4 *>(src);
    uint4 *d = reinterpret_cast<uint4 *>(dst);
#pragma unroll
    for (int k = 0; k < N; ++k) d[k] = s[k];
}

template <typename R>
__device__ __forceinline__ void store_rec(DemRec<R> *pk, int64_t i, const double x[3], const double u[3],
                                          const double w[3], double d, R m)
{
    DemRec<R> r;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        r.x[a] = x[a];
        r.u[a] = (R)u[a];
        r.w[a] = (R)w[a];
    }
    r.d = d;
    r.m = m;
    r.pad = (R)0;
    copy_quads<sizeof(DemRec<R>) / 16>(&r, pk + i);
}

// what the lubrication reads of a record (all but the spin and the padding), in
// 16-byte pieces: the first 48 or 64 bytes
template <typename R> __host__ __device__ constexpr int rec_pieces()
{
    return (4 * sizeof(double) + 4 * sizeof(R)) / 16;
}
template <typename R> __device__ __forceinline__ void unpack_rec(const uint4 *pieces, PV &v)
{
    DemRec<R> r;
    copy_quads<rec_pieces<R>()>(pieces, &r);
    v.d = r.d;
    v.m = (double)r.m;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        v.x[a] = r.x[a];
        v.u[a] = (double)r.u[a];
    }
}
template <typename R> __device__ __forceinline__ void load_rec(const DemRec<R> *pk, int64_t i, PV &v)
{
    unpack_rec<R>(reinterpret_cast<const uint4 *>(pk + i), v);
}
template <typename R> __device__ __forceinline__ void load_spin(const DemRec<R> *pk, int64_t i, double w[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) w[a] = (double)pk[i].w[a];
}

// Once a step has flagged instability (non-finite or runaway particles),
// the domain's state is no longer meaningful and is reported at the next
// sync. The binning and neighbour-search kernels then do nothing: positions
// that are no longer finite all clamp into one cell, and sorting or
// scanning such a bin would take time quadratic in the particle count.
// (These kernels have no barriers, so a per-thread check is safe.)
__device__ __forceinline__ bool halted(const Desc &D) { return *(volatile const int *)D.flags != 0; }

// whether this step starts with a reordering of the slots (need[1] is set
// during a step and cleared by the first drag spreading of the next)
__device__ __forceinline__ bool reorder_due(const Desc &D) { return D.pt.need[1] != 0 && !halted(D); }

__device__ __forceinline__ void min_image(const Geo &g, double dx[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a)
        if (g.per[a]) {
            // lengths as kernel arguments: converted here they would sit in 18 VGPRs
            const double d = dx[a];
            dx[a] = d > g.half[a] ? d - g.len[a] : (d < -g.half[a] ? d + g.len[a] : d);
        }
}

// Verlet lists (neighbour search for the sums of Eq. forces_collision,
// Eq. torques_collision and Eq. lubrication_force, which only reach
// (d_i + d_j)/2 + h_c). A list holds the slots of every particle within that
// reach plus a skin, in ascending insertion index, so the force sums run in an
// order that does not depend on when the list was built. Rebuilt only when a
// particle could move half the skin from where it was at the build within the
// next subcycle (integrate_particle); slots do not move between two builds.
//
// One wavefront per particle: the lanes take the rows of bins around it, then
// the candidates of those rows (found by a search in the rows' running counts);
// accepted ones are compacted by ballot and ranked by insertion index among
// themselves in LDS. 3.17 M dense spheres, 260 candidates and 29.6 entries each:
// 6 ms per build; 24 ms when one thread per particle walked the rows and
// kept its list sorted in global memory.
//
// Entry t of slot i is stored at list_base(i) + 64 t: the lists of 64
// consecutive slots are interleaved, so that a wavefront with one lane per
// particle reads 64 consecutive entries.
constexpr int kListLds = 512;  // entries per wavefront sorted in LDS; longer lists are sorted in place

__device__ __forceinline__ int64_t list_base(const Parts &P, int64_t i)
{
    return (i >> 6) * ((int64_t)P.nbr << 6) + (i & 63);
}

// cells c-r..c+r of one axis: `count` of them from lo (wrapped where it leaves
// the domain; all cells once where the range covers a periodic axis)
__device__ __forceinline__ void search_range(int c, int r, int n, int per, int &lo, int &count)
{
    lo = c - r;
    count = 2 * r + 1;
    if (per) {
        if (count >= n) {
            lo = 0;
            count = n;
        }
        return;
    }
    const int hi = min(c + r, n - 1);
    lo = max(lo, 0);
    count = hi - lo + 1;
}

// position and diameter from a record
template <typename R>
__device__ __forceinline__ void load_sphere(const DemRec<R> *pk, int64_t i, double x[3], double &d)
{
    const double2 *q = reinterpret_cast<const double2 *>(pk + i);
    const double2 a = q[0], b = q[1];
    x[0] = a.x;
    x[1] = a.y;
    x[2] = b.x;
    d = b.y;
}

// the list of slot i, by one wavefront; lds: 2 kListLds ints of its own. Neighbours
// beyond the capacity raise FLAG_NLIST if `flag`.
template <typename R>
__device__ __forceinline__ void build_list(const Desc &D, const DemRec<R> *pk, int64_t i, int lane, int *lds,
                                           bool flag)
{
    const Parts &P = D.pt;
    int *sid = lds, *ssl = lds + kListLds;
    const int64_t cap = P.cap;
    const double gap = (D.p.use_lub ? fmax(D.p.h_c, 0.0) : 0.0) + D.p.vskin;
    const int r = D.p.rbin, n0 = D.g.n[0];
    double xi[3], ri;
    load_sphere(pk, i, xi, ri);
    ri *= 0.5;
    int lo[3], ct[3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
        search_range(clampi((int)floor(xi[a]), 0, D.g.n[a] - 1), r, D.g.n[a], D.g.per[a], lo[a], ct[a]);
    // an x-row is one contiguous run of bins, or two where it wraps
    const int nrun = lo[0] < 0 || lo[0] + ct[0] > n0 ? 2 : 1;
    const int nseg = nrun * ct[1] * ct[2];
    const int64_t base = list_base(P, i);
    int m = 0;
    for (int g0 = 0; g0 < nseg; g0 += 64) {
        const int g = g0 + lane;
        int q0 = 0, cnt = 0;
        if (g < nseg) {
            const int half = g % nrun, row = g / nrun;
            const int y = wrap1(lo[1] + row % ct[1], D.g.n[1]), z = wrap1(lo[2] + row / ct[1], D.g.n[2]);
            int a = lo[0], b = lo[0] + ct[0];  // bins a..b-1
            if (nrun == 2) {
                if (a < 0) { a += n0; b += n0; }
                if (half) { a = 0; b -= n0; } else b = n0;
            }
            q0 = D.b.start[cidx(D.g, a, y, z)];
            cnt = D.b.start[cidx(D.g, b - 1, y, z) + 1] - q0;
        }
        int incl = cnt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(incl, off, 64);
            if (lane >= off) incl += t;
        }
        const int total = __shfl(incl, 63, 64);
        for (int k0 = 0; k0 < total; k0 += 64) {
            const int k = k0 + lane;
            // the row of candidate k: the number of rows that end at or before it
            int row = 0;
#pragma unroll
            for (int step = 32; step > 0; step >>= 1)
                if (__shfl(incl, row + step - 1, 64) <= k) row += step;
            const int q = __shfl(q0, row & 63, 64) + k - (__shfl(incl, row & 63, 64) - __shfl(cnt, row & 63, 64));
            int j = -1;
            if (k < total) {
                j = D.b.list[q];
                double dx[3], dj;
                load_sphere(pk, j, dx, dj);
#pragma unroll
                for (int a = 0; a < 3; ++a) dx[a] -= xi[a];
                min_image(D.g, dx);
                const double reach = ri + 0.5 * dj + gap;
                if (j == i || dot3(dx, dx) >= reach * reach) j = -1;
            }
            const uint64_t acc = __ballot(j >= 0);
            if (j >= 0) {
                const int t = m + __popcll(acc & ((1ull << lane) - 1));
                if (t < kListLds) {
                    sid[t] = P.id[j];
                    ssl[t] = j;
                } else if (t < P.nbr) {
                    P.nlist[base + 64 * (int64_t)t] = j;
                }
            }
            m += __popcll(acc);
        }
    }
    if (m > P.nbr) {
        if (flag && lane == 0) atomicOr(D.flags, FLAG_NLIST);
        m = P.nbr;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (m <= kListLds) {
        for (int e = lane; e < m; e += 64) {
            const int key = sid[e];
            int rank = 0;
            for (int t = 0; t < m; ++t) rank += sid[t] < key;
            P.nlist[base + 64 * (int64_t)rank] = ssl[e];
        }
    } else if (lane == 0) {
        for (int t = 0; t < m; ++t) {
            const int j = t < kListLds ? ssl[t] : P.nlist[base + 64 * (int64_t)t];
            const int key = P.id[j];
            int b = t - 1;
            while (b >= 0 && P.id[P.nlist[base + 64 * (int64_t)b]] > key) {
                P.nlist[base + 64 * (int64_t)(b + 1)] = P.nlist[base + 64 * (int64_t)b];
                --b;
            }
            P.nlist[base + 64 * (int64_t)(b + 1)] = j;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (lane == 0) {
        P.nnb[i] = m;
#pragma unroll
        for (int a = 0; a < 3; ++a) P.xbuild[a * cap + i] = xi[a];
    }
}

template <typename R> __global__ __launch_bounds__(kBlock) void k_nlist(Desc D, bool flag)
{
    __shared__ int lds[kBlock / 64][2 * kListLds];
    const Parts &P = D.pt;
    if (P.need[0] == 0 || halted(D)) return;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // a workgroup takes a run of slots, whose candidates it then finds in its cache
    const int64_t per = (P.np + gridDim.x - 1) / gridDim.x, b0 = xcd_remap(blockIdx.x, gridDim.x) * per;
    const int64_t b1 = b0 + per < P.np ? b0 + per : P.np;
    for (int64_t i = b0 + wv; i < b1; i += kBlock / 64)
        build_list<R>(D, (const DemRec<R> *)P.pk, i, lane, lds[wv], flag);
}

// what the last substep of a subcycle does besides integrating
enum : int {
    SUB_LAST = 1,  // du_p/dt, kernel stencil of the new position, bin count, list check
    SUB_AM = 2,    // the next subcycle's added-mass force (without lift, except before a step's end)
    SUB_END = 4    // the last subcycle of a step: ask for a reordering ahead of the next step
};

// One semi-implicit Euler substep of particle i (R5: u and omega first,
// then x) under the contact and lubrication force F and torque Tq of the
// substep and the subcycle's frozen F_const, with the wall, skin and
// finiteness checks; rec: where the particle's new DEM record goes. The last
// substep of a subcycle leaves everything that the next one reads of the
// particle: du_p/dt, the kernel stencil and, while they are in registers, the
// added-mass force (a4 without lift), so that no separate pass over the
// particles does it.
//
// FUSED: own is the particle's view in the substep's record src. Position,
// diameter (and the FP64 form's mass) are taken from it and the position goes
// back to the state arrays at the subcycle's end only; wavefronts without any
// torque leave the spins alone. A substep then moves 236 B per particle (FP32
// form, without the lists) instead of 390, a lone substep with everything it
// leaves for the next subcycle 356 instead of 560.
template <typename R, bool FUSED>
__device__ __forceinline__ void integrate_particle(const Desc &D, const Cells<R> &C, int64_t i, int sub,
                                                   const double F[3], const double Tq[3], const PV &own,
                                                   const DemRec<R> *src, DemRec<R> *rec)
{
    const Parts &P = D.pt;
    const int64_t cap = P.cap;
    const bool single = D.p.n_dem == 1;  // the subcycle starts at this substep's start
    const double d = FUSED ? own.d : P.d[i];
    const double m = FUSED && sizeof(R) == 8 ? own.m : P.rho[i] * sphere_volume(d);
    const double I = m * d * d / 10.0;
    const double dt = D.p.dt_dem;
    // loaded together: between the stores below each load would wait for its own
    // trip to memory (substep of 18 thousand dense spheres 15.3 -> 14.9 us)
    double u0[3], Fc[3], xs[3], xb[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t k = a * cap + i;
        u0[a] = P.u[k];
        Fc[a] = P.Fc[k];
        xs[a] = single ? 0.0 : P.xstart[k];
        xb[a] = sub & SUB_LAST ? P.xbuild[k] : 0.0;
    }
    double x[3], u[3], w[3], acc[3];
    const bool spin = !FUSED || __any(Tq[0] != 0.0 || Tq[1] != 0.0 || Tq[2] != 0.0);
    if (!spin) load_spin<R>(src, i, w);
    int bad = 0;
    double ahead2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t k = a * cap + i;
        const double x0 = FUSED ? own.x[a] : P.x[k];
        u[a] = u0[a] + dt * (Fc[a] + F[a]) / m;
        P.u[k] = u[a];
        if (spin) {
            w[a] = P.w[k] + dt * Tq[a] / I;
            P.w[k] = w[a];
        }
        double xa = x0 + dt * u[a];
        const double L = D.g.len[a];
        if (D.g.per[a]) {
            if (xa >= L) xa -= L;
            else if (xa < 0.0) {
                xa += L;
                if (xa >= L) xa = 0.0;
            }
        } else if (!(xa > 0.0 && xa < L)) {
            bad |= FLAG_WALL;
        }
        if (!isfinite(xa) || !isfinite(u[a])) bad |= FLAG_NONFINITE;
        if (!FUSED || (sub & SUB_LAST)) P.x[k] = xa;
        x[a] = xa;
        double dx = xa - (single ? x0 : xs[a]);
        if (D.g.per[a]) dx -= L * rint(dx / L);
        if (fabs(dx) > D.p.skin) bad |= FLAG_SKIN;
        if (sub & SUB_LAST) {
            acc[a] = (u[a] - (single ? u0[a] : P.ustart[k])) / D.p.dt_int;
            P.a[k] = acc[a];
            double db = xa - xb[a];
            if (D.g.per[a]) db -= L * rint(db / L);
            const double reach = fabs(db) + D.p.skin;
            ahead2 += reach * reach;
        }
    }
    if (bad) atomicOr(D.flags, bad);
    // the record feeds the next substep's pair loop
    store_rec<R>(rec, i, x, u, w, d, FUSED ? (R)own.m : (R)m);
    if (!(sub & SUB_LAST)) return;
    // A list holds every pair within reach as long as no particle has moved
    // vskin/2 since its build. The next subcycle adds at most `skin` per axis
    // (else it is flagged), so the farthest a particle can get in it is the
    // corner |db| + skin of a box: rebuild first where that lies vskin/2 away.
    // (Comparing the axes one by one with vskin/2 - skin would let two spheres
    // close in by 0.17 along a diagonal, with a skin of 0.1.) At a step's end the
    // reordering (and with it the rebuild) is asked for a little earlier, so that
    // rebuilds fall on step starts, after a reordering.
    const double limit2 = 0.25 * D.p.vskin * D.p.vskin;
    if (ahead2 > limit2) P.need[0] = P.need[1] = 1;
    else if ((sub & SUB_END) && ahead2 > 0.92 * 0.92 * limit2) P.need[1] = 1;
    atomicAdd(&D.b.cnt[particle_cell(D.g, x[0], x[1], x[2])], 1);
    // the stencil of a position outside the domain or not finite is not taken
    // (the step is flagged, the state no longer meaningful)
    if (bad || halted(D)) return;
    Stencil st;
    store_stencil(D, i, x, st);
    if (sub & SUB_AM) {
        R Du[3] = {(R)0, (R)0, (R)0};
        interp_dudt<R>(D, C, st, Du);
        am_store<R>(D, i, Du, d, acc, u, x);
    }
}

// Contact and lubrication force and torque on every particle from its list.
//
// G lanes share a particle and take its entries l, l + G, ... One lane per
// particle is the least work; with few particles it leaves the chip idle and
// every lane with a long chain of dependent loads (see dem_lanes for the choice
// and what it measured). Whatever G is, each sum runs in list order, so all give
// the same bits: with G > 1 the pair terms of a run of kRun G entries go through
// LDS and lane a < 3 of the group adds component a.
//
// Lubrication of every pair within reach comes first; overlapping pairs are
// marked and their contacts evaluated afterwards, run by run. Contacts are few
// (4e-4 per sphere in a dense suspension), and evaluated inline the whole
// wavefront would step through the contact code for them. Lubrication, contacts
// and the walls are summed apart and added at the end. The pass is bound by
// FP64 instruction issue (66 % of the SIMD cycles without the integration, 59 %
// with it) and by the latency of the record gathers. Forces and integration of a
// substep of 3.17 M dense spheres (29.6 list entries each): 1.28 ms as two
// passes with a lane per record, 0.78 ms. Not kept: non-temporal loads of the
// lists or of the state touched once (0 to +7 % time).
// The minimum image is skipped by wavefronts with no particle within reach of a
// periodic boundary.

// the pair (pi, pj): adds the lubrication force to F; whether the spheres overlap
__device__ __forceinline__ bool dem_pair(const Desc &D, const PV &pi, const PV &pj, double gap, bool wrap, double F[3])
{
    double dx[3] = {pj.x[0] - pi.x[0], pj.x[1] - pi.x[1], pj.x[2] - pi.x[2]};
    if (wrap) min_image(D.g, dx);
    const double rsum = 0.5 * (pi.d + pj.d);
    const double reach = rsum + gap;
    const double dist2 = dot3(dx, dx);
    if (dist2 >= reach * reach) return false;
    const double dist = sqrt_pos(dist2);
    const double delta = rsum - dist;
    if (D.p.use_lub) {
        const double inv = rcp64(dist);
        const double n[3] = {dx[0] * inv, dx[1] * inv, dx[2] * inv};
        pair_lubrication(D.p, pi, pj, n, delta, F);
    }
    return delta > 0.0;
}

constexpr int kRun = 2;  // entries per lane and run, several lanes per particle
constexpr int kDemLds = 4096;  // bytes of LDS per wavefront: 64 records' pieces or a run's terms
static_assert(64 * 4 * sizeof(uint4) <= kDemLds, "");

// one lane per particle: the slots of entry t of four groups of 16 lists, and the
// calling lane's piece q of those four records (see below)
__device__ __forceinline__ void load_slots(const int *Sw, int r0, int t, uint32_t top, uint32_t &i0, uint32_t &i1,
                                           uint32_t &i2, uint32_t &i3)
{
    Sw += 64 * t;
    // places beyond a list's end hold anything: kept within the records, not used
    i0 = min((uint32_t)Sw[r0], top);
    i1 = min((uint32_t)Sw[r0 + 16], top);
    i2 = min((uint32_t)Sw[r0 + 32], top);
    i3 = min((uint32_t)Sw[r0 + 48], top);
}
// (Off: the type of a byte offset into the records, 32 bits where they fit 4 GiB)
template <typename R, typename Off>
__device__ __forceinline__ uint4 load_piece(const DemRec<R> *src, uint32_t q16, uint32_t i)
{
    return *reinterpret_cast<const uint4 *>(reinterpret_cast<const char *>(src) + ((Off)i * (Off)sizeof(DemRec<R>) + q16));
}
template <typename R, typename Off>
__device__ __forceinline__ void load_pieces(const DemRec<R> *src, uint32_t q16, uint32_t i0, uint32_t i1, uint32_t i2,
                                            uint32_t i3, uint4 &p0, uint4 &p1, uint4 &p2, uint4 &p3)
{
    p0 = load_piece<R, Off>(src, q16, i0);
    p1 = load_piece<R, Off>(src, q16, i1);
    p2 = load_piece<R, Off>(src, q16, i2);
    p3 = load_piece<R, Off>(src, q16, i3);
}

template <typename R, int G, typename Off>
__device__ __forceinline__ void dem_particle(const Desc &D, const DemRec<R> *src, int64_t i, int l, char *lds,
                                             PV &pi, double Fs[3], double Tq[3])
{
    constexpr int kPieces = rec_pieces<R>();
    const Parts &P = D.pt;
    load_rec<R>(src, i, pi);
    double F[3] = {0.0, 0.0, 0.0}, Fl[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < 3; ++a) Tq[a] = 0.0;
    const double gap = D.p.use_lub ? fmax(D.p.h_c, 0.0) : 0.0;
    const int n = P.nnb[i];
    const int *S = P.nlist + list_base(P, i);
    bool edge = false;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        if (D.g.per[a]) edge |= pi.x[a] < D.p.reach_max || pi.x[a] > D.g.len[a] - D.p.reach_max;
    const bool wrap = __any(edge);
    const double ri = 0.5 * pi.d;
    const auto contact_of = [&](int64_t j, double Fc[3], double tq[3]) {
        PV pj;
        load_rec<R>(src, j, pj);
        double wi[3], wj[3];
        load_spin<R>(src, i, wi);
        load_spin<R>(src, j, wj);
        double dx[3] = {pj.x[0] - pi.x[0], pj.x[1] - pi.x[1], pj.x[2] - pi.x[2]};
        min_image(D.g, dx);
        return pair_contact(D.p, pi, wi, pj, wj, dx, Fc, tq);
    };
    if constexpr (G == 1) {
        // Four lanes load a neighbour's record together, a 16-byte piece each,
        // and every lane takes its own neighbour's pieces from LDS: a lane that
        // loads its record alone touches its cache line once per piece, and
        // those lookups (64 lanes, 3 pieces, 1 per cycle and CU) took as long as
        // the arithmetic. Piece q of lane r's record lies at place q ^ (r/4 % 4),
        // which keeps the 16 lanes of one LDS access on different banks. The
        // pieces of the next entry and the slots of the one after are in flight
        // while an entry is evaluated.
        uint4 *T = (uint4 *)lds;
        const int lane = threadIdx.x & 63, r0 = lane >> 2, q = lane & 3;
        // (the wavefront's lists start at a uniform address)
        const int64_t wave = __builtin_amdgcn_readfirstlane((int)(i >> 6));
        const int *Sw = P.nlist + wave * ((int64_t)P.nbr << 6);
        const uint32_t top = (uint32_t)(P.np - 1);
        int nmax = n;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) nmax = max(nmax, __shfl_xor(nmax, off, 64));
        nmax = __builtin_amdgcn_readfirstlane(nmax);
        uint32_t i0 = 0, i1 = 0, i2 = 0, i3 = 0;
        uint4 p0, p1, p2, p3;
        if (nmax > 0) {
            load_slots(Sw, r0, 0, top, i0, i1, i2, i3);
            load_pieces<R, Off>(src, 16 * q, i0, i1, i2, i3, p0, p1, p2, p3);
            load_slots(Sw, r0, min(1, nmax - 1), top, i0, i1, i2, i3);
        }
        // marks of overlapping pairs, one bit for 2^sh entries (one entry up to 64)
        int sh = 0;
        while ((nmax - 1) >> sh >= 64) ++sh;
        uint64_t touch = 0;
        for (int t = 0; t < nmax; ++t) {
            const int w = r0 * 4 + (q ^ (r0 >> 2));
            T[w] = p0;
            T[w + 64] = p1;
            T[w + 128] = p2;
            T[w + 192] = p3;
            load_pieces<R, Off>(src, 16 * q, i0, i1, i2, i3, p0, p1, p2, p3);
            load_slots(Sw, r0, min(t + 2, nmax - 1), top, i0, i1, i2, i3);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            uint4 own[4];
#pragma unroll
            for (int k = 0; k < kPieces; ++k) own[k] = T[lane * 4 + (k ^ ((lane >> 2) & 3))];
            if (t < n) {
                PV pj;
                unpack_rec<R>(own, pj);
                if (__builtin_expect(dem_pair(D, pi, pj, gap, wrap, Fl), 0)) {
                    asm volatile("");  // a branch, not selects: rarely taken
                    touch |= 1ull << (t >> sh);
                }
            }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) F[a] = Tq[a] = 0.0;
        while (touch) {
            const int t0 = __builtin_ctzll(touch) << sh;
            touch &= touch - 1;
            for (int t = t0; t < min(n, t0 + (1 << sh)); ++t) {
                double Fc[3], tq[3];
                if (!contact_of(S[64 * t], Fc, tq)) continue;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    F[a] += Fc[a];
                    Tq[a] += ri * tq[a];
                }
            }
        }
    } else {
        constexpr int RS = 3 * 64 + 2;  // stride of one round, keeping the components on other banks
        static_assert(sizeof(double) * kRun * RS <= kDemLds, "terms of a run");
        double *T = (double *)lds;
        const int lane = threadIdx.x & 63, g0 = lane & ~(G - 1);
        constexpr int NC = (3 + G - 1) / G;
        // the slots of the next run are in flight while a run is evaluated, those
        // of the first are fetched along with the list's length (entries beyond it
        // are read but not used)
        int next[kRun];
        const auto load_run = [&](int s0) {
#pragma unroll
            for (int r = 0; r < kRun; ++r) next[r] = S[64 * min(s0 + r * G + l, P.nbr - 1)];
        };
        load_run(0);
        double sum[NC] = {};  // components l, l + G < 3 of Fl
        for (int s0 = 0; s0 < n; s0 += kRun * G) {
            int js[kRun];
#pragma unroll
            for (int r = 0; r < kRun; ++r) js[r] = s0 + r * G + l < n ? next[r] : (int)i;
            load_run(s0 + kRun * G);
            PV pj[kRun];
#pragma unroll
            for (int r = 0; r < kRun; ++r) load_rec<R>(src, js[r], pj[r]);
            bool touch[kRun];
#pragma unroll
            for (int r = 0; r < kRun; ++r) {
                double f[3] = {0.0, 0.0, 0.0};
                touch[r] = s0 + r * G + l < n && dem_pair(D, pi, pj[r], gap, wrap, f);
#pragma unroll
                for (int a = 0; a < 3; ++a) T[r * RS + a * 64 + lane] = f[a];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int m = min(n - s0, kRun * G);
#pragma unroll
            for (int k = 0; k < NC; ++k)
                if (l + k * G < 3)
#pragma unroll 4
                    for (int e = 0; e < m; ++e) sum[k] += T[(e / G) * RS + (l + k * G) * 64 + g0 + (e & (G - 1))];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int r = 0; r < kRun; ++r) {
                uint64_t b = (__ballot(touch[r]) >> g0) & ((1ull << G) - 1);
                while (b) {
                    const int t = __builtin_ctzll(b);
                    b &= b - 1;
                    double Fc[3] = {0.0, 0.0, 0.0}, tq[3] = {0.0, 0.0, 0.0};
                    if (l == t) contact_of(js[r], Fc, tq);
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        F[a] += __shfl(Fc[a], g0 + t, 64);
                        Tq[a] += ri * __shfl(tq[a], g0 + t, 64);
                    }
                }
            }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) Fl[a] = __shfl(sum[a / G], g0 + a % G, 64);
    }
    if (!(D.g.per[0] && D.g.per[1] && D.g.per[2])) {
        double wi[3];
        load_spin<R>(src, i, wi);
        wall_interaction(D.p, D.g, pi, wi, F, Tq);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) Fs[a] = F[a] + Fl[a];
}

// FUSE: the substep's integration follows in the same pass. Substeps then
// alternate between the two record buffers (odd: from pk2 to pk), reading the
// records of the substep's start and writing the integrated ones to the other
// buffer, so that no thread sees another's update.
// (4 waves per SIMD in the FP32 form with one lane per particle, which needs 129
// registers otherwise)
template <typename R, int G, bool FUSE, typename Off>
__global__ __launch_bounds__(kBlock, sizeof(R) == 4 && G == 1 ? 4 : 1) void k_dem_force(Desc D, Cells<R> C, int sub, int odd)
{
    __shared__ __align__(16) char lds[kBlock / 64][kDemLds];
    char *T = lds[threadIdx.x >> 6];
    const Parts &P = D.pt;
    DemRec<R> *pk = (DemRec<R> *)P.pk, *pk2 = (DemRec<R> *)P.pk2;
    const int64_t v = gidx();
    int64_t i = v / G;
    const int l = (int)(v % G);
    // a wavefront with particles keeps all its lanes (they load for each other);
    // lanes beyond the last particle repeat it and store nothing
    const bool own = i < P.np;
    if ((v & ~(int64_t)63) / G >= P.np) return;
    if (!own) i = P.np - 1;
    double F[3], Tq[3];
    PV pi;
    dem_particle<R, G, Off>(D, FUSE && odd ? pk2 : pk, i, l, T, pi, F, Tq);
    if (!own || (G > 1 && l != 0)) return;
    if constexpr (FUSE) {
        integrate_particle<R, true>(D, C, i, sub, F, Tq, pi, odd ? pk2 : pk, odd ? pk : pk2);
    } else {
        const int64_t cap = P.cap;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            P.Fdem[a * cap + i] = F[a];
            P.Tdem[a * cap + i] = Tq[a];
        }
    }
}

// All substeps of a subcycle in one launch of one workgroup, for particles that
// fit into one (np <= kBlock, one lane each, short lists): a substep of so few
// takes less time than its launch. The particles meet at a barrier after every substep; the
// records alternate as above. One sphere at a wall, 50 substeps: 97 us,
// 280 us as 50 launches (and twice that as 100 with the integration apart).
template <typename R>
__global__ __launch_bounds__(kBlock) void k_dem_subcycle(Desc D, Cells<R> C, int sub_last)
{
    __shared__ __align__(16) char lds[kBlock / 64][kDemLds];
    char *T = lds[threadIdx.x >> 6];
    const Parts &P = D.pt;
    const bool own = threadIdx.x < P.np;
    const int64_t i = own ? threadIdx.x : P.np - 1;
    const bool wave = (int64_t)(threadIdx.x & ~63u) < P.np;  // wavefronts without particles only meet the others
    DemRec<R> *a = (DemRec<R> *)P.pk, *b = (DemRec<R> *)P.pk2;
    for (int t = 0; t < D.p.n_dem; ++t) {
        if (wave) {
            double F[3], Tq[3];
            PV pi;
            dem_particle<R, 1, uint32_t>(D, a, i, 0, T, pi, F, Tq);
            if (own) integrate_particle<R, true>(D, C, i, t == D.p.n_dem - 1 ? sub_last : 0, F, Tq, pi, a, b);
        }
        __syncthreads();
        DemRec<R> *c = a;
        a = b;
        b = c;
    }
}

// Blocked slot order (see Order): block row r
// = (block, lz, ly) with blocks row-major over the domain and rows y-fastest
// inside a block; its cells are x0 <= x < x1 of row (y, z). Rows of the
// padded last blocks that fall outside the domain are empty.
__device__ __forceinline__ bool order_row(const Desc &D, int64_t r, int &x0, int &x1, int &y, int &z)
{
    const Order &O = D.o;
    const int64_t per = (int64_t)O.ob[1] * O.ob[2];
    const int64_t blk = r / per, lr = r - blk * per;
    const int ly = (int)(lr % O.ob[1]), lz = (int)(lr / O.ob[1]);
    const int bxi = (int)(blk % O.nb[0]);
    const int byi = (int)((blk / O.nb[0]) % O.nb[1]);
    const int bzi = (int)(blk / ((int64_t)O.nb[0] * O.nb[1]));
    y = byi * O.ob[1] + ly;
    z = bzi * O.ob[2] + lz;
    x0 = bxi * O.ob[0];
    x1 = min(x0 + O.ob[0], D.g.n[0]);
    return y < D.g.n[1] && z < D.g.n[2];
}

__device__ __forceinline__ int order_row_count(const Desc &D, int x0, int x1, int y, int z, int &s0)
{
    s0 = D.b.start[cidx(D.g, x0, y, z)];
    return D.b.start[cidx(D.g, x1 - 1, y, z) + 1] - s0;
}

// particles per block row, scanned within blocks of kScanPerBlock rows
__global__ __launch_bounds__(kBlock) void k_order_scan(Desc D)
{
    __shared__ int wsum[kBlock / 64];
    if (!reorder_due(D)) return;
    const int64_t n = D.o.nrows;
    const int64_t base = (int64_t)blockIdx.x * kScanPerBlock + (int64_t)threadIdx.x * kScanItems;
    int v[kScanItems];
    int tot = 0;
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) {
        int x0, x1, y, z, s0;
        v[t] = (base + t < n && order_row(D, base + t, x0, x1, y, z)) ? order_row_count(D, x0, x1, y, z, s0) : 0;
        tot += v[t];
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = tot;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int run = incl - tot, btot = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        const int ws = wsum[w];
        if (w < wv) run += ws;
        btot += ws;
    }
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) {
        if (base + t < n) D.o.rowoff[base + t] = run;
        run += v[t];
    }
    if (threadIdx.x == kBlock - 1) D.o.rowsum[blockIdx.x] = btot;
}

// porder[p] = place in the blocked order of the p-th entry of the sorted slot list
__global__ __launch_bounds__(kBlock) void k_order_fill(Desc D)
{
    if (!reorder_due(D)) return;
    const int64_t r = gidx();
    if (r >= D.o.nrows) return;
    int x0, x1, y, z, s0;
    if (!order_row(D, r, x0, x1, y, z)) return;
    const int cnt = order_row_count(D, x0, x1, y, z, s0);
    const int off = D.o.rowoff[r] + D.o.rowsum[r / kScanPerBlock];
    for (int k = 0; k < cnt; ++k) D.o.porder[s0 + k] = off + k;
}

// semi-implicit Euler with the fluid forces frozen (Sec. 3.3); periodic wrap;
// the last substep of a subcycle also prepares the next one (integrate_particle)
template <typename R> __global__ __launch_bounds__(kBlock) void k_integrate(Desc D, Cells<R> C, int sub)
{
    const int64_t i = gidx();
    const Parts &P = D.pt;
    if (i >= P.np) return;
    const int64_t cap = P.cap;
    const double F[3] = {P.Fdem[i], P.Fdem[cap + i], P.Fdem[2 * cap + i]};
    const double Tq[3] = {P.Tdem[i], P.Tdem[cap + i], P.Tdem[2 * cap + i]};
    integrate_particle<R, false>(D, C, i, sub, F, Tq, PV(), (const DemRec<R> *)nullptr, (DemRec<R> *)P.pk);
}

__global__ __launch_bounds__(kBlock) void k_bin_count(Desc D)
{
    const int64_t i = gidx();
    const Parts &P = D.pt;
    if (i >= P.np || halted(D)) return;
    const int64_t cap = P.cap;
    atomicAdd(&D.b.cnt[particle_cell(D.g, P.x[i], P.x[cap + i], P.x[2 * cap + i])], 1);
}

// exclusive scan of cnt into loc and bsum; resets cnt
__global__ __launch_bounds__(kBlock) void k_scan_block(Desc D, int both)
{
    __shared__ int wsum[kBlock / 64];
    const int64_t nc = D.g.nc;
    const int64_t base = (int64_t)blockIdx.x * kScanPerBlock + (int64_t)threadIdx.x * kScanItems;
    static_assert(kScanItems == 8, "two 16-byte vectors per thread");
    // a thread's 8 counts are 32-byte aligned: two vector loads, scalar
    // loads only for the last, ragged chunk
    const bool full = base + kScanItems <= nc;
    int v[kScanItems];
    if (full) {
        const int4 a = *reinterpret_cast<const int4 *>(D.b.cnt + base);
        const int4 b = *reinterpret_cast<const int4 *>(D.b.cnt + base + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
        for (int t = 0; t < kScanItems; ++t) v[t] = base + t < nc ? D.b.cnt[base + t] : 0;
    }
    int tot = 0;
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) tot += v[t];
    // wavefront-shuffle scan, then the wavefront totals (one barrier)
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = tot;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int run = incl - tot, btot = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        const int ws = wsum[w];
        if (w < wv) run += ws;
        btot += ws;
    }
    int o[kScanItems];
#pragma unroll
    for (int t = 0; t < kScanItems; ++t) {
        o[t] = run;
        run += v[t];
    }
    if (full) {
        *reinterpret_cast<int4 *>(D.b.loc + base) = make_int4(o[0], o[1], o[2], o[3]);
        *reinterpret_cast<int4 *>(D.b.loc + base + 4) = make_int4(o[4], o[5], o[6], o[7]);
        *reinterpret_cast<int4 *>(D.b.cnt + base) = make_int4(0, 0, 0, 0);
        *reinterpret_cast<int4 *>(D.b.cnt + base + 4) = make_int4(0, 0, 0, 0);
    } else {
#pragma unroll
        for (int t = 0; t < kScanItems; ++t)
            if (base + t < nc) {
                D.b.loc[base + t] = o[t];
                D.b.cnt[base + t] = 0;
            }
    }
    if (!both) {
        if (threadIdx.x == kBlock - 1) D.b.bsum[blockIdx.x] = btot;
        return;
    }
    // The last workgroup to get here scans the block sums (both levels in one
    // launch). Sums and count go through atomics at device scope, which all XCDs
    // see at once; the sum's has returned before the count's is issued. That the
    // two are seen in this order is the hardware's (an atomic that has returned
    // its old value is done where every XCD looks), not the memory model's, which
    // asks for release order; that writes the XCD's whole L2 back per workgroup:
    // 88 us on 128^3 cells.
    __shared__ int last;
    if (threadIdx.x == 0) {
        int old = __hip_atomic_exchange(D.b.bsum + blockIdx.x, btot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(old) : : "memory");
        last = __hip_atomic_fetch_add(D.b.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    __shared__ int tsum[kBlock / 64];
    const int nb = (int)gridDim.x, per = (nb + kBlock - 1) / kBlock, b0 = threadIdx.x * per;
    int sum = 0;
    for (int t = b0; t < min(b0 + per, nb); ++t)
        sum += __hip_atomic_load(D.b.bsum + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int pre = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(pre, off, 64);
        if (lane >= off) pre += y;
    }
    if (lane == 63) tsum[wv] = pre;
    __syncthreads();
    pre -= sum;
    for (int w = 0; w < wv; ++w) pre += tsum[w];
    for (int t = b0; t < min(b0 + per, nb); ++t) {
        const int v = __hip_atomic_load(D.b.bsum + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        D.b.bsum[t] = pre;
        pre += v;
    }
    if (threadIdx.x == kBlock - 1) {
        D.b.start[nc] = pre;
        *D.b.done = 0;
    }
}

// exclusive scan of the block sums, one block of 1024 threads
// (gate: skipped while *gate is 0)
__global__ __launch_bounds__(1024) void k_scan_top(int *bsum, int nb, int *total, const int *gate)
{
    __shared__ int sh[1024];
    if (gate && *gate == 0) return;
    const int per = (nb + 1023) / 1024;
    const int b0 = threadIdx.x * per;
    int tot = 0;
    for (int t = 0; t < per; ++t)
        if (b0 + t < nb) tot += bsum[b0 + t];
    sh[threadIdx.x] = tot;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int add = threadIdx.x >= (unsigned)off ? sh[threadIdx.x - off] : 0;
        __syncthreads();
        sh[threadIdx.x] += add;
        __syncthreads();
    }
    int run = sh[threadIdx.x] - tot;
    for (int t = 0; t < per; ++t)
        if (b0 + t < nb) {
            const int v = bsum[b0 + t];
            bsum[b0 + t] = run;
            run += v;
        }
    if (threadIdx.x == 1023) *total = sh[1023];
}

// start of bin c in the slot list from the block-local prefix and the block offset
__device__ __forceinline__ int bin_start(const Bins &B, int64_t c)
{
    return B.loc[c] + B.bsum[c / kScanPerBlock];
}

__global__ __launch_bounds__(kBlock) void k_place(Desc D)
{
    const int64_t i = gidx();
    const Parts &P = D.pt;
    if (i >= P.np || halted(D)) return;
    const int64_t cap = P.cap;
    const int64_t c = particle_cell(D.g, P.x[i], P.x[cap + i], P.x[2 * cap + i]);
    const int pos = bin_start(D.b, c) + atomicAdd(&D.b.cnt[c], 1);
    D.b.list[pos] = (int)i;
}

// order each bin by insertion index (so that every sum over a bin runs in a
// history-independent order), write the final bin offsets, reset the counts
__global__ __launch_bounds__(kBlock) void k_cellsort(Desc D)
{
    const int64_t nc = D.g.nc;
    const int64_t c = gidx();
    if (c >= nc || halted(D)) return;
    D.b.cnt[c] = 0;
    const int p0 = bin_start(D.b, c), p1 = c + 1 < nc ? bin_start(D.b, c + 1) : D.b.start[nc];
    D.b.start[c] = p0;
    const int *id = D.pt.id;
    int *L = D.b.list;
    for (int a = p0 + 1; a < p1; ++a) {
        const int v = L[a];
        const int key = id[v];
        int b = a - 1;
        while (b >= p0 && id[L[b]] > key) {
            L[b + 1] = L[b];
            --b;
        }
        L[b + 1] = v;
    }
}

// Reordering of the slots, at a step's start when the lists are due (need[1]):
// into the order of the sorted list (cells row by row), or of the blocked order.
// Particles move far less than a cell between two rebuilds, so the slots stay
// close to cell order meanwhile, and every pass reads neighbours almost in
// order; moving the state every subcycle instead cost 338 us of the 14.7 ms
// subcycle on 3.17 M dense spheres (and a 410 us lookup of the neighbours' new
// slots), 53 of 340 us on 391 k dilute ones. k_reorder writes the new order to
// the permutation targets, k_reorder_back copies it home (pointers are baked
// into captured graphs) and requests the lists.
__global__ __launch_bounds__(kBlock) void k_reorder(Desc D)
{
    if (!reorder_due(D)) return;
    const Parts &P = D.pt;
    const int64_t p = gidx();
    if (p >= P.np) return;
    const int64_t cap = P.cap;
    const int src = D.b.list[p];
    const int64_t s = D.t.dem_order ? (int64_t)D.o.porder[p] : p;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        P.x2[a * cap + s] = P.x[a * cap + src];
        P.u2[a * cap + s] = P.u[a * cap + src];
        P.w2[a * cap + s] = P.w[a * cap + src];
        P.a2[a * cap + s] = P.a[a * cap + src];
    }
    P.d2[s] = P.d[src];
    P.rho2[s] = P.rho[src];
    P.id2[s] = P.id[src];
    P.nnb2[s] = P.nnb[src];
    P.pos2[s] = (int)p;
}

// Where the DEM pass dominates, k_reorder_back also orders each group of kBlock
// slots by the length of the particle's last list, longest first: a wavefront of
// the DEM pass runs as long as its longest list, and 64 neighbouring dense
// spheres hold 29.6 entries in the mean and 41 at most. A coupled step of 100
// substeps on 396 k / 3.17 M such spheres: 12.8 / 101 ms unsorted, 11.7 / 94 ms
// sorted in groups of 256, 12.8 / 100 ms in groups of 1024 (whose wavefronts
// share fewer neighbours).
__host__ __device__ __forceinline__ bool sort_lengths(const Desc &D) { return D.p.n_dem >= 3; }
__global__ __launch_bounds__(kBlock) void k_reorder_back(Desc D)
{
    __shared__ int len[kBlock];
    if (!reorder_due(D)) return;
    const Parts &P = D.pt;
    const int64_t base = (int64_t)blockIdx.x * kBlock, s = base + threadIdx.x;
    if (s == 0) P.need[0] = 1;
    int64_t f = s;
    if (sort_lengths(D)) {
        const int n = s < P.np ? P.nnb2[s] : -1;
        len[threadIdx.x] = n;
        __syncthreads();
        int rank = 0;
        for (int t = 0; t < kBlock; ++t) rank += len[t] > n || (len[t] == n && t < (int)threadIdx.x);
        f = base + rank;
    }
    if (s >= P.np) return;
    const int64_t cap = P.cap;
    double x[3], u[3], w[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        x[a] = P.x2[a * cap + s];
        u[a] = P.u2[a * cap + s];
        w[a] = P.w2[a * cap + s];
        P.x[a * cap + f] = x[a];
        P.u[a * cap + f] = u[a];
        P.w[a * cap + f] = w[a];
        P.a[a * cap + f] = P.a2[a * cap + s];
    }
    const double d = P.d2[s], rho = P.rho2[s];
    P.d[f] = d;
    P.rho[f] = rho;
    P.id[f] = P.id2[s];
    D.b.list[P.pos2[s]] = (int)f;
    Stencil st;
    store_stencil(D, f, x, st);
    const double m = rho * sphere_volume(d);
    if (P.swf) store_rec<float>((DemRec<float> *)P.pk, f, x, u, w, d, (float)m);
    else store_rec<double>((DemRec<double> *)P.pk, f, x, u, w, d, m);
}

// ---------------------------------------------------------------------------
// a10: fused GNS-LBM collide + stream (Eq. LBM_Equation, Eq. LBM_EQ,
// Eq. Forcing, Eq. MacVel), push form: reads the post-stream PDFs of its own
// cell, writes the post-collision values to x + c_q. Links leaving through a
// wall reflect in place into the opposite direction (half-way bounce-back).
// ---------------------------------------------------------------------------
// GNS-BGK collision with Guo forcing of one cell (the post-collision values
// of all 19 directions, before streaming)
// Per-cell relaxation time tau_e = tau_* + tau_t (Eq. tau_e; Alg. 1, before
// the GNS-LBM step), in the storage precision R:
//  - Eilers (Eq. visc_eilers with the denominator 1 - eps_p/eps_cp of Eilers'
//    form; [mu] = 2.5, eps_cp = 0.64) through Eq. visc_tau_*:
//    tau_* = 1/2 + (tau - 1/2) (1 + 1.25 eps_p/(1 - eps_p/0.64))^2;
//  - Smagorinsky (Eq. visc_turb, C_s = 0.1, dx = 1): tau_t is the positive
//    root of tau_t^2 + tau_* tau_t = C_s^2 Qbar/(2 rho c_s^4), Qbar =
//    sqrt(2 sum Q_ab Q_ab), Q_ab = sum_q c_qa c_qb (f_q - f_q^eq).
template <typename R>
__device__ __forceinline__ R relax_time(const Desc &D, R ep, R rho, const R f[19], const R feq[19])
{
    const R one = (R)1;
    R tau = (R)D.p.tau;
    if (D.p.use_eilers) {
        const R b = one + (R)1.25 * ep / (one - ep / (R)0.64);
        tau = (R)0.5 + ((R)D.p.tau - (R)0.5) * b * b;
    }
    if (D.p.use_les) {
        R qxx = 0, qyy = 0, qzz = 0, qxy = 0, qxz = 0, qyz = 0;
#pragma unroll
        for (int q = 1; q < 19; ++q) {
            const R n = f[q] - feq[q];
            if (CX(q) != 0) qxx += n;
            if (CY(q) != 0) qyy += n;
            if (CZ(q) != 0) qzz += n;
            if (CX(q) * CY(q) > 0) qxy += n; else if (CX(q) * CY(q) < 0) qxy -= n;
            if (CX(q) * CZ(q) > 0) qxz += n; else if (CX(q) * CZ(q) < 0) qxz -= n;
            if (CY(q) * CZ(q) > 0) qyz += n; else if (CY(q) * CZ(q) < 0) qyz -= n;
        }
        const R qq = qxx * qxx + qyy * qyy + qzz * qzz + (R)2 * (qxy * qxy + qxz * qxz + qyz * qyz);
        const R qbar = sqrt((R)2 * qq);
        // C_s^2 Qbar / (2 rho c_s^4) with C_s^2 = 0.01, 1/c_s^4 = 9
        const R rhs = (R)0.045 * qbar / rho;
        tau += (R)0.5 * (sqrt(tau * tau + (R)4 * rhs) - tau);
    }
    return tau;
}

template <typename R, bool VISC>
__device__ __forceinline__ void collide_cell(const Desc &D, const Cells<R> &C, int64_t c, R post[19], int &bad)
{
    const int64_t nc = D.g.nc;
    R f[19];
#pragma unroll
    for (int q = 0; q < 19; ++q) f[q] = C.df_src[q * nc + c];
    R r = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        r += f[q];
        if (CX(q) > 0) jx += f[q]; else if (CX(q) < 0) jx -= f[q];
        if (CY(q) > 0) jy += f[q]; else if (CY(q) < 0) jy -= f[q];
        if (CZ(q) > 0) jz += f[q]; else if (CZ(q) < 0) jz -= f[q];
    }
    const R one = (R)1;
    const R rho = one + r;
    const R fx = C.facc[c], fy = C.facc[nc + c], fz = C.facc[2 * nc + c];
    const R half = (R)0.5;
    const R ux = (jx + half * fx) / rho, uy = (jy + half * fy) / rho, uz = (jz + half * fz) / rho;
    const R eps = one - C.epsp[c];
    const R ieps = one / eps;
    const R uu = ux * ux + uy * uy + uz * uz;
    // non-finite PDFs make rho or u non-finite; |u| > 0.1 leaves the low-Mach
    // range in which the equilibrium expansion holds
    if (!isfinite(rho) || !isfinite(uu)) bad = FLAG_FLUID_NONFINITE;
    else if (uu > (R)0.01) bad = FLAG_MACH;
    if (VISC) {
        R feq[19];
#pragma unroll
        for (int q = 0; q < 19; ++q) {
            const R cu = (R)CX(q) * ux + (R)CY(q) * uy + (R)CZ(q) * uz;
            const R w = (R)WQ(q);
            feq[q] = w * r + w * rho * ((R)3 * cu + (R)4.5 * cu * cu * ieps - (R)1.5 * uu * ieps);
        }
        const R tau = relax_time<R>(D, C.epsp[c], rho, f, feq);
        const R om = one / tau;
        const R pre = one - half / tau;
#pragma unroll
        for (int q = 0; q < 19; ++q) {
            const R cu = (R)CX(q) * ux + (R)CY(q) * uy + (R)CZ(q) * uz;
            const R w = (R)WQ(q);
            const R gx = (R)3 * (R)CX(q) - (R)3 * ux * ieps + (R)9 * cu * (R)CX(q) * ieps;
            const R gy = (R)3 * (R)CY(q) - (R)3 * uy * ieps + (R)9 * cu * (R)CY(q) * ieps;
            const R gz = (R)3 * (R)CZ(q) - (R)3 * uz * ieps + (R)9 * cu * (R)CZ(q) * ieps;
            const R F = w * pre * (gx * fx + gy * fy + gz * fz);
            post[q] = f[q] + (feq[q] - f[q]) * om + F;
        }
        return;
    }
    const R om = (R)D.p.omega;
    const R pre = (R)(1.0 - 0.5 / D.p.tau);
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        const R cu = (R)CX(q) * ux + (R)CY(q) * uy + (R)CZ(q) * uz;
        const R w = (R)WQ(q);
        const R feq = w * r + w * rho * ((R)3 * cu + (R)4.5 * cu * cu * ieps - (R)1.5 * uu * ieps);
        const R gx = (R)3 * (R)CX(q) - (R)3 * ux * ieps + (R)9 * cu * (R)CX(q) * ieps;
        const R gy = (R)3 * (R)CY(q) - (R)3 * uy * ieps + (R)9 * cu * (R)CY(q) * ieps;
        const R gz = (R)3 * (R)CZ(q) - (R)3 * uz * ieps + (R)9 * cu * (R)CZ(q) * ieps;
        const R F = w * pre * (gx * fx + gy * fy + gz * fz);
        post[q] = f[q] + (feq - f[q]) * om + F;
    }
}

// push streaming: direction q of cell (i, j, k) goes to (i, j, k) + c_q,
// wrapped on periodic axes; where it would leave through a wall it returns
// into the opposite direction of the same cell (half-way bounce-back)
template <typename R, bool VISC>
__global__ __launch_bounds__(kBlock) void k_stream_collide(Desc D, Cells<R> C)
{
    const int64_t nc = D.g.nc;
    const int64_t c = gidx();
    if (c == 0) *D.stepc += 1;
    if (c >= nc) return;
    int i, j, k;
    cell_coords(D.g, c, i, j, k);
    R post[19];
    int bad = 0;
    collide_cell<R, VISC>(D, C, c, post, bad);
    if (bad) atomicOr(D.flags, bad);
    const bool wall_x = !D.g.per[0], wall_y = !D.g.per[1], wall_z = !D.g.per[2];
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        int t0 = i + CX(q), t1 = j + CY(q), t2 = k + CZ(q);
        bool wall = false;
        if (CX(q) != 0 && (t0 < 0 || t0 >= D.g.n[0])) {
            if (wall_x) wall = true; else t0 = t0 < 0 ? t0 + D.g.n[0] : t0 - D.g.n[0];
        }
        if (CY(q) != 0 && (t1 < 0 || t1 >= D.g.n[1])) {
            if (wall_y) wall = true; else t1 = t1 < 0 ? t1 + D.g.n[1] : t1 - D.g.n[1];
        }
        if (CZ(q) != 0 && (t2 < 0 || t2 >= D.g.n[2])) {
            if (wall_z) wall = true; else t2 = t2 < 0 ? t2 + D.g.n[2] : t2 - D.g.n[2];
        }
        if (wall) C.df_dst[OPP(q) * nc + c] = post[q];
        else C.df_dst[q * nc + cidx(D.g, t0, t1, t2)] = post[q];
    }
}

// ---------------------------------------------------------------------------
// reductions for the diagnostics (two passes, fixed order: deterministic)
// per-block partials: [0] sum drho, [1..3] sum j, [4] sum eps, [5] min eps,
// [6] sum u_f,z, [7] max |u_bar|, [8..10] sum m u, [11] sum u_z
// ---------------------------------------------------------------------------
constexpr int kDiag = kDiagValues;

template <typename R>
__global__ __launch_bounds__(kBlock) void k_diag(Desc D, Cells<R> C, const R *df, double *part)
{
    __shared__ double sh[kDiag][kBlock];
    const int64_t nc = D.g.nc, np = D.pt.np, cap = D.pt.cap;
    double acc[kDiag] = {0, 0, 0, 0, 0, 1e300, 0, 0, 0, 0, 0, 0};
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t c = gidx(); c < nc; c += stride) {
        double r = 0, jx = 0, jy = 0, jz = 0;
#pragma unroll
        for (int q = 0; q < 19; ++q) {
            const double f = (double)df[q * nc + c];
            r += f;
            jx += CX(q) * f;
            jy += CY(q) * f;
            jz += CZ(q) * f;
        }
        const double e = 1.0 - (double)C.epsp[c];
        const double rho = 1.0 + r;
        const double ub0 = (jx + 0.5 * e * D.p.fb[0]) / rho;
        const double ub1 = (jy + 0.5 * e * D.p.fb[1]) / rho;
        const double ub2 = (jz + 0.5 * e * D.p.fb[2]) / rho;
        acc[0] += r;
        acc[1] += jx;
        acc[2] += jy;
        acc[3] += jz;
        acc[4] += e;
        acc[5] = fmin(acc[5], e);
        acc[6] += ub2 / e;
        acc[7] = fmax(acc[7], sqrt(ub0 * ub0 + ub1 * ub1 + ub2 * ub2));
    }
    // in the order of the sorted list, by cell and insertion index: the sums then do
    // not depend on the slots, which differ with the last rebuild and the tuning
    for (int64_t q = gidx(); q < np; q += stride) {
        const int64_t i = D.b.list[q];
        const double m = D.pt.rho[i] * sphere_volume(D.pt.d[i]);
        acc[8] += m * D.pt.u[i];
        acc[9] += m * D.pt.u[cap + i];
        acc[10] += m * D.pt.u[2 * cap + i];
        acc[11] += D.pt.u[2 * cap + i];
    }
#pragma unroll
    for (int t = 0; t < kDiag; ++t) sh[t][threadIdx.x] = acc[t];
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if (threadIdx.x < (unsigned)off) {
#pragma unroll
            for (int t = 0; t < kDiag; ++t) {
                const double a = sh[t][threadIdx.x], b = sh[t][threadIdx.x + off];
                sh[t][threadIdx.x] = t == 5 ? fmin(a, b) : (t == 7 ? fmax(a, b) : a + b);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < kDiag) part[(int64_t)blockIdx.x * kDiag + threadIdx.x] = sh[threadIdx.x][0];
}

__global__ void k_diag_final(const double *part, int nblk, double *out)
{
    const int t = threadIdx.x;
    if (t >= kDiag) return;
    double a = t == 5 ? 1e300 : 0.0;
    for (int b = 0; b < nblk; ++b) {
        const double v = part[(int64_t)b * kDiag + t];
        a = t == 5 ? fmin(a, v) : (t == 7 ? fmax(a, v) : a + v);
    }
    out[t] = a;
}

template <typename R>
__global__ void k_zero(R *p, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = (R)0;
}

template <typename A, typename B>
__global__ void k_convert(const A *src, B *dst, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = (B)src[i];
}

// stored solid fraction -> fluid volume fraction 1 - eps_p, FP64
template <typename A> __global__ void k_fluid_fraction(const A *src, double *dst, int64_t nc)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += stride)
        dst[c] = 1.0 - (double)src[c];
}

// [nc][4] -> [3][nc] doubles
template <typename A> __global__ void k_vec4_to_soa(const A *src, double *dst, int64_t nc)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += stride)
#pragma unroll
        for (int b = 0; b < 3; ++b) dst[b * nc + c] = (double)src[4 * c + b];
}

// Particle state for the host: slot order [3][cap] -> insertion order [np][3]
// (one write of 24 contiguous bytes per particle and vector) and [np]
// scalars, whichever are asked for. Written to the permutation targets, which
// hold nothing between two reorderings, so reading allocates nothing.
__global__ __launch_bounds__(kBlock) void k_pack_particles(Desc D, int what)
{
    const Parts &P = D.pt;
    const int64_t s = gidx();
    if (s >= P.np) return;
    const int64_t id = P.id[s];
    const double *vec[4] = {P.x, P.u, P.w, P.a};
    double *out[4] = {P.x2, P.u2, P.w2, P.a2};
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (what & (1 << t))
#pragma unroll
            for (int a = 0; a < 3; ++a) out[t][3 * id + a] = vec[t][a * P.cap + s];
    if (what & PACK_D) P.d2[id] = P.d[s];
    if (what & PACK_RHO) P.rho2[id] = P.rho[s];
}
// force by insertion index [3][cap] -> [np][3]
__global__ __launch_bounds__(kBlock) void k_pack_vec(const double *src, int64_t cap, int64_t n, double *out)
{
    const int64_t i = gidx();
    if (i >= n) return;
#pragma unroll
    for (int a = 0; a < 3; ++a) out[3 * i + a] = src[a * cap + i];
}

// component w of [nc][4]
template <typename A> __global__ void k_vec4_w(const A *src, double *dst, int64_t nc)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < nc; c += stride) dst[c] = (double)src[4 * c + 3];
}

__global__ void k_set_step(long long *s, long long v) { *s = v; }
__global__ void k_set_int(int *p, int v) { *p = v; }

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static inline unsigned nblocks(int64_t n, int64_t per = kBlock)
{
    return (unsigned)((n + per - 1) / per);
}
static inline unsigned grid_stride_blocks(int64_t n)
{
    int64_t b = (n + kBlock - 1) / kBlock;
    if (b > 8192) b = 8192;
    if (b < 1) b = 1;
    return (unsigned)b;
}

// Residency of the streaming cell passes: unused dynamic LDS caps the
// workgroups per CU (160 KB of LDS per CU); -1 is the measured default (4
// workgroups of 256 threads, 4 waves per SIMD, for the FP32 stream-collide)
static inline unsigned cell_lds_bytes(int cell_waves, unsigned dflt)
{
    if (cell_waves < 0) return dflt;
    if (cell_waves == 0) return 0u;
    return (160u * 1024u / (unsigned)cell_waves) & ~255u;
}
template <typename R> void launch_moments(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    hipLaunchKernelGGL(k_moments<R>, dim3(nblocks(D.g.nc)), dim3(kBlock), cell_lds_bytes(D.t.cell_waves, 0u), s, D,
                       C);
}
template <typename R> void launch_cellfields(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    hipLaunchKernelGGL(k_cellfields<R>, dim3(nblocks(D.g.nc)), dim3(kBlock), 0, s, D, C);
}
template <typename R> void launch_curl(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    hipLaunchKernelGGL(k_curl<R>, dim3(nblocks(D.g.nc)), dim3(kBlock), 0, s, D, C);
}
// added-mass pass: one thread per particle (its 3-component stencil reads
// are cheap enough that LDS staging of the halo does not pay). With lift it
// reads 9 components per stencil cell and uses LDS tiles (16x4x8 cells in
// FP32, 16x4x4 in FP64 to stay within 64 KiB of LDS), or one thread per
// particle under gather variant 3.
template <typename R> void launch_part_am(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    if (D.pt.np == 0) return;
    if (!D.p.use_lift) {
        hipLaunchKernelGGL((k_part_am<R, false>), dim3(nblocks(D.pt.np)), dim3(kBlock), 0, s, D, C);
        return;
    }
    if (D.t.gather == 3) {
        hipLaunchKernelGGL((k_part_am<R, true>), dim3(nblocks(D.pt.np)), dim3(kBlock), 0, s, D, C);
        return;
    }
    constexpr int TZ = sizeof(R) == 4 ? 8 : 4;
    dim3 grid((D.g.n[0] + 15) / 16, (D.g.n[1] + 3) / 4, (D.g.n[2] + TZ - 1) / TZ);
    hipLaunchKernelGGL((k_part_tile<R, PASS_AML, 16, 4, TZ, 256>), grid, dim3(256), 0, s, D, C, 0);
}
// gather variants (chosen per domain by the autotuner, else by particle
// density): 0 tiles of 16x4x8 cells (two per thread, up to 256 staged
// particles); 1 16x4x4 (384); 2 8x4x4 (640); 3 one thread per cell from
// global memory; 4 16x4x16 (four per thread, 512). All give bit-identical
// results: every cell sums its bins in the same order and precision.
// Periodic axes thinner than 3 cells use the per-cell gather.
template <typename R, int MODE> void launch_gather(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    const bool thin = (D.g.per[0] && D.g.n[0] < 3) || (D.g.per[1] && D.g.n[1] < 3) || (D.g.per[2] && D.g.n[2] < 3);
    if (thin || D.t.gather == 3) {
        hipLaunchKernelGGL((k_gather_cells<R, MODE>), dim3(nblocks(D.g.nc)), dim3(kBlock), 0, s, D, C);
        return;
    }
    int v = D.t.gather;
    if (v < 0 || v >= kGatherVariants) {
        const double density = D.g.nc > 0 ? (double)D.pt.np / (double)D.g.nc : 0.0;
        v = density < 0.3 ? 0 : (density < 1.0 ? 1 : 2);
    }
    if (v == 0) {
        dim3 grid((D.g.n[0] + 15) / 16, (D.g.n[1] + 3) / 4, (D.g.n[2] + 7) / 8);
        hipLaunchKernelGGL((k_gather_tile<R, MODE, 16, 4, 4, 2, 256>), grid, dim3(256), 0, s, D, C);
    } else if (v == 1) {
        dim3 grid((D.g.n[0] + 15) / 16, (D.g.n[1] + 3) / 4, (D.g.n[2] + 3) / 4);
        hipLaunchKernelGGL((k_gather_tile<R, MODE, 16, 4, 4, 1, 384>), grid, dim3(256), 0, s, D, C);
    } else if (v == 2) {
        dim3 grid((D.g.n[0] + 7) / 8, (D.g.n[1] + 3) / 4, (D.g.n[2] + 3) / 4);
        hipLaunchKernelGGL((k_gather_tile<R, MODE, 8, 4, 4, 1, 640>), grid, dim3(128), 0, s, D, C);
    } else {
        dim3 grid((D.g.n[0] + 15) / 16, (D.g.n[1] + 3) / 4, (D.g.n[2] + 15) / 16);
        hipLaunchKernelGGL((k_gather_tile<R, MODE, 16, 4, 4, 4, 512>), grid, dim3(256), 0, s, D, C);
    }
}
template <typename R> void launch_gather_am(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    launch_gather<R, MODE_AM>(D, C, s);
}
// drag/pressure pass: LDS tiles, or one thread per particle reading its
// stencil cells from global memory (gather variant 3)
template <typename R> void launch_part_drag(const Desc &D, const Cells<R> &C, int record, hipStream_t s)
{
    if (D.pt.np == 0) return;
    if (D.t.gather == 3) {
        hipLaunchKernelGGL(k_part_drag<R>, dim3(nblocks(D.pt.np)), dim3(kBlock), 0, s, D, C, record);
        return;
    }
    const auto tiles = [&](int ty, int tz) {
        return dim3((D.g.n[0] + 15) / 16, (D.g.n[1] + ty - 1) / ty, (D.g.n[2] + tz - 1) / tz);
    };
    // FP32, 2^19 cells and more: tiles of 16x8x8 cells (a halo of 1.76 cells per
    // owned cell, 58 KB), which below that leave CUs without a tile; 16x4x4 there
    // (2.53, 21 KB). A coupled step, 16x8x8 / 16x4x4: 128^3 3.07 / 3.15 ms, 97x90x101
    // 3.69 / 3.68, batch of 12 boxes of 17^3 to 46^3 5.6 / 5.1. FP64: 16x4x4 (41 KB)
    // as long as all tiles are resident at once (3 on each of 256 CUs), else 16x4x8
    // (2.11, 69 KB): 61x53x71 12.6 us against 17.4, 16^3 and 32x32x64 1 to 3 % of a
    // step faster with 16x4x4.
    const dim3 small = tiles(4, 4);
    if (sizeof(R) == 4 && D.g.nc >= (int64_t)1 << 19)
        hipLaunchKernelGGL((k_part_tile<R, PASS_DRAG, 16, sizeof(R) == 4 ? 8 : 4, sizeof(R) == 4 ? 8 : 4, 512>),
                           tiles(8, 8), dim3(512), 0, s, D, C, record);
    else if (sizeof(R) == 8 && (int64_t)small.x * small.y * small.z > 3 * 256)
        hipLaunchKernelGGL((k_part_tile<R, PASS_DRAG, 16, 4, sizeof(R) == 8 ? 8 : 4, 256>), tiles(4, 8), dim3(256), 0, s,
                           D, C, record);
    else
        hipLaunchKernelGGL((k_part_tile<R, PASS_DRAG, 16, 4, 4, 256>), small, dim3(256), 0, s, D, C, record);
}
template <typename R> void launch_gather_fd(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    launch_gather<R, MODE_FD>(D, C, s);
}
template <typename R> void launch_gather_eps(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    launch_gather<R, MODE_EPS>(D, C, s);
}
template <typename R> void launch_gather_eps_uf(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    launch_gather<R, MODE_EPS_UF>(D, C, s);
}
template <typename R> void launch_gather_eps_am(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    launch_gather<R, MODE_EPS_AM>(D, C, s);
}
// The per-cell relaxation time (Eilers, LES) is a separate instance so that
// the constant-tau kernel keeps its code.
// Residency cap: the FP32 instances need few registers and would run 5 or 8
// waves per SIMD. Reserving 40,000 B of (unused) dynamic LDS per 256-thread
// workgroup limits a CU (160 KiB of LDS) to 4 workgroups, 4 waves per SIMD,
// which is fastest for this kernel's 38 PDF streams: on 256 x 256 x 512
// cells 8 waves/SIMD take 1.175 ms, 6 1.15 ms, 5 1.14 ms, 4 1.125 ms and
// 3 1.33 ms. The FP64 instances already run at 4 and 3 waves per SIMD.
template <typename R> void launch_stream_collide(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    const unsigned lds = cell_lds_bytes(D.t.cell_waves, sizeof(R) == 4 ? 40000u : 0u);
    if (D.p.use_eilers || D.p.use_les)
        hipLaunchKernelGGL((k_stream_collide<R, true>), dim3(nblocks(D.g.nc)), dim3(kBlock), lds, s, D, C);
    else
        hipLaunchKernelGGL((k_stream_collide<R, false>), dim3(nblocks(D.g.nc)), dim3(kBlock), lds, s, D, C);
}
template <typename R> void launch_zero(R *p, int64_t n, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_zero<R>, dim3(grid_stride_blocks(n)), dim3(kBlock), 0, s, p, n);
}
template <typename R> void launch_fluid_fraction(const R *src, double *dst, int64_t nc, hipStream_t s)
{
    if (nc > 0)
        hipLaunchKernelGGL((k_fluid_fraction<R>), dim3(grid_stride_blocks(nc)), dim3(kBlock), 0, s, src, dst, nc);
}
template <typename R> void launch_vec4_to_double(const R *src, double *dst, int64_t nc, hipStream_t s)
{
    if (nc > 0)
        hipLaunchKernelGGL((k_vec4_to_soa<R>), dim3(grid_stride_blocks(nc)), dim3(kBlock), 0, s, src, dst, nc);
}
template <typename R> void launch_vec4_w_to_double(const R *src, double *dst, int64_t nc, hipStream_t s)
{
    if (nc > 0) hipLaunchKernelGGL((k_vec4_w<R>), dim3(grid_stride_blocks(nc)), dim3(kBlock), 0, s, src, dst, nc);
}
template <typename R> void launch_to_double(const R *src, double *dst, int64_t n, hipStream_t s)
{
    if (n > 0)
        hipLaunchKernelGGL((k_convert<R, double>), dim3(grid_stride_blocks(n)), dim3(kBlock), 0, s, src, dst, n);
}
template <typename R> void launch_from_double(const double *src, R *dst, int64_t n, hipStream_t s)
{
    if (n > 0)
        hipLaunchKernelGGL((k_convert<double, R>), dim3(grid_stride_blocks(n)), dim3(kBlock), 0, s, src, dst, n);
}
int diag_blocks(const Desc &D)
{
    int64_t n = D.g.nc > D.pt.np ? D.g.nc : D.pt.np;
    int64_t b = (n + kBlock - 1) / kBlock;
    if (b > kDiagMaxBlocks) b = kDiagMaxBlocks;
    return (int)(b < 1 ? 1 : b);
}

// Scratch of the allocation-free diagnostics (lbdem_diagnostics_noalloc):
// the per-block partials and the final values of k_diag / k_diag_final,
// 12 x 1024 + 16 doubles (98.4 KB), one copy per device for the life of the
// process. Host code never names the array itself (on the host it is only a
// stand-in): it uses the device address that hipGetSymbolAddress returns,
// looked up once per device with that device current.
static __device__ __align__(256) double scratch[kDiagScratchDoubles];

double *diag_scratch_on_device(int device)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static double *addr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        int cur = -1;
        if (hipGetDevice(&cur) != hipSuccess || cur != device) return nullptr;
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
        addr[device] = static_cast<double *>(p);
    }
    return addr[device];
}
template <typename R>
void launch_diag(const Desc &D, const Cells<R> &C, const R *df, double *partials, int nblk, double *out,
                 hipStream_t s)
{
    hipLaunchKernelGGL(k_diag<R>, dim3(nblk), dim3(kBlock), 0, s, D, C, df, partials);
    hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(64), 0, s, (const double *)partials, nblk, out);
}

// Lanes per particle of the DEM pass. Fewer lanes are less work in all (the sums
// through LDS, the particle's record and, fused, its integration are then
// shared by more entries); more lanes fill the chip and shorten the chain of
// dependent loads, as long as each has entries enough and all wavefronts are
// resident at once: three on each of 1024 SIMDs, 98,304 particles with two lanes
// and 24,576 with eight.
// A step of 4 x 10 substeps on a jittered lattice, FP64, ms with 1 / 2 / 8 lanes:
//   list entries about    9                    14                   36
//    4,096 particles   0.56 / 0.48 / 0.45   0.90 / 0.70 / 0.52   1.29 / 0.95 / 0.56
//   24,389             0.65 / 0.55 / 0.58   0.99 / 0.77 / 0.71   1.39 / 1.03 / 0.78
//   32,768             0.66 / 0.57 / 0.70   1.00 / 0.78 / 0.87   1.41 / 1.05 / 0.97
//   50,653             0.73 / 0.68 / 0.94   1.06 / 0.96 / 1.20   1.47 / 1.29 / 1.33
//   97,336             0.96 / 0.89 / 1.43   1.41 / 1.26 / 1.87   1.93 / 1.66 / 2.07
//  110,592 (103,823)   0.98 / 1.08 / 1.60   1.43 / 1.57 / 2.10   1.84 / 2.11 / 2.23
// (FP32 within 10 % of these ratios.) With fewer than six entries the lanes find
// little to share (42,808 particles with 3.5: 3.86 / 3.86 / 4.58). Up to 256
// particles one lane means a single launch per subcycle; crowded ones are still
// better off with eight: 216 with 33 entries, 4 x 50 substeps, 7.0 / 3.7 / 1.8.
static inline int dem_lanes(const Desc &D)
{
    const int64_t n = D.pt.np;
    const double r = D.p.reach_max, mean = (double)n / (double)D.g.nc * (4.0 / 3.0) * M_PI * r * r * r;
    if (n > 98304 || mean < 6.0) return 1;
    return mean >= 12.0 && n <= (mean < 20.0 ? 24576 : 32768) ? 8 : 2;
}
template <typename R, bool FUSE>
static void launch_dem(const Desc &D, const Cells<R> &C, int sub, int odd, hipStream_t s)
{
    if (D.pt.np == 0) return;
    const int g = dem_lanes(D);
    const dim3 grid(nblocks(D.pt.np * g)), blk(kBlock);
    if (g == 8) hipLaunchKernelGGL((k_dem_force<R, 8, FUSE, uint32_t>), grid, blk, 0, s, D, C, sub, odd);
    else if (g == 2) hipLaunchKernelGGL((k_dem_force<R, 2, FUSE, uint32_t>), grid, blk, 0, s, D, C, sub, odd);
    else if ((uint64_t)D.pt.np * sizeof(DemRec<R>) <= UINT32_MAX)
        hipLaunchKernelGGL((k_dem_force<R, 1, FUSE, uint32_t>), grid, blk, 0, s, D, C, sub, odd);
    else
        hipLaunchKernelGGL((k_dem_force<R, 1, FUSE, uint64_t>), grid, blk, 0, s, D, C, sub, odd);
}
template <typename R> void launch_dem_force(const Desc &D, const Cells<R> &C, hipStream_t s)
{
    launch_dem<R, false>(D, C, 0, 0, s);
}
bool dem_substep_fused(const Desc &D)
{
    return D.t.fuse != 0;
}
static inline int sub_flags(const Desc &D, int last, int step_end)
{
    if (!last) return 0;
    return SUB_LAST | (step_end ? SUB_END : (D.p.use_lift ? 0 : SUB_AM));
}
// whether a subcycle's substeps run in one launch (enqueued for substep 0 only)
bool dem_subcycle_single(const Desc &D)
{
    return dem_substep_fused(D) && D.p.n_dem > 1 && D.pt.np <= kBlock && dem_lanes(D) == 1;
}
template <typename R>
void launch_dem_substep_fused(const Desc &D, const Cells<R> &C, int k, int sub, hipStream_t s)
{
    if (D.pt.np == 0) return;
    const bool single = dem_subcycle_single(D);
    const int f = sub_flags(D, single || sub == D.p.n_dem - 1, k == D.p.n_int - 1);
    if (single)
        hipLaunchKernelGGL(k_dem_subcycle<R>, dim3(1), dim3((unsigned)((D.pt.np + 63) / 64 * 64)), 0, s, D, C, f);
    else
        launch_dem<R, true>(D, C, f, sub & 1, s);
}
bool dem_sorts_lengths(const Desc &D) { return sort_lengths(D); }
// slots into the order of the sorted list, or the blocked one, if due
void launch_reorder(const Desc &D, hipStream_t s)
{
    if (D.pt.np == 0) return;
    if (D.t.dem_order) {
        const unsigned nb = nblocks(D.o.nrows, kScanPerBlock);
        hipLaunchKernelGGL(k_order_scan, dim3(nb), dim3(kBlock), 0, s, D);
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, D.o.rowsum, (int)nb, D.o.rowsum + nb, D.pt.need + 1);
        hipLaunchKernelGGL(k_order_fill, dim3(nblocks(D.o.nrows)), dim3(kBlock), 0, s, D);
    }
    hipLaunchKernelGGL(k_reorder, dim3(nblocks(D.pt.np)), dim3(kBlock), 0, s, D);
    hipLaunchKernelGGL(k_reorder_back, dim3(nblocks(D.pt.np, kBlock)), dim3(kBlock), 0, s, D);
}
template <typename R> void launch_nlist(const Desc &D, hipStream_t s, bool flag)
{
    if (D.pt.np <= 0) return;
    // few workgroups, as most launches find nothing to do (one wavefront per
    // particle at a build). Idle, the launch is 1 to 3 % of a step of one DEM
    // substep per subcycle; built by the DEM pass instead, up to 64 lists after
    // one another per wavefront, the lists of 13.8 k spheres due every third
    // subcycle made it 0.99 ms long, not 0.77
    const int64_t nb = (D.pt.np + kBlock / 64 - 1) / (kBlock / 64);
    hipLaunchKernelGGL(k_nlist<R>, dim3((unsigned)(nb < 2048 ? nb : 2048)), dim3(kBlock), 0, s, D, flag);
}
template <typename R> void launch_integrate(const Desc &D, const Cells<R> &C, int last, int step_end, hipStream_t s)
{
    if (D.pt.np > 0)
        hipLaunchKernelGGL(k_integrate<R>, dim3(nblocks(D.pt.np)), dim3(kBlock), 0, s, D, C,
                           sub_flags(D, last, step_end));
}
void launch_bin_count(const Desc &D, hipStream_t s)
{
    if (D.pt.np > 0) hipLaunchKernelGGL(k_bin_count, dim3(nblocks(D.pt.np)), dim3(kBlock), 0, s, D);
}
void launch_bin_build(const Desc &D, hipStream_t s)
{
    const unsigned nb = nblocks(D.g.nc, kScanPerBlock);
    // both levels in one launch for up to 256 workgroups (2^19 cells): 113 of them
    // 5.0 us against 4.8 + 4.6; the count, one address, takes 1024 of them longer
    // than the second launch (19.2 us against 7.5 + 4.6)
    const int both = nb <= 256;
    hipLaunchKernelGGL(k_scan_block, dim3(nb), dim3(kBlock), 0, s, D, both);
    if (!both)
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, D.b.bsum, (int)nb, D.b.start + D.g.nc,
                           (const int *)nullptr);
    if (D.pt.np > 0) hipLaunchKernelGGL(k_place, dim3(nblocks(D.pt.np)), dim3(kBlock), 0, s, D);
    hipLaunchKernelGGL(k_cellsort, dim3(nblocks(D.g.nc)), dim3(kBlock), 0, s, D);
}
void launch_pack_particles(const Desc &D, int what, hipStream_t s)
{
    if (D.pt.np > 0) hipLaunchKernelGGL(k_pack_particles, dim3(nblocks(D.pt.np)), dim3(kBlock), 0, s, D, what);
}
void launch_pack_vec(const double *src, int64_t cap, int64_t n, double *out, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_pack_vec, dim3(nblocks(n)), dim3(kBlock), 0, s, src, cap, n, out);
}
void launch_zero_int(int *p, int64_t n, hipStream_t s) { launch_zero<int>(p, n, s); }
void launch_set_int(int *p, int v, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_int, dim3(1), dim3(1), 0, s, p, v);
}
void launch_set_step(long long *stepc, long long v, hipStream_t s)
{
    hipLaunchKernelGGL(k_set_step, dim3(1), dim3(1), 0, s, stepc, v);
}

#define LBDEM_INST(R)                                                                                     \
    template void launch_moments<R>(const Desc &, const Cells<R> &, hipStream_t);                          \
    template void launch_cellfields<R>(const Desc &, const Cells<R> &, hipStream_t);                       \
    template void launch_curl<R>(const Desc &, const Cells<R> &, hipStream_t);                            \
    template void launch_dem_force<R>(const Desc &, const Cells<R> &, hipStream_t);                       \
    template void launch_dem_substep_fused<R>(const Desc &, const Cells<R> &, int, int, hipStream_t);      \
    template void launch_nlist<R>(const Desc &, hipStream_t, bool);                                        \
    template void launch_integrate<R>(const Desc &, const Cells<R> &, int, int, hipStream_t);              \
    template void launch_part_am<R>(const Desc &, const Cells<R> &, hipStream_t);                          \
    template void launch_gather_am<R>(const Desc &, const Cells<R> &, hipStream_t);                        \
    template void launch_part_drag<R>(const Desc &, const Cells<R> &, int, hipStream_t);                        \
    template void launch_gather_fd<R>(const Desc &, const Cells<R> &, hipStream_t);                        \
    template void launch_gather_eps<R>(const Desc &, const Cells<R> &, hipStream_t);                       \
    template void launch_gather_eps_am<R>(const Desc &, const Cells<R> &, hipStream_t);                    \
    template void launch_gather_eps_uf<R>(const Desc &, const Cells<R> &, hipStream_t);                    \
    template void launch_stream_collide<R>(const Desc &, const Cells<R> &, hipStream_t);                   \
    template void launch_zero<R>(R *, int64_t, hipStream_t);                                                \
    template void launch_to_double<R>(const R *, double *, int64_t, hipStream_t);                          \
    template void launch_vec4_to_double<R>(const R *, double *, int64_t, hipStream_t);                     \
    template void launch_vec4_w_to_double<R>(const R *, double *, int64_t, hipStream_t);                   \
    template void launch_fluid_fraction<R>(const R *, double *, int64_t, hipStream_t);                     \
    template void launch_from_double<R>(const double *, R *, int64_t, hipStream_t);                        \
    template void launch_diag<R>(const Desc &, const Cells<R> &, const R *, double *, int, double *, hipStream_t);

LBDEM_INST(float)
LBDEM_INST(double)

}  // namespace lbdem
