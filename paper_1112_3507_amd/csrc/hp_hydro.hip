// hp_hydro.hip -- the steps of the fractional-step algorithm either side of the pressure solve.
//
// Section 2, "The Algorithm": before the solve, steps (iv)-(v) form the right-hand side f of
// eq. fpoiss (one component) or eq. fpoiss2 (two components), here multiplied by dt^2 like the
// operator (b = dt^2 f):
//
//     b = m (P^n - dt u^n . grad P^n) - dt div u* - (2 dt / 3)(m / rho^n) G
//         - (3 dt / 4) m R_gas T^n div(rho^n kappa_c grad c^n),      m = 1 / (rho^n c2^n),
//
// with grad P^n from the density-weighted interface pressure of eq. pbnd and the central
// difference of eq. nablaP, and div u* from the interface velocity of eq. step1 applied to
// u* = (rho u)* / rho^{n+1}. After the solve, steps (vii)-(ix) update the momentum
// (eq. momupdate, grad P by eqs. pbnd and nablaP with rho^{n+1}), the interface velocities
// (step (viii): u*_{i+1/2} - dt (P_{i+1} - P_i) / h * 2 / (rho_{i+1} + rho_i)) and the total energy
// (eq. enupdate: e* - dt (P div u^{n+1} + u^{n+1} . grad P), div from the new interface
// velocities, u^{n+1} = (rho u)^{n+1} / rho^{n+1} at the cell).
//
// Boundaries as in the solve: periodic axes wrap; at a closed (Neumann) boundary the interface
// velocity is zero and the interface pressure is the cell's own; an axis of one cell has no
// gradient or divergence. The interface value of rho kappa_c is the mean of its two cells.
//
// Both passes walk z columns over natural-order FP64 arrays (HBM-bound, about 1 flop per byte):
// workgroups of 64 columns in x and a few rows in y so that x neighbours come from the same cache lines and
// y neighbours from rows the workgroup itself loads; the z neighbours stay in registers.
#include "hp.h"
#include "hp_internal.h"

namespace {

struct HGeo {
    int n[3];
    int per[3];   // 1: periodic with n >= 2 (wrap faces)
    double h[3];
    double dt;
};

// Neighbour of cell c along axis d in direction s (+1 / -1): its coordinate in *t, false when
// there is no face (closed boundary).
__device__ __forceinline__ bool neighbour(const HGeo& g, int d, int c, int s, int* t) {
    int q = c + s;
    const int n = g.n[d];
    if (q < 0 || q >= n) {
        if (!g.per[d]) return false;
        q = q < 0 ? n - 1 : 0;
    }
    *t = q;
    return true;
}

__device__ __forceinline__ int64_t cell(const HGeo& g, int i, int j, int k) {
    return i + (int64_t)g.n[0] * (j + (int64_t)g.n[1] * k);
}

// eq. pbnd: the pressure at the interface between cells a and b
__device__ __forceinline__ double pbnd(double pa, double ra, double pb, double rb) {
    return (pb * ra + pa * rb) / (ra + rb);
}

struct RhsArgs {
    const double *rho_n, *c2_n, *p_n, *mom_n, *rho_np1, *mom_star, *visc, *temp_n, *conc_n, *rkc_n;
    double r_gas;
    int64_t N;
    double* b;
};

// z planes per chunk of a column pass with `tiles` column tiles per plane and `threads` threads per
// workgroup: up to 32, fewer (not under 2) where the launch would leave the 256 CUs short of 2048
// threads each. A chunk loads its first planes' z neighbours again, so longer ones read less; at
// 48 x 32 x 44 chunks of 2 against 4 planes took the update from 10.1 to 7.0 us, at 96 x 80 x 72
// (16 before) from 39.6 to 19.8, and single planes made the advection there slower (25 for 22).
static int hydro_chunk(int nz, int64_t tiles, int threads) {
    const int64_t want = (int64_t)256 * 2048 / threads;   // workgroups that fill the GPU once
    const int64_t kz = nz * tiles / want;
    return (int)(kz < 2 ? 2 : kz > 32 ? 32 : kz);
}

constexpr int kHRows = 4;  // rows of a column tile

// Column tile (64 x kHRows columns, one chunk of kz planes) of this workgroup of a 1-D grid. The
// hardware hands workgroup L to XCD L % 8; numbering the tiles so that each XCD takes one
// contiguous range of them (whole x-y planes of chunks) keeps the y neighbour rows of a tile in
// the L2 of the XCD that reads them.
struct HTiles {
    int tx, ty, tz, kz;
};

__device__ __forceinline__ void htile(const HTiles& t, int& i, int& j, int& k0) {
    const unsigned total = (unsigned)t.tx * t.ty * t.tz;
    unsigned L = blockIdx.x;
    if ((total & 7u) == 0) L = (L & 7u) * (total >> 3) + (L >> 3);
    i = (int)(L % (unsigned)t.tx) * 64 + (threadIdx.x & 63);
    j = (int)((L / (unsigned)t.tx) % (unsigned)t.ty) * kHRows + (threadIdx.x >> 6);
    k0 = (int)(L / ((unsigned)t.tx * t.ty)) * t.kz;
}

static HTiles htiles(const int n[3]) {
    const int tx = (n[0] + 63) / 64, ty = (n[1] + kHRows - 1) / kHRows;
    const int kz = hydro_chunk(n[2], (int64_t)tx * ty, 64 * kHRows);
    return HTiles{tx, ty, (n[2] + kz - 1) / kz, kz};
}

// Neighbours of the cells of one axis, as the three values (low neighbour, cell, high neighbour)
// of each array, and whether the two faces exist.
struct Line {
    bool lo, hi;
    double p[3], rn[3], r1[3], ms[3], c[3], k[3];
};

// The contributions of one axis to the rhs (steps (iv)-(v)): u_d (grad P^n)_d, (div u*)_d and the
// d-part of div(rho kappa_c grad c); ih = 1/h_d.
__device__ __forceinline__ void rhs_axis(const Line& L, double ud, double ih, bool tc, double& adv, double& divu,
                                         double& dc) {
    const double phi = L.hi ? pbnd(L.p[1], L.rn[1], L.p[2], L.rn[2]) : L.p[1];
    const double plo = L.lo ? pbnd(L.p[0], L.rn[0], L.p[1], L.rn[1]) : L.p[1];
    adv += ud * ((phi - plo) * ih);
    const double uhi = L.hi ? (L.ms[1] + L.ms[2]) / (L.r1[1] + L.r1[2]) : 0.0;
    const double ulo = L.lo ? (L.ms[0] + L.ms[1]) / (L.r1[0] + L.r1[1]) : 0.0;
    divu += (uhi - ulo) * ih;
    if (tc) {
        const double fhi = L.hi ? 0.5 * (L.k[1] + L.k[2]) * (L.c[2] - L.c[1]) * ih : 0.0;
        const double flo = L.lo ? 0.5 * (L.k[0] + L.k[1]) * (L.c[1] - L.c[0]) * ih : 0.0;
        dc += (fhi - flo) * ih;
    }
}

// x or y neighbour line of cell a (coordinate c along axis d, stride st): the neighbours from
// memory, the cell itself from the z ring Z; ms is the momentum component of axis d
__device__ __forceinline__ void load_line(const HGeo& g, const RhsArgs& A, const double* ms, int d, int c, int64_t a,
                                          int64_t st, bool tc, const Line& Z, Line& L) {
    int tl, th;
    L.lo = neighbour(g, d, c, -1, &tl);
    L.hi = neighbour(g, d, c, 1, &th);
    const int64_t bl = L.lo ? a + (int64_t)(tl - c) * st : a, bh = L.hi ? a + (int64_t)(th - c) * st : a;
    L.p[1] = Z.p[1];
    L.rn[1] = Z.rn[1];
    L.r1[1] = Z.r1[1];
    L.ms[1] = ms[a];
    L.c[1] = Z.c[1];
    L.k[1] = Z.k[1];
    const int64_t idx[2] = {bl, bh};
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int q = 2 * e;
        L.p[q] = A.p_n[idx[e]];
        L.rn[q] = A.rho_n[idx[e]];
        L.r1[q] = A.rho_np1[idx[e]];
        L.ms[q] = ms[idx[e]];
        L.c[q] = tc ? A.conc_n[idx[e]] : 0.0;
        L.k[q] = tc ? A.rkc_n[idx[e]] : 0.0;
    }
}

// One thread per (x, y) column walking kz planes: the x and y neighbours come from memory (the
// x ones from the same cache lines), the z neighbours of the six stencil arrays from a ring of
// registers (each plane is loaded once per column). Every load of a plane is issued whatever the
// geometry (a missing neighbour, or an axis of one cell, reads the cell itself and contributes
// nothing): with loads under branches the compiler cannot count what is in flight and waited
// for the next plane's z loads before using this plane's values.
// TC: the two-component terms (temp_n, conc_n, rkc_n given); VISC: the viscous term (visc given).
template <bool TC, bool VISC>
__global__ __launch_bounds__(64 * kHRows) void k_pressure_rhs(HGeo g, HTiles t, RhsArgs A) {
    int i, j, k0;
    htile(t, i, j, k0);
    if (i >= g.n[0] || j >= g.n[1]) return;
    const int nz = g.n[2];
    const int k1 = min(k0 + t.kz, nz);
    const int64_t sxy = (int64_t)g.n[0] * g.n[1];
    constexpr bool tc = TC;
    const double ih[3] = {1.0 / g.h[0], 1.0 / g.h[1], 1.0 / g.h[2]};
    const double* msz = A.mom_star + 2 * A.N;
    const int64_t col = cell(g, i, j, 0);
    // ring: z line values of planes k-1, k, k+1 (position 0, 1, 2)
    Line Z;
    auto load_plane = [&](int kp, int q) {
        const int64_t a = col + (int64_t)kp * sxy;
        Z.p[q] = A.p_n[a];
        Z.rn[q] = A.rho_n[a];
        Z.r1[q] = A.rho_np1[a];
        Z.ms[q] = msz[a];
        Z.c[q] = tc ? A.conc_n[a] : 0.0;
        Z.k[q] = tc ? A.rkc_n[a] : 0.0;
    };
    int tz = k0;
    load_plane(neighbour(g, 2, k0, -1, &tz) ? tz : k0, 0);
    load_plane(k0, 1);
    for (int k = k0; k < k1; ++k) {
        Z.lo = nz > 1 && neighbour(g, 2, k, -1, &tz);
        tz = k;
        Z.hi = nz > 1 && neighbour(g, 2, k, 1, &tz);
        load_plane(tz, 2);
        const int64_t a = col + (int64_t)k * sxy;
        const double irn = 1.0 / Z.rn[1];
        const double m = irn / A.c2_n[a];
        double adv = 0.0, divu = 0.0, dc = 0.0;
        // (an axis of one cell has no faces: its lines contribute exact zeros)
        Line L;
        load_line(g, A, A.mom_star, 0, i, a, 1, tc, Z, L);
        rhs_axis(L, A.mom_n[a] * irn, ih[0], tc, adv, divu, dc);
        load_line(g, A, A.mom_star + A.N, 1, j, a, g.n[0], tc, Z, L);
        rhs_axis(L, A.mom_n[A.N + a] * irn, ih[1], tc, adv, divu, dc);
        rhs_axis(Z, A.mom_n[2 * A.N + a] * irn, ih[2], tc, adv, divu, dc);
        double b = m * (Z.p[1] - g.dt * adv) - g.dt * divu;
        if constexpr (VISC) b -= (2.0 * g.dt / 3.0) * (m * irn) * A.visc[a];
        if (tc) b -= (3.0 * g.dt / 4.0) * m * A.r_gas * A.temp_n[a] * dc;
        A.b[a] = b;
        // the ring moves up one plane
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            Z.p[q] = Z.p[q + 1];
            Z.rn[q] = Z.rn[q + 1];
            Z.r1[q] = Z.r1[q + 1];
            Z.ms[q] = Z.ms[q + 1];
            Z.c[q] = Z.c[q + 1];
            Z.k[q] = Z.k[q + 1];
        }
    }
}

struct UpdArgs {
    const double *p, *rho_np1, *mom_star, *e_star;
    double *mom_out, *uface_out, *e_out;
    int64_t N;
};

// The updates of one axis (steps (vii)-(viii)): grad P with rho^{n+1}, the high interface
// velocity u^{n+1} (returned through uf) and the axis' part of its divergence
__device__ __forceinline__ double upd_axis(bool lo, bool hi, const double* p, const double* r, const double* ms,
                                           double dt, double ih, double& uf, double& divn) {
    const double phi = hi ? pbnd(p[1], r[1], p[2], r[2]) : p[1];
    const double plo = lo ? pbnd(p[0], r[0], p[1], r[1]) : p[1];
    uf = hi ? (ms[1] + ms[2]) / (r[1] + r[2]) - dt * (p[2] - p[1]) * ih * 2.0 / (r[2] + r[1]) : 0.0;
    const double ul = lo ? (ms[0] + ms[1]) / (r[0] + r[1]) - dt * (p[1] - p[0]) * ih * 2.0 / (r[1] + r[0]) : 0.0;
    divn += (uf - ul) * ih;
    return (phi - plo) * ih;
}

__global__ __launch_bounds__(64 * kHRows) void k_pressure_update(HGeo g, HTiles t, UpdArgs A) {
    int i, j, k0;
    htile(t, i, j, k0);
    if (i >= g.n[0] || j >= g.n[1]) return;
    const int nz = g.n[2];
    const int k1 = min(k0 + t.kz, nz);
    const int64_t sxy = (int64_t)g.n[0] * g.n[1];
    const double ih[3] = {1.0 / g.h[0], 1.0 / g.h[1], 1.0 / g.h[2]};
    const double* msz = A.mom_star + 2 * A.N;
    const int64_t col = cell(g, i, j, 0);
    double zp[3] = {0.0, 0.0, 0.0}, zr[3] = {1.0, 1.0, 1.0}, zm[3] = {0.0, 0.0, 0.0};
    auto load_plane = [&](int kp, int q) {
        const int64_t a = col + (int64_t)kp * sxy;
        zp[q] = A.p[a];
        zr[q] = A.rho_np1[a];
        zm[q] = msz[a];
    };
    // (unconditional loads, as in k_pressure_rhs: an axis of one cell has no faces and its
    // terms are exact zeros)
    int tz = k0;
    load_plane(neighbour(g, 2, k0, -1, &tz) ? tz : k0, 0);
    load_plane(k0, 1);
    for (int k = k0; k < k1; ++k) {
        const bool zlo = nz > 1 && neighbour(g, 2, k, -1, &tz);
        tz = k;
        const bool zhi = nz > 1 && neighbour(g, 2, k, 1, &tz);
        load_plane(tz, 2);
        const int64_t a = col + (int64_t)k * sxy;
        const int c[2] = {i, j};
        const int64_t st[2] = {1, g.n[0]};
        double gp[3] = {0.0, 0.0, 0.0}, uf[3] = {0.0, 0.0, 0.0}, divn = 0.0;
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            int tl, th;
            const bool lo = neighbour(g, d, c[d], -1, &tl), hi = neighbour(g, d, c[d], 1, &th);
            const int64_t bl = lo ? a + (int64_t)(tl - c[d]) * st[d] : a;
            const int64_t bh = hi ? a + (int64_t)(th - c[d]) * st[d] : a;
            const double* ms = A.mom_star + (int64_t)d * A.N;
            const double pv[3] = {A.p[bl], zp[1], A.p[bh]};
            const double rv[3] = {A.rho_np1[bl], zr[1], A.rho_np1[bh]};
            const double mv[3] = {ms[bl], ms[a], ms[bh]};
            gp[d] = upd_axis(lo, hi, pv, rv, mv, g.dt, ih[d], uf[d], divn);
        }
        gp[2] = upd_axis(zlo, zhi, zp, zr, zm, g.dt, ih[2], uf[2], divn);
        // step (vii): momentum; step (ix): e^{n+1} = e* - dt (P div u^{n+1} + u^{n+1} . grad P)
        const double ir = 1.0 / zr[1];
        double ug = 0.0;
        for (int d = 0; d < 3; ++d) {
            const double md = A.mom_star[(int64_t)d * A.N + a] - g.dt * gp[d];
            A.mom_out[(int64_t)d * A.N + a] = md;
            A.uface_out[(int64_t)d * A.N + a] = uf[d];
            ug += (md * ir) * gp[d];
        }
        A.e_out[a] = A.e_star[a] - g.dt * (zp[1] * divn + ug);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            zp[q] = zp[q + 1];
            zr[q] = zr[q + 1];
            zm[q] = zm[q + 1];
        }
    }
}

// ---- the explicit advective part (steps (i)-(iii)) and the equation of state ----

// the cell that stands at coordinate q along axis d, up to a few past either end: wrapped on a
// periodic axis, the edge cell repeated beyond a closed boundary (a zero-gradient mirror for the
// reconstruction)
__device__ __forceinline__ int reach(const HGeo& g, int d, int q) {
    const int n = g.n[d];
    if (g.per[d]) return ((q % n) + n) % n;
    return q < 0 ? 0 : (q >= n ? n - 1 : q);
}

// second-order ENO: the smaller in magnitude of the two one-sided differences (ties: the second)
__device__ __forceinline__ double eno_slope(double dm, double dp) { return fabs(dm) < fabs(dp) ? dm : dp; }

// the flux through the interface between cells of values ql (low) and qh (high) and slopes sl, sh,
// the value reconstructed on the upwind side of the interface velocity u (selected, then added: a
// choice between two sums compiles to divergent branches)
__device__ __forceinline__ double eno_flux(double u, double ql, double sl, double qh, double sh) {
    const bool up = u >= 0.0;
    const double q = up ? ql : qh, s = up ? sl : -sh;
    return u * (q + 0.5 * s);
}

// flux through the high interface of a cell minus that through its low one, from the cells at
// -2 .. +2 along the axis
__device__ __forceinline__ double axis_div(double ul, double uh, double v0, double v1, double v2, double v3, double v4) {
    const double d0 = v1 - v0, d1 = v2 - v1, d2 = v3 - v2, d3 = v4 - v3;
    const double s = eno_slope(d1, d2);
    return eno_flux(uh, v2, s, v3, eno_slope(d2, d3)) - eno_flux(ul, v1, eno_slope(d0, d1), v2, s);
}

// eq. step1: the interface velocity from the momenta and densities of its two cells; zero at a
// closed boundary
__device__ __forceinline__ double step1(bool face, double ma, double mb, double ra, double rb) {
    return face ? (ma + mb) / (ra + rb) : 0.0;
}

struct AdvArgs {
    const double* q[5];  // rho, the three momenta, e
    double* out[5];
};

// Column tiles of the advection: 32 x 8 columns (whole 256-byte lines in x, and the fewest halo cells
// that leaves), chunks of kz planes.
constexpr int kAdvX = 32, kAdvY = 8, kAdvThreads = kAdvX * kAdvY;
static_assert(4 * kAdvX + 4 * kAdvY <= kAdvThreads, "one halo cell per thread");

// q* = q - dt div(flux) for the five conserved fields (rho, three momenta, e), the fluxes through
// the interfaces of every cell from eq. step1 and the upwind reconstruction.
//
// A workgroup walks a tile of columns through kz planes. Each plane of the tile goes through LDS
// with two cells of halo on every side (own cells from registers, one halo cell per thread from
// memory), so the eight x and y neighbours of a field cost one load; the z neighbours stay in a
// ring of four planes, and the flux through a cell's low z interface is the one its lower
// neighbour computed. The next plane's loads are in flight while a plane is computed. Bound by
// memory: 380 us at 256^3 for 1.4 GB read (the halo rows come from beyond the L2 as often as not)
// and 0.67 GB written; one thread per cell, with every neighbour from memory and every flux
// twice, took 1041 us. Tiles of 512 threads left one workgroup per CU (510 us) or spilled.
__global__ __launch_bounds__(kAdvThreads, 3) void k_advect(HGeo g, HTiles t, AdvArgs A) {
    constexpr int TX = kAdvX, TY = kAdvY, PX = TX + 4, PY = TY + 4;
    __shared__ double tile[2][5][PY * PX];
    // each XCD takes one contiguous range of tiles (see htile)
    const unsigned total = (unsigned)t.tx * t.ty * t.tz;
    unsigned L = blockIdx.x;
    if ((total & 7u) == 0) L = (L & 7u) * (total >> 3) + (L >> 3);
    const int x0 = (int)(L % (unsigned)t.tx) * TX, y0 = (int)((L / (unsigned)t.tx) % (unsigned)t.ty) * TY;
    const int k0 = (int)(L / ((unsigned)t.tx * t.ty)) * t.kz, k1 = min(k0 + t.kz, g.n[2]);
    const int tid = threadIdx.x, lx = tid % TX, ly = tid / TX;
    const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
    const int i = x0 + lx, j = y0 + ly;
    // Positions past the end of an axis hold what its last cells see there (their halo); nothing
    // past the second is read by a cell of the grid.
    auto colx = [&](int q) { return reach(g, 0, min(q, nx + 1)); };
    auto coly = [&](int q) { return reach(g, 1, min(q, ny + 1)); };
    const int64_t sxy = (int64_t)nx * ny;
    const int own = colx(i) + nx * coly(j);
    // the thread's halo cell: two rows below and above the tile, two columns left and right
    int hx = 0, hy = 0;
    const bool halo = tid < 4 * TX + 4 * TY;
    if (tid < 4 * TX) {
        const int r = tid / TX;
        hx = lx;
        hy = r < 2 ? r - 2 : TY + r - 2;
    } else if (halo) {
        const int c = (tid - 4 * TX) & 3;
        hx = c < 2 ? c - 2 : TX + c - 2;
        hy = (tid - 4 * TX) >> 2;
    }
    const int hcell = colx(x0 + hx) + nx * coly(y0 + hy);
    const int hat = (hy + 2) * PX + hx + 2, at = (ly + 2) * PX + lx + 2;
    const double ih[3] = {1.0 / g.h[0], 1.0 / g.h[1], 1.0 / g.h[2]};
    const bool xl = g.per[0] || i > 0, xh = g.per[0] || i < nx - 1;
    const bool yl = g.per[1] || j > 0, yh = g.per[1] || j < ny - 1;
    const bool inside = i < nx && j < ny;

    double q0[5], q1[5], q2[5], q3[5], fz[5], hv[5];
    auto load = [&](double* v, int cell_, int k) {
        const int64_t a = cell_ + (int64_t)reach(g, 2, k) * sxy;
#pragma unroll
        for (int f = 0; f < 5; ++f) v[f] = A.q[f][a];
    };
    load(q0, own, k0 - 2);
    load(q1, own, k0 - 1);
    load(q2, own, k0);
    load(q3, own, k0 + 1);
    load(hv, hcell, k0);
    {
        const double u = step1(g.per[2] || k0 > 0, q1[3], q2[3], q1[0], q2[0]);
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            const double d1 = q2[f] - q1[f];
            fz[f] = eno_flux(u, q1[f], eno_slope(q1[f] - q0[f], d1), q2[f], eno_slope(d1, q3[f] - q2[f]));
            q0[f] = q1[f];
            q1[f] = q2[f];
            q2[f] = q3[f];
        }
    }
    load(q3, own, k0 + 2);
    // one plane from v0 .. v3, planes k-1 .. k+2 of the own column; v0 then takes plane k+3, so that
    // the ring turns by the names below and nothing is copied
    auto plane = [&](int k, double* v0, double* v1, double* v2, double* v3) {
        double(*p)[PY * PX] = tile[k & 1];
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            p[f][at] = v1[f];
            if (halo) p[f][hat] = hv[f];
        }
        __syncthreads();  // (the other slot's readers passed the previous plane's barrier)
        load(hv, hcell, min(k + 1, k1 - 1));
        // interface velocities; zero on an axis of one cell, whose fluxes then cancel to zero
        const double uxl = step1(xl, p[1][at - 1], v1[1], p[0][at - 1], v1[0]);
        const double uxh = step1(xh, v1[1], p[1][at + 1], v1[0], p[0][at + 1]);
        const double uyl = step1(yl, p[2][at - PX], v1[2], p[0][at - PX], v1[0]);
        const double uyh = step1(yh, v1[2], p[2][at + PX], v1[0], p[0][at + PX]);
        const double uzh = step1(g.per[2] || k < nz - 1, v1[3], v2[3], v1[0], v2[0]);
        const int64_t a = own + (int64_t)k * sxy, an = own + (int64_t)reach(g, 2, k + 3) * sxy;
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            const double* c = p[f] + at;
            double div = axis_div(uxl, uxh, c[-2], c[-1], v1[f], c[1], c[2]) * ih[0];
            div += axis_div(uyl, uyh, c[-2 * PX], c[-PX], v1[f], c[PX], c[2 * PX]) * ih[1];
            const double d1 = v2[f] - v1[f];
            const double fh = eno_flux(uzh, v1[f], eno_slope(v1[f] - v0[f], d1), v2[f], eno_slope(d1, v3[f] - v2[f]));
            v0[f] = A.q[f][an];
            div += (fh - fz[f]) * ih[2];
            fz[f] = fh;
            if (inside) A.out[f][a] = v1[f] - g.dt * div;
        }
    };
    for (int k = k0; k < k1;) {
        plane(k, q0, q1, q2, q3);
        if (++k == k1) break;
        plane(k, q1, q2, q3, q0);
        if (++k == k1) break;
        plane(k, q2, q3, q0, q1);
        if (++k == k1) break;
        plane(k, q3, q0, q1, q2);
        ++k;
    }
}

// ideal gas: P = (gamma - 1)(e - |rho u|^2 / (2 rho)), c_s^2 = gamma P / rho
__global__ __launch_bounds__(256) void k_eos(const double* __restrict__ rho, const double* __restrict__ mom,
                                             const double* __restrict__ e, double gamma, double* __restrict__ p,
                                             double* __restrict__ c2, int64_t N) {
    const int64_t a = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (a >= N) return;
    const double r = rho[a], mx = mom[a], my = mom[N + a], mz = mom[2 * N + a];
    const double pa = (gamma - 1.0) * (e[a] - 0.5 * (mx * mx + my * my + mz * mz) / r);
    p[a] = pa;
    if (c2) c2[a] = gamma * pa / r;
}

}  // namespace

namespace hp {

int hydro_launch_advect(const int n[3], const int bc[3], const double h[3], double dt, const double* rho,
                        const double* mom, const double* e, double* rho_out, double* mom_out, double* e_out,
                        hipStream_t s) {
    HGeo g;
    for (int d = 0; d < 3; ++d) {
        g.n[d] = n[d];
        g.per[d] = (bc[d] == HP_BC_PERIODIC && n[d] >= 2);
        g.h[d] = h[d];
    }
    g.dt = dt;
    const int64_t N = (int64_t)n[0] * n[1] * n[2];
    AdvArgs A{{rho, mom, mom + N, mom + 2 * N, e}, {rho_out, mom_out, mom_out + N, mom_out + 2 * N, e_out}};
    HTiles t{(n[0] + kAdvX - 1) / kAdvX, (n[1] + kAdvY - 1) / kAdvY, 1, 1};
    t.kz = hydro_chunk(n[2], (int64_t)t.tx * t.ty, kAdvThreads);
    t.tz = (n[2] + t.kz - 1) / t.kz;
    hipLaunchKernelGGL(k_advect, dim3((unsigned)((int64_t)t.tx * t.ty * t.tz)), dim3(kAdvThreads), 0, s, g, t, A);
    return hipGetLastError() == hipSuccess ? HP_OK : HP_EHIP;
}

int hydro_launch_eos(int64_t N, const double* rho, const double* mom, const double* e, double gamma, double* p,
                     double* c2, hipStream_t s) {
    hipLaunchKernelGGL(k_eos, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, rho, mom, e, gamma, p, c2, N);
    return hipGetLastError() == hipSuccess ? HP_OK : HP_EHIP;
}

int hydro_launch_rhs(const int n[3], const int bc[3], const double h[3], double dt, const hp_rhs_fields* f,
                     double* rhs, hipStream_t s) {
    HGeo g;
    for (int d = 0; d < 3; ++d) {
        g.n[d] = n[d];
        g.per[d] = (bc[d] == HP_BC_PERIODIC && n[d] >= 2);
        g.h[d] = h[d];
    }
    g.dt = dt;
    RhsArgs A{f->rho_n, f->c2_n, f->p_n, f->mom_n, f->rho_np1, f->mom_star, f->visc, f->temp_n, f->conc_n,
              f->rkc_n, f->r_gas, (int64_t)n[0] * n[1] * n[2], rhs};
    const HTiles t = htiles(n);
    const dim3 grid((unsigned)t.tx * t.ty * t.tz);
    if (f->temp_n && f->visc)
        hipLaunchKernelGGL((k_pressure_rhs<true, true>), grid, dim3(64 * kHRows), 0, s, g, t, A);
    else if (f->temp_n)
        hipLaunchKernelGGL((k_pressure_rhs<true, false>), grid, dim3(64 * kHRows), 0, s, g, t, A);
    else if (f->visc)
        hipLaunchKernelGGL((k_pressure_rhs<false, true>), grid, dim3(64 * kHRows), 0, s, g, t, A);
    else
        hipLaunchKernelGGL((k_pressure_rhs<false, false>), grid, dim3(64 * kHRows), 0, s, g, t, A);
    return hipGetLastError() == hipSuccess ? HP_OK : HP_EHIP;
}

int hydro_launch_update(const int n[3], const int bc[3], const double h[3], double dt,
                        const hp_update_fields* f, hipStream_t s) {
    HGeo g;
    for (int d = 0; d < 3; ++d) {
        g.n[d] = n[d];
        g.per[d] = (bc[d] == HP_BC_PERIODIC && n[d] >= 2);
        g.h[d] = h[d];
    }
    g.dt = dt;
    UpdArgs A{f->p, f->rho_np1, f->mom_star, f->e_star, f->mom_out, f->uface_out, f->e_out,
              (int64_t)n[0] * n[1] * n[2]};
    const HTiles t = htiles(n);
    hipLaunchKernelGGL(k_pressure_update, dim3((unsigned)t.tx * t.ty * t.tz), dim3(64 * kHRows), 0, s, g, t, A);
    return hipGetLastError() == hipSuccess ? HP_OK : HP_EHIP;
}

}  // namespace hp
