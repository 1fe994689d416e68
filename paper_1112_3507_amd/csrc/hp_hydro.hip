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
// The passes walk z over natural-order FP64 arrays (HBM-bound, about 1 flop per byte) in tiles of 32 x 8
// columns, one thread each: a plane of the tile and its halo goes through LDS, so that a cell's values and what
// depends on them alone are loaded and computed once; the z neighbours stay in registers.
#include "hp.h"
#include "hp_internal.h"

#include <type_traits>

namespace {

struct HGeo {
    int n[3];
    int per[3];   // 1: periodic with n >= 2 (wrap faces)
    double h[3];
    double dt;
};

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

// z planes per chunk of a pass with `tiles` column tiles of `threads` threads per plane. A chunk loads its first planes' z
// neighbours again, so longer ones read less, and there have to be enough of them for 256 CUs. Counted in
// workgroups of 256 threads, two per CU are enough from 4096 tiles' planes on (kz = 8; right-hand side at 256 x 256 x 32: 16
// planes 40 us, 8 43, 4 47); below that kz is at most 3, and at least 2 (96 x 80 x 72: 1, 2, 4 and 16 planes take 24, 17, 19 and 24
// us there). More than 16 planes pay only where eight workgroups per CU remain (256^3, advection: 32 planes 406 us, 16
// 424; 192^3: 199 and 195).
static int hydro_chunk(int nz, int64_t tiles, int threads) {
    const int64_t planes = nz * tiles * threads / 256;
    const int64_t kz = planes >= 4096 ? (planes < 512 * 16 ? planes / 512 : 16) : planes / 1024;
    return (int)(kz < 2 ? 2 : planes / 2048 < kz ? kz : planes / 2048 > 32 ? 32 : planes / 2048);
}

// the cell that stands at coordinate q along axis d, up to a few past either end: wrapped on a
// periodic axis, the edge cell repeated beyond a closed boundary (a zero-gradient mirror for the
// reconstruction; behind a face that doesn't exist nothing is used)
__device__ __forceinline__ int reach(const HGeo& g, int d, int q) {
    const int n = g.n[d];
    if (g.per[d]) return ((q % n) + n) % n;
    return q < 0 ? 0 : (q >= n ? n - 1 : q);
}

// How a pass takes a box, by column tiles and chunks of kz planes, one thread per column. FORM_BOX: tiles of 32 x 8 columns
// (whole 256-byte lines in x, and the fewest halo cells that leaves). 1 .. kFlatRows: boxes of so many rows, 64 columns by
// all of them, whose y neighbours are in the tile itself (most rows of a 32 x 8 tile would repeat what
// others do: 1024 x 1 x 1024 cells take 21, 20 and 27 us so in right-hand side, update and advection, 77, 78 and 102
// there; 1024 x 4 x 1024 96, 98 and 112 instead of 119, 128 and 159; from five rows on 32 x 8 is no slower than the 64 x 4
// columns, every neighbour from memory, were before). FORM_PLANE: 32 x 8 on a single plane, without the loads of z
// neighbours (4096 x 4096 x 1: right-hand side and update 308 and 349 us, 493 and 509 with them; the advection, for which it
// makes no difference, takes such a plane as a box).
constexpr int FORM_BOX = 0, kFlatRows = 4, FORM_PLANE = 5;
constexpr int kTileX = 32, kTileY = 8, kFlatX = 64;

static int form_of(const int n[3]) { return n[1] <= kFlatRows ? n[1] : n[2] == 1 ? FORM_PLANE : FORM_BOX; }
constexpr int rows_of(int form) { return form >= 1 && form <= kFlatRows ? form : 0; }  // 0: 32 x 8
constexpr int threads_of(int form) { return rows_of(form) ? kFlatX * rows_of(form) : kTileX * kTileY; }

// go(the form of the box n as a constant)
template <typename F>
static void with_form(const int n[3], F&& go) {
    switch (form_of(n)) {
        case 1: go(std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 3: go(std::integral_constant<int, 3>{}); break;
        case 4: go(std::integral_constant<int, 4>{}); break;
        case FORM_PLANE: go(std::integral_constant<int, FORM_PLANE>{}); break;
        default: go(std::integral_constant<int, FORM_BOX>{}); break;
    }
}

// The hardware hands workgroup L to XCD L % 8; the tiles are numbered so that each XCD takes one contiguous range of them
// (whole x-y planes of chunks), which keeps the halo rows of a tile in the L2 of the XCD that reads them.
struct HTiles {
    int tx, ty, tz, kz;
};

static HTiles htiles(const int n[3]) {
    const int form = form_of(n), w = rows_of(form) ? kFlatX : kTileX, r = rows_of(form) ? rows_of(form) : kTileY;
    const int tx = (n[0] + w - 1) / w, ty = (n[1] + r - 1) / r;
    const int kz = hydro_chunk(n[2], (int64_t)tx * ty, threads_of(form));
    return HTiles{tx, ty, (n[2] + kz - 1) / kz, kz};
}

// A thread's place in its tile with a halo of H cells, and the halo cell that it brings. Positions past the end of
// an axis hold what its last cells see there (their halo); nothing past those is read by a cell of the grid.
template <int H, int FORM>
struct Place {
    static constexpr int NY = rows_of(FORM), TX = NY ? kFlatX : kTileX, PX = TX + 2 * H;
    static constexpr int cells = PX * (NY ? NY : kTileY + 2 * H);  // of a plane of the tile
    static_assert(NY || 2 * H * (kTileX + kTileY) <= threads_of(FORM), "one halo cell per thread");
    int i, j, k0, k1;
    int own, hcell;     // columns of the plane: the thread's, its halo cell's
    int at, hat;        // their places in the tile
    bool halo, beside;  // it brings a halo cell; one left or right of the tile (else below or above)
    bool inside, xl, xh, yl, yh;  // the column is one of the grid's; its faces exist
    int yo[2 * H];      // all rows in the tile: from `at` to the y neighbours -H .. -1, 1 .. H
    __device__ __forceinline__ Place(const HGeo& g, const HTiles& t) {
        const unsigned total = (unsigned)t.tx * t.ty * t.tz;
        unsigned L = blockIdx.x;
        if ((total & 7u) == 0) L = (L & 7u) * (total >> 3) + (L >> 3);
        const int x0 = (int)(L % (unsigned)t.tx) * TX, y0 = NY ? 0 : (int)((L / (unsigned)t.tx) % (unsigned)t.ty) * kTileY;
        k0 = (int)(L / ((unsigned)t.tx * t.ty)) * t.kz;
        k1 = min(k0 + t.kz, g.n[2]);
        const int tid = threadIdx.x, lx = tid % TX, ly = tid / TX, nx = g.n[0], ny = g.n[1];
        i = x0 + lx;
        j = y0 + ly;
        auto colx = [&](int q) { return reach(g, 0, min(q, nx + H - 1)); };
        auto coly = [&](int q) { return NY ? q : reach(g, 1, min(q, ny + H - 1)); };
        own = colx(i) + nx * coly(j);
        int hx = 0, hy = 0;
        if constexpr (NY) {
            beside = true;
            halo = lx < 2 * H;
            hx = lx < H ? lx - H : TX + lx - H;
            hy = ly;
            at = ly * PX + lx + H;
            hat = ly * PX + hx + H;
#pragma unroll
            for (int q = 0; q < 2 * H; ++q) yo[q] = NY > 1 ? (reach(g, 1, j + (q < H ? q - H : q - H + 1)) - j) * PX : 0;
        } else {
            beside = tid >= 2 * H * kTileX;
            halo = tid < 2 * H * (kTileX + kTileY);
            if (!beside) {
                const int r = tid / kTileX;
                hx = lx;
                hy = r < H ? r - H : kTileY + r - H;
            } else if (halo) {
                const int q = tid - 2 * H * kTileX, c = q % (2 * H);
                hx = c < H ? c - H : kTileX + c - H;
                hy = q / (2 * H);
            }
            hat = (hy + H) * PX + hx + H;
            at = (ly + H) * PX + lx + H;
        }
        hcell = colx(x0 + hx) + nx * coly(y0 + hy);
        inside = i < nx && j < ny;
        xl = g.per[0] || i > 0;
        xh = g.per[0] || i < nx - 1;
        yl = g.per[1] || j > 0;
        yh = g.per[1] || j < ny - 1;
    }
    // from `at` to the y neighbour d rows on
    __device__ __forceinline__ int y(int d) const { return NY ? yo[d < 0 ? d + H : d + H - 1] : d * PX; }
};

// What a cell of the rhs reads at its neighbours, one value of it per array; of the momentum mom_star the
// component of the axis at hand.
struct RhsCell {
    double p, rn, r1, ms, c, k;
};

// A face between cells a and b: the pressure there, the interface velocity and the flux of the two-component term.
// Where there is none: the cell's own pressure, zero.
struct RhsFace {
    double p, u, f;
};
template <bool TC>
__device__ __forceinline__ RhsFace rhs_face(bool face, const RhsCell& a, const RhsCell& b, double own, double ih) {
    return {face ? pbnd(a.p, a.rn, b.p, b.rn) : own, face ? (a.ms + b.ms) / (a.r1 + b.r1) : 0.0,
            TC && face ? 0.5 * (a.k + b.k) * (b.c - a.c) * ih : 0.0};
}

// The right-hand side by tiles (see k_advect): the arrays with neighbours in x and y go through LDS with one cell of
// halo, the next plane's own values and the halo are loaded a plane ahead, and the low z face of a cell is
// the high one of the plane before. Bound by memory: 375 us at 256^3 for 80 B read and 8 written per cell;
// 414 us with every neighbour from memory, the planes of 8 workgroups per CU thrashing the L2.
// TC: the two-component terms (temp_n, conc_n, rkc_n given); VISC: the viscous term (visc given).
template <bool TC, bool VISC, int FORM>
__global__ __launch_bounds__(threads_of(FORM), TC ? (VISC && rows_of(FORM) ? 2 : 3) : 4) void k_pressure_rhs(HGeo g, HTiles t, RhsArgs A) {
    using P = Place<1, FORM>;
    constexpr bool Z = FORM != FORM_PLANE;
    constexpr int NA = TC ? 7 : 5;  // p, rho_n, rho_np1, mom_star x and y, conc, rkc
    __shared__ double tile[2][NA][P::cells];
    const P o(g, t);
    const int nz = g.n[2];
    const int64_t sxy = (int64_t)g.n[0] * g.n[1];
    const double ih[3] = {1.0 / g.h[0], 1.0 / g.h[1], 1.0 / g.h[2]};
    struct Own {
        double p, rn, r1, m[3], c, k;  // m: mom_star
        double mn[3], c2, visc, temp;
    };
    auto load = [&](Own& v, int k) {
        const int64_t a = o.own + (int64_t)reach(g, 2, k) * sxy;
        v.p = A.p_n[a];
        v.rn = A.rho_n[a];
        v.r1 = A.rho_np1[a];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            v.m[d] = A.mom_star[(int64_t)d * A.N + a];
            v.mn[d] = A.mom_n[(int64_t)d * A.N + a];
        }
        v.c2 = A.c2_n[a];
        if (TC) {
            v.c = A.conc_n[a];
            v.k = A.rkc_n[a];
            v.temp = A.temp_n[a];
        }
        if (VISC) v.visc = A.visc[a];
    };
    RhsCell h;
    auto load_halo = [&](int k) {
        const int64_t a = o.hcell + (int64_t)k * sxy;
        h.p = A.p_n[a];
        h.rn = A.rho_n[a];
        h.r1 = A.rho_np1[a];
        h.ms = A.mom_star[(o.beside ? 0 : A.N) + a];
        if (TC) {
            h.c = A.conc_n[a];
            h.k = A.rkc_n[a];
        }
    };
    auto along = [&](const Own& v, int d) { return RhsCell{v.p, v.rn, v.r1, v.m[d], TC ? v.c : 0.0, TC ? v.k : 0.0}; };
    Own q0, q1, q2;
    if (Z) load(q2, o.k0 - 1);
    load(q0, o.k0);
    if (Z) load(q1, o.k0 + 1);
    if (o.halo) load_halo(o.k0);
    RhsFace zlo = rhs_face<TC>(Z && nz > 1 && (g.per[2] || o.k0 > 0), along(q2, 2), along(q0, 2), q0.p, ih[2]);
    // one plane from v, its own values, and w, the next one's; x then takes plane k + 2
    auto plane = [&](int k, const Own& v, const Own& w, Own& x) {
        double(*s)[P::cells] = tile[k & 1];
        const RhsCell mine = along(v, 0);
        s[0][o.at] = v.p;
        s[1][o.at] = v.rn;
        s[2][o.at] = v.r1;
        s[3][o.at] = v.m[0];
        s[4][o.at] = v.m[1];
        if (TC) {
            s[NA - 2][o.at] = v.c;
            s[NA - 1][o.at] = v.k;
        }
        if (o.halo) {
            s[0][o.hat] = h.p;
            s[1][o.hat] = h.rn;
            s[2][o.hat] = h.r1;
            s[o.beside ? 3 : 4][o.hat] = h.ms;
            if (TC) {
                s[NA - 2][o.hat] = h.c;
                s[NA - 1][o.hat] = h.k;
            }
        }
        __syncthreads();  // (the other slot's readers passed the previous plane's barrier)
        if (Z) load(x, min(k + 2, o.k1));
        if (Z && o.halo) load_halo(min(k + 1, o.k1 - 1));
        auto cell_at = [&](int d, int off) {
            const int q = o.at + off;
            return RhsCell{s[0][q], s[1][q], s[2][q], s[3 + d][q], TC ? s[NA - 2][q] : 0.0, TC ? s[NA - 1][q] : 0.0};
        };
        const double irn = 1.0 / v.rn;
        const double m = irn / v.c2;
        double adv = 0.0, divu = 0.0, dc = 0.0;
        auto axis = [&](const RhsFace& lo, const RhsFace& hi, int d) {
            adv += (v.mn[d] * irn) * ((hi.p - lo.p) * ih[d]);
            divu += (hi.u - lo.u) * ih[d];
            if (TC) dc += (hi.f - lo.f) * ih[d];
        };
        // (an axis of one cell has no faces: its lines contribute exact zeros)
        axis(rhs_face<TC>(o.xl, cell_at(0, -1), mine, v.p, ih[0]), rhs_face<TC>(o.xh, mine, cell_at(0, 1), v.p, ih[0]), 0);
        const RhsCell my = along(v, 1);
        axis(rhs_face<TC>(o.yl, cell_at(1, o.y(-1)), my, v.p, ih[1]), rhs_face<TC>(o.yh, my, cell_at(1, o.y(1)), v.p, ih[1]), 1);
        const RhsFace zhi = rhs_face<TC>(Z && nz > 1 && (g.per[2] || k < nz - 1), along(v, 2), along(w, 2), v.p, ih[2]);
        axis(zlo, zhi, 2);
        zlo = zhi;
        double b = m * (v.p - g.dt * adv) - g.dt * divu;
        if constexpr (VISC) b -= (2.0 * g.dt / 3.0) * (m * irn) * v.visc;
        if (TC) b -= (3.0 * g.dt / 4.0) * m * A.r_gas * v.temp * dc;
        if (o.inside) A.b[o.own + (int64_t)k * sxy] = b;
    };
    for (int k = o.k0; k < o.k1;) {
        plane(k, q0, q1, q2);
        if (++k == o.k1) break;
        plane(k, q1, q2, q0);
        if (++k == o.k1) break;
        plane(k, q2, q0, q1);
        ++k;
    }
}

struct UpdArgs {
    const double *p, *rho_np1, *mom_star, *e_star;
    double *mom_out, *uface_out, *e_out;
    int64_t N;
};

// What a cell of the update reads at its neighbours; of the momentum the component of the axis at hand.
struct UpdCell {
    double p, r, ms;
};

// A face between cells a and b (steps (vii)-(viii)): the pressure there with rho^{n+1}, and the interface
// velocity u^{n+1}. Where there is none: the cell's own pressure, zero.
struct UpdFace {
    double p, u;
};
__device__ __forceinline__ UpdFace upd_face(bool face, const UpdCell& a, const UpdCell& b, double own, double dt, double ih) {
    return {face ? pbnd(a.p, a.r, b.p, b.r) : own,
            face ? (a.ms + b.ms) / (a.r + b.r) - dt * (b.p - a.p) * ih * 2.0 / (b.r + a.r) : 0.0};
}

// The updates after the solve by tiles, as in k_pressure_rhs. Bound by memory: 396 us at 256^3 for 48 B read and 56
// written per cell; 472 us with every neighbour from memory.
template <int FORM>
__global__ __launch_bounds__(threads_of(FORM)) void k_pressure_update(HGeo g, HTiles t, UpdArgs A) {
    using P = Place<1, FORM>;
    constexpr bool Z = FORM != FORM_PLANE;
    __shared__ double tile[2][4][P::cells];  // p, rho, mom_star x and y
    const P o(g, t);
    const int nz = g.n[2];
    const int64_t sxy = (int64_t)g.n[0] * g.n[1];
    const double ih[3] = {1.0 / g.h[0], 1.0 / g.h[1], 1.0 / g.h[2]};
    struct Own {
        double p, r, m[3], e;
    };
    auto load = [&](Own& v, int k) {
        const int64_t a = o.own + (int64_t)reach(g, 2, k) * sxy;
        v.p = A.p[a];
        v.r = A.rho_np1[a];
#pragma unroll
        for (int d = 0; d < 3; ++d) v.m[d] = A.mom_star[(int64_t)d * A.N + a];
        v.e = A.e_star[a];
    };
    UpdCell h;
    auto load_halo = [&](int k) {
        const int64_t a = o.hcell + (int64_t)k * sxy;
        h = UpdCell{A.p[a], A.rho_np1[a], A.mom_star[(o.beside ? 0 : A.N) + a]};
    };
    auto along = [&](const Own& v, int d) { return UpdCell{v.p, v.r, v.m[d]}; };
    Own q0, q1, q2;
    if (Z) load(q2, o.k0 - 1);
    load(q0, o.k0);
    if (Z) load(q1, o.k0 + 1);
    if (o.halo) load_halo(o.k0);
    UpdFace zlo = upd_face(Z && nz > 1 && (g.per[2] || o.k0 > 0), along(q2, 2), along(q0, 2), q0.p, g.dt, ih[2]);
    auto plane = [&](int k, const Own& v, const Own& w, Own& x) {
        double(*s)[P::cells] = tile[k & 1];
        s[0][o.at] = v.p;
        s[1][o.at] = v.r;
        s[2][o.at] = v.m[0];
        s[3][o.at] = v.m[1];
        if (o.halo) {
            s[0][o.hat] = h.p;
            s[1][o.hat] = h.r;
            s[o.beside ? 2 : 3][o.hat] = h.ms;
        }
        __syncthreads();  // (the other slot's readers passed the previous plane's barrier)
        if (Z) load(x, min(k + 2, o.k1));
        if (Z && o.halo) load_halo(min(k + 1, o.k1 - 1));
        auto cell_at = [&](int d, int off) { return UpdCell{s[0][o.at + off], s[1][o.at + off], s[2 + d][o.at + off]}; };
        double gp[3], uf[3], divn = 0.0;
        auto axis = [&](const UpdFace& lo, const UpdFace& hi, int d) {
            uf[d] = hi.u;
            divn += (hi.u - lo.u) * ih[d];
            gp[d] = (hi.p - lo.p) * ih[d];
        };
        // (an axis of one cell has no faces and its terms are exact zeros)
        const UpdCell mx = along(v, 0), my = along(v, 1);
        axis(upd_face(o.xl, cell_at(0, -1), mx, v.p, g.dt, ih[0]), upd_face(o.xh, mx, cell_at(0, 1), v.p, g.dt, ih[0]), 0);
        axis(upd_face(o.yl, cell_at(1, o.y(-1)), my, v.p, g.dt, ih[1]),
             upd_face(o.yh, my, cell_at(1, o.y(1)), v.p, g.dt, ih[1]), 1);
        const UpdFace zhi = upd_face(Z && nz > 1 && (g.per[2] || k < nz - 1), along(v, 2), along(w, 2), v.p, g.dt, ih[2]);
        axis(zlo, zhi, 2);
        zlo = zhi;
        // step (vii): momentum; step (ix): e^{n+1} = e* - dt (P div u^{n+1} + u^{n+1} . grad P)
        const int64_t a = o.own + (int64_t)k * sxy;
        const double ir = 1.0 / v.r;
        double ug = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double md = v.m[d] - g.dt * gp[d];
            if (o.inside) {
                A.mom_out[(int64_t)d * A.N + a] = md;
                A.uface_out[(int64_t)d * A.N + a] = uf[d];
            }
            ug += (md * ir) * gp[d];
        }
        if (o.inside) A.e_out[a] = v.e - g.dt * (v.p * divn + ug);
    };
    for (int k = o.k0; k < o.k1;) {
        plane(k, q0, q1, q2);
        if (++k == o.k1) break;
        plane(k, q1, q2, q0);
        if (++k == o.k1) break;
        plane(k, q2, q0, q1);
        ++k;
    }
}

// ---- the explicit advective part (steps (i)-(iii)) and the equation of state ----

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

// q* = q - dt div(flux) for the five conserved fields (rho, three momenta, e), the fluxes through
// the interfaces of every cell from eq. step1 and the upwind reconstruction.
//
// A workgroup walks its tile of columns through kz planes. Each plane of the tile goes through LDS
// with two cells of halo on every side (own cells from registers, one halo cell per thread from
// memory), so the eight x and y neighbours of a field cost one load; the z neighbours stay in a
// ring of four planes, and the flux through a cell's low z interface is the one its lower
// neighbour computed. The next plane's loads are in flight while a plane is computed. Bound by
// memory: 380 us at 256^3 for 1.4 GB read (the halo rows come from beyond the L2 as often as not)
// and 0.67 GB written; one thread per cell, with every neighbour from memory and every flux
// twice, took 1041 us. Tiles of 512 threads left one workgroup per CU (510 us) or spilled.
template <int FORM>
__global__ __launch_bounds__(threads_of(FORM), 3) void k_advect(HGeo g, HTiles t, AdvArgs A) {
    using P = Place<2, FORM>;
    __shared__ double tile[2][5][P::cells];
    const P o(g, t);
    const int k0 = o.k0, k1 = o.k1, own = o.own, at = o.at, hat = o.hat, hcell = o.hcell, nz = g.n[2];
    const bool halo = o.halo, xl = o.xl, xh = o.xh, yl = o.yl, yh = o.yh, inside = o.inside;
    const int64_t sxy = (int64_t)g.n[0] * g.n[1];
    const double ih[3] = {1.0 / g.h[0], 1.0 / g.h[1], 1.0 / g.h[2]};

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
        double(*p)[P::cells] = tile[k & 1];
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            p[f][at] = v1[f];
            if (halo) p[f][hat] = hv[f];
        }
        __syncthreads();  // (the other slot's readers passed the previous plane's barrier)
        load(hv, hcell, min(k + 1, k1 - 1));
        // interface velocities; zero on an axis of one cell, whose fluxes then cancel to zero
        const double *r = p[0] + at, *mx = p[1] + at, *my = p[2] + at;
        const int yl1 = o.y(-1), yh1 = o.y(1), yl2 = o.y(-2), yh2 = o.y(2);
        const double uxl = step1(xl, mx[-1], v1[1], r[-1], v1[0]);
        const double uxh = step1(xh, v1[1], mx[1], v1[0], r[1]);
        const double uyl = step1(yl, my[yl1], v1[2], r[yl1], v1[0]);
        const double uyh = step1(yh, v1[2], my[yh1], v1[0], r[yh1]);
        const double uzh = step1(g.per[2] || k < nz - 1, v1[3], v2[3], v1[0], v2[0]);
        const int64_t a = own + (int64_t)k * sxy, an = own + (int64_t)reach(g, 2, min(k + 3, k1 + 1)) * sxy;
#pragma unroll
        for (int f = 0; f < 5; ++f) {
            const double* c = p[f] + at;
            double div = axis_div(uxl, uxh, c[-2], c[-1], v1[f], c[1], c[2]) * ih[0];
            div += axis_div(uyl, uyh, c[yl2], c[yl1], v1[f], c[yh1], c[yh2]) * ih[1];
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
    const HTiles t = htiles(n);
    with_form(n, [&](auto form) {
        constexpr int F = decltype(form)::value == FORM_PLANE ? FORM_BOX : decltype(form)::value;
        hipLaunchKernelGGL(k_advect<F>, dim3((unsigned)((int64_t)t.tx * t.ty * t.tz)), dim3(threads_of(F)), 0, s, g, t, A);
    });
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
    auto go = [&](auto tc, auto visc) {
        constexpr bool TC = decltype(tc)::value, VISC = decltype(visc)::value;
        with_form(n, [&](auto form) {
            constexpr int F = decltype(form)::value;
            hipLaunchKernelGGL((k_pressure_rhs<TC, VISC, F>), dim3((unsigned)t.tx * t.ty * t.tz), dim3(threads_of(F)), 0, s,
                               g, t, A);
        });
    };
    using Yes = std::true_type;
    using No = std::false_type;
    if (f->temp_n && f->visc) go(Yes{}, Yes{});
    else if (f->temp_n) go(Yes{}, No{});
    else if (f->visc) go(No{}, Yes{});
    else go(No{}, No{});
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
    with_form(n, [&](auto form) {
        constexpr int F = decltype(form)::value;
        hipLaunchKernelGGL(k_pressure_update<F>, dim3((unsigned)t.tx * t.ty * t.tz), dim3(threads_of(F)), 0, s, g, t, A);
    });
    return hipGetLastError() == hipSuccess ? HP_OK : HP_EHIP;
}

}  // namespace hp
