// hp_coarse.hip -- the coarsest multigrid level: its dense operator, assembled on the device, and
// the operator's inverse by blocked symmetric elimination.
//
// The coarsest level holds at most a few thousand cells, so the V-cycle solves it exactly with
// one dense matrix-vector product by the stored inverse. The operator is the same seven-point
// flux-form matrix as on every other level (paper, Section 2, eq. Poiss times dt^2 with the
// coefficients of eqs. cpoiss/kappapoiss and the face factor of step (viii)); it is symmetric
// positive definite when m > 0 and rho > 0, so elimination needs no pivoting and every pivot
// (a diagonal entry of a Schur complement) is positive.
//
// The unknowns are cut into blocks of at most kB, each within a layer of the grid along one axis (or a few thin
// layers). A step eliminates a set of blocks a that don't couple with each other, by the symmetric sweep: with D_a
// the inverse of the diagonal block that the steps before left, P_aJ = D_a A_aJ,
//     A_IJ <- A_IJ - sum_a A_Ia P_aJ,   A_aJ <- P_aJ,   A_Ia <- A_Ia D_a,   A_aa <- -D_a,
// and after the last step the array holds minus the inverse. A layer couples with its neighbours alone, so
// every other layer goes at once, then every other one of those left (of 8 layers 4, 2, 1, 1): 8 x 8 x 8 cells
// take 8 steps where one block after the other takes 16, 16 x 16 cells 4 instead of 8.
//
// The steps are a chain of launches, bound by latency: pivots one after the other, and what a launch costs. So
// a step is one launch, a workgroup per tile (I, J), I <= J: it updates its tile, and where that is the diagonal
// block of a pivot of the next step, inverts it at once (k_inverse_step). The products are matrix
// instructions, whose operand layout is that of the rows as they lie in memory, and by symmetry
// also that of the columns. A step takes 9 to 11 us, 6 of them the 32 pivots of the next. New coefficients
// took 225 us on 96 x 56 x 192 cells (504 coarsest ones) and 141 on 64 x 64 (256) when this came in, 475 and 265 with
// two launches per 32 pivots, swept one at a time through LDS (15 us), and every block on its own.
#include "hp_device.h"
#include "hp_internal.h"

#include <algorithm>
#include <cmath>

namespace hp {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kB = 32;    // widest block (a tile: kB x kB, padded with the identity)
constexpr int kTile = kB * kB;
constexpr int kSet = 8;   // most blocks eliminated in one step

// ---- plan (host) ----

// Layers of the grid along an axis, `group` of them taken together; the sets in which they are eliminated.
namespace {
struct Layers {
    int axis = 0;
    std::vector<int> first, size;       // of each: first layer, unknowns
    std::vector<std::vector<int>> sets;
    int steps = 0, blocks = 0;
    // us that the steps take: 10 each for what a step waits for, 3 per 1000 tiles (measured up to 28,680 tiles)
    double time() const { return steps * (10.0 + 0.003 * (0.5 * blocks * (blocks + 1))); }
};

Layers layers_along(const int n[3], const int per[3], int axis, int group) {
    Layers L;
    L.axis = axis;
    const int cells = n[0] * n[1] * n[2] / n[axis];
    for (int f = 0; f < n[axis]; f += group) {
        L.first.push_back(f);
        L.size.push_back(std::min(group, n[axis] - f) * cells);
        L.blocks += (L.size.back() + kB - 1) / kB;
    }
    std::vector<int> left(L.first.size());
    for (size_t q = 0; q < left.size(); ++q) left[q] = (int)q;
    while (!left.empty()) {
        std::vector<int> set, rest;
        for (size_t q = 0; q < left.size(); ++q) {
            // every other one; on a ring the last one is the first one's neighbour
            const bool next_to_first = per[axis] && q > 0 && q + 1 == left.size();
            if (q % 2 == 0 && !next_to_first && (int)set.size() < kSet) set.push_back(left[q]);
            else rest.push_back(left[q]);
        }
        int chunks = 0;
        for (int l : set) chunks = std::max(chunks, (L.size[l] + kB - 1) / kB);
        L.steps += chunks;
        L.sets.push_back(set);
        left = rest;
    }
    return L;
}

// Thin layers are taken together to at most kB unknowns, and the axis is the one of the fewest steps. Above 512 unknowns the
// tiles' number counts, too: where the layers don't fill their blocks (17 cells of 32), more of them taken together
// do, and the plan of the least time is taken. That bounds the workspace as well: 17 x 1 x 239 cells 28 steps, 96 MB and
// 1016 us instead of 32, 266 MB and 3035; it is never above 120 MB, and from 1600 unknowns on smaller than the
// inverse (132 MB there).
Layers choose_layers(const int n[3], const int per[3]) {
    const int unknowns = n[0] * n[1] * n[2];
    Layers best;
    for (int d = 2; d >= 0; --d) {
        const int cells = unknowns / n[d], thin = std::max(1, kB / cells);
        for (int group = thin; group == thin || (unknowns > 512 && group <= n[d] && group * cells <= 512); ++group) {
            Layers o = layers_along(n, per, d, group);
            if (best.sets.empty() || (unknowns > 512 ? o.time() < best.time() : o.steps < best.steps)) best = o;
        }
    }
    return best;
}
}  // namespace

InversePlan plan_inverse(const int n[3], const int per[3]) {
    InversePlan P;
    P.n = n[0] * n[1] * n[2];
    const Layers L = choose_layers(n, per);
    const int axis = L.axis;
    P.steps = L.steps;
    // blocks (size, step, slot) in the order of the layers, and their unknowns
    std::vector<int> blocks, perm, set_of(L.first.size()), slot_of(L.first.size()), step_of(L.sets.size());
    for (size_t s = 0, at = 0; s < L.sets.size(); ++s) {
        int chunks = 0;
        for (size_t q = 0; q < L.sets[s].size(); ++q) {
            set_of[L.sets[s][q]] = (int)s;
            slot_of[L.sets[s][q]] = (int)q;
            chunks = std::max(chunks, (L.size[L.sets[s][q]] + kB - 1) / kB);
        }
        step_of[s] = (int)at;
        at += chunks;
    }
    std::vector<int> sets((size_t)L.steps * kSet, -1);
    const int u = axis == 0 ? 1 : 0, v = axis == 2 ? 1 : 2;
    const int stride[3] = {1, n[0], n[0] * n[1]};
    for (size_t l = 0; l < L.first.size(); ++l) {
        const int chunks = (L.size[l] + kB - 1) / kB, width = (L.size[l] + chunks - 1) / chunks;
        const int layers = L.size[l] / (n[u] * n[v]);
        std::vector<int> cells;
        for (int k = L.first[l]; k < L.first[l] + layers; ++k)
            for (int j = 0; j < n[v]; ++j)
                for (int i = 0; i < n[u]; ++i) cells.push_back(k * stride[axis] + j * stride[v] + i * stride[u]);
        for (int c = 0; c < chunks; ++c) {
            const int step = step_of[set_of[l]] + c, id = (int)blocks.size() / 2;
            sets[(size_t)step * kSet + slot_of[l]] = id;
            blocks.push_back(step);
            blocks.push_back(slot_of[l]);
            for (int q = 0; q < kB; ++q)
                perm.push_back(q < width && c * width + q < L.size[l] ? cells[c * width + q] : -1);
        }
    }
    P.blocks = (int)blocks.size() / 2;
    P.tables = blocks;
    P.tables.insert(P.tables.end(), sets.begin(), sets.end());
    P.tables.insert(P.tables.end(), perm.begin(), perm.end());
    P.doubles = (int64_t)P.blocks * (P.blocks + 1) / 2 * kTile + 2 * kSet * (int64_t)(P.blocks + 1) * kTile;
    P.ints = (int64_t)P.tables.size() + 2 * kSet * (int64_t)P.blocks;
    return P;
}

// ---- device ----

namespace {

struct InverseArgs {
    const int* blocks;  // per block: its step, its slot in the step's set
    const int* sets;    // per step: kSet blocks (-1: none)
    const int* perm;    // per block: its kB unknowns (-1: padding)
    int* nonzero;       // [step parity][slot][block]: whether the panel's tile holds anything
    double* tiles;      // upper tiles (I, J), row-major: tile J (J + 1) / 2 + I
    double* panels;     // [step parity][slot][block]: row tiles of the step's pivots
    double* diag;       // [step parity][slot]: inverses of their diagonal blocks
    int nb, n, step;
    const double *rho, *m;
    int nx, ny, nz, px, py, pz;
    double cx, cy, cz;
    int face_rule;
    double* out;
    int* flag;
};

__device__ __forceinline__ f64x4 mfma(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// The operator's entries (a[e], b), natural indices (-1: none): a lane's part of a tile's quadrant. On a diagonal
// tile one of them may be a diagonal entry. Every load is issued before the first is waited for.
__device__ __forceinline__ f64x4 operator_entries(const InverseArgs& p, const int (&a)[4], int b, bool diagonal) {
    const int at = max(b, 0), row = at / p.nx, i = at - row * p.nx, k = row / p.ny, j = row - k * p.ny;
    const int sy = p.nx, sz = p.nx * p.ny;
    // the neighbours in the order x-, x+, y-, y+, z-, z+ (a diagonal entry sums their faces in that order)
    const int nb[6] = {i > 0 ? at - 1 : p.px ? at + (p.nx - 1) : -1,  i < p.nx - 1 ? at + 1 : p.px ? at - (p.nx - 1) : -1,
                       j > 0 ? at - sy : p.py ? at + (p.ny - 1) * sy : -1, j < p.ny - 1 ? at + sy : p.py ? at - (p.ny - 1) * sy : -1,
                       k > 0 ? at - sz : p.pz ? at + (p.nz - 1) * sz : -1, k < p.nz - 1 ? at + sz : p.pz ? at - (p.nz - 1) * sz : -1};
    const double cd[3] = {p.cx, p.cy, p.cz};
    const double rb = p.rho[at], mb = p.m[at];
    double ra[4], rn[6];
#pragma unroll
    for (int e = 0; e < 4; ++e) ra[e] = p.rho[max(a[e], 0)];
    if (diagonal)
#pragma unroll
        for (int f = 0; f < 6; ++f) rn[f] = p.rho[nb[f] >= 0 ? nb[f] : at];
    auto kappa = [&](double x, double y) { return p.face_rule == 1 ? 0.5 * (1.0 / x + 1.0 / y) : 2.0 / (x + y); };
    double own = mb;
    if (diagonal)
#pragma unroll
        for (int f = 0; f < 6; ++f)
            if (nb[f] >= 0) own += cd[f >> 1] * kappa(rb, rn[f]);
    f64x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        double w = 0.0;
#pragma unroll
        for (int f = 0; f < 6; ++f)
            if (a[e] == nb[f]) w -= cd[f >> 1];
        if (w != 0.0) w *= kappa(ra[e], rb);
        v[e] = a[e] < 0 || b < 0 ? 0.0 : a[e] == b ? own : w;
    }
    return v;
}

// Minus the inverse of a 32 x 32 matrix held by a wave as four 16 x 16 results of the matrix instruction (lane l, value
// i: row l / 16 + 4 i, column l % 16), by symmetric sweeps of four pivots. Rows 4 q .. 4 q + 3 of a tile are then value q
// of every lane, in the layout of the instruction's right operand, and by symmetry columns 4 q .. in that of its
// left operand: nothing moves between lanes but the 4 x 4 pivot block. Returns whether every pivot is positive
// and finite.
__device__ __forceinline__ bool sweep_32(f64x4 (&v)[2][2]) {
    const int lane = threadIdx.x & 63, k = lane >> 4, j = lane & 3;
    const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
    bool good = true;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int tq = q >> 2, rq = q & 3;
        const double row[2] = {v[tq][0][rq], v[tq][1][rq]}, src = row[tq];
        auto at = [&](int r, int c) { return of_lane(src, 4 * rq + c + 16 * r); };
        const double a00 = at(0, 0), a01 = at(0, 1), a02 = at(0, 2), a03 = at(0, 3), a11 = at(1, 1), a12 = at(1, 2),
                     a13 = at(1, 3), a22 = at(2, 2), a23 = at(2, 3), a33 = at(3, 3);
        // the inverse of [X Y; Y^T Z], 2 x 2 each, by X's inverse and that of S = Z - Y^T X^-1 Y
        // (of a pivot that is zero or not finite the reciprocal is not finite; the flag is taken from the pivot itself)
        const double det = a00 * a11 - a01 * a01, rd = fast_rcp(det);
        const double x00 = a11 * rd, x01 = -a01 * rd, x11 = a00 * rd;
        const double w00 = x00 * a02 + x01 * a12, w01 = x00 * a03 + x01 * a13;  // W = X^-1 Y
        const double w10 = x01 * a02 + x11 * a12, w11 = x01 * a03 + x11 * a13;
        const double s00 = a22 - (a02 * w00 + a12 * w10), s01 = a23 - (a02 * w01 + a12 * w11),
                     s11 = a33 - (a03 * w01 + a13 * w11);
        const double dets = s00 * s11 - s01 * s01, rs = fast_rcp(dets);
        const double d22 = s11 * rs, d23 = -s01 * rs, d33 = s00 * rs;
        const double d02 = -(w00 * d22 + w01 * d23), d03 = -(w00 * d23 + w01 * d33);
        const double d12 = -(w10 * d22 + w11 * d23), d13 = -(w10 * d23 + w11 * d33);
        const double d00 = x00 - (d02 * w00 + d03 * w01), d01 = x01 - (d02 * w10 + d03 * w11),
                     d11 = x11 - (d12 * w10 + d13 * w11);
        good = good && a00 > 0.0 && a00 < INFINITY && det > 0.0 && det < INFINITY && s00 > 0.0 && s00 < INFINITY &&
               dets > 0.0 && dets < INFINITY;
        // entry (lane % 4, lane / 16) of the inverse
        auto pick = [](int e, double a, double b, double c, double d) { return e & 2 ? (e & 1 ? d : c) : (e & 1 ? b : a); };
        const double inv = pick(j, pick(k, d00, d01, d02, d03), pick(k, d01, d11, d12, d13), pick(k, d02, d12, d22, d23),
                                pick(k, d03, d13, d23, d33));
        const double prow[2] = {mfma(inv, row[0], zero)[0], mfma(inv, row[1], zero)[0]};
        // the lanes that hold the pivots' own columns (of tile column tq): these become A_iK D
        const bool own = ((lane & 15) >> 2) == rq;
#pragma unroll
        for (int tj = 0; tj < 2; ++tj) {
            const bool mine = own && tj == tq;
            const double b = mine ? inv : -prow[tj];
#pragma unroll
            for (int ti = 0; ti < 2; ++ti) {
                f64x4 c = v[ti][tj];
                if (tj == tq)
#pragma unroll
                    for (int e = 0; e < 4; ++e) c[e] = own ? 0.0 : c[e];
                v[ti][tj] = mfma(row[ti], b, c);
            }
            v[tq][tj][rq] = mine ? -inv : prow[tj];
        }
    }
    return good;
}

enum { STEP_FIRST, STEP_INNER, STEP_LAST };

// One step on one tile, a wave per 16 x 16 quadrant; its pivots' row tiles and inverted diagonal blocks are there from the
// launch before (STEP_FIRST: no pivots, the tile is assembled), and those of the next step are left for the
// next launch. No workgroup reads what another one writes in the same launch. STEP_LAST writes the inverse.
template <int MODE>
__global__ __launch_bounds__(256) void k_inverse_step(InverseArgs p) {
    __shared__ double lds[2][8][2][64];  // -P of a pivot, by rows of four and column half; at the end the tile
    const int t = blockIdx.x;
    int J = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while ((J + 1) * (J + 2) / 2 <= t) ++J;
    while (J * (J + 1) / 2 > t) --J;
    const int I = t - J * (J + 1) / 2;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, qi = wave >> 1, qj = wave & 1;
    const int k = lane >> 4, c = lane & 15;
    const int here = p.step & 1, then = here ^ 1, next = p.step + 1;
    const int step_i = p.blocks[2 * I], slot_i = p.blocks[2 * I + 1], step_j = p.blocks[2 * J], slot_j = p.blocks[2 * J + 1];
    double* const tile = p.tiles + (int64_t)t * kTile + (16 * qi + k) * kB + 16 * qj + c;
    f64x4 acc;
    if constexpr (MODE == STEP_FIRST) {
        const int b = p.perm[J * kB + 16 * qj + c];
        int a[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = p.perm[I * kB + 16 * qi + k + 4 * e];
        acc = operator_entries(p, a, b, I == J);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (I == J && a[e] < 0 && 16 * qi + k + 4 * e == 16 * qj + c) acc[e] = 1.0;  // padding
    } else {
        int in[kSet], full[kSet];  // the step's pivots, and whether both tiles of the product hold anything
#pragma unroll
        for (int a = 0; a < kSet; ++a) {
            in[a] = p.sets[p.step * kSet + a];
            const int* const nz = p.nonzero + (here * kSet + a) * p.nb;
            full[a] = nz[I] & nz[J];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = tile[4 * e * kB];
        const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
        // rows 4 i .. of a tile, columns of this lane's half
        auto rows = [&](const double* tile, int half, int i) { return tile[(4 * i + k) * kB + 16 * half + c]; };
        auto panel = [&](int a, int block) { return p.panels + ((int64_t)(here * kSet + a) * p.nb + block) * kTile; };
        auto diag = [&](int a) { return p.diag + (here * kSet + a) * kTile; };
        // A^T B (the first by its columns), quadrant (half_a, half_b)
        auto product = [&](const double* A, int half_a, const double* B, int half_b) {
            double x[8], y[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                x[i] = rows(A, half_a, i);
                y[i] = rows(B, half_b, i);
            }
            f64x4 s = zero;
#pragma unroll
            for (int i = 0; i < 8; ++i) s = mfma(x[i], y[i], s);
            return s;
        };
        const bool pi = step_i == p.step, pj = step_j == p.step;
        if (pi && pj) {
            // (two pivots of a step don't couple: that tile stays zero)
            if (I == J)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] = -diag(slot_i)[(16 * qi + k + 4 * e) * kB + 16 * qj + c];
        } else if (pi) {
            acc = product(diag(slot_i), qi, panel(slot_i, J), qj);
        } else if (pj) {
            acc = product(panel(slot_j, I), qi, diag(slot_j), qj);
        } else {
            int turn = 0;
#pragma unroll
            for (int a = 0; a < kSet; ++a) {
                if (in[a] < 0 || !full[a]) continue;
                // this wave's rows of P, then the product with all of them
                const f64x4 s = product(diag(a), qi, panel(a, J), qj);
#pragma unroll
                for (int e = 0; e < 4; ++e) lds[turn][4 * qi + e][qj][lane] = -s[e];
                double x[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = rows(panel(a, I), qi, i);
                __syncthreads();
#pragma unroll
                for (int i = 0; i < 8; ++i) acc = mfma(x[i], lds[turn][i][qj][lane], acc);
                turn ^= 1;
            }
        }
    }
    if constexpr (MODE == STEP_LAST) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // (the lower half of a diagonal tile is left out: the inverse is exactly symmetric)
            const int row = 16 * qi + k + 4 * e, col = 16 * qj + c, a = p.perm[I * kB + row], b = p.perm[J * kB + col];
            if (a < 0 || b < 0 || (I == J && row > col)) continue;
            p.out[(int64_t)a * p.n + b] = -acc[e];
            p.out[(int64_t)b * p.n + a] = -acc[e];
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) tile[4 * e * kB] = acc[e];
    const bool ni = step_i == next, nj = step_j == next;
    if (!ni && !nj) return;
    const int any = __syncthreads_or(acc[0] != 0.0 || acc[1] != 0.0 || acc[2] != 0.0 || acc[3] != 0.0);
    auto leave = [&](int slot, int block, bool turned) {
        double* const to = p.panels + ((int64_t)(then * kSet + slot) * p.nb + block) * kTile;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 16 * qi + k + 4 * e, col = 16 * qj + c;
            to[turned ? col * kB + row : row * kB + col] = acc[e];
        }
        if (threadIdx.x == 0) p.nonzero[(then * kSet + slot) * p.nb + block] = any;
    };
    if (I != J) {
        if (ni) leave(slot_i, J, false);
        if (nj) leave(slot_j, I, true);
        return;
    }
    // the next step's pivot block: its inverse, by the first wave
    double* const own = &lds[0][0][0][0];
#pragma unroll
    for (int e = 0; e < 4; ++e) own[(wave * 4 + e) * 64 + lane] = acc[e];
    __syncthreads();
    if (wave) return;
    f64x4 v[2][2];
    auto take = [&] {
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[w >> 1][w & 1][e] = own[(w * 4 + e) * 64 + lane];
    };
    take();
    // Where the diagonal holds values beyond 2^+-256, rows and columns are divided by powers of two near its square
    // roots, before the sweep and after it: the sweep's 2 x 2 determinants would leave the range otherwise. (As the
    // factors are powers of two, no other bit would change; always doing it cost 0.4 us a step. The loops are rolled up:
    // beside a pass over memory longer code took 2 us a step to fetch.)
    __shared__ int half[kB];
    const int r = lane & 31, q = r & 15, diagonal = ((r >> 4) * 12 + (q >> 2)) * 64 + 16 * (q & 3) + q;  // entry (r, r)
    const int mine = ((int)(((const unsigned*)own)[2 * diagonal + 1] >> 20 & 0x7ffu) - 1023) >> 1;
    const bool far = __any(abs(mine) > 128);
    auto down = [&](int e) { return -(half[16 * (e >> 3) + k + 4 * (e & 3)] + half[16 * (e >> 2 & 1) + c]); };
    if (far) {
        half[r] = mine;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll 1
        for (int e = 0; e < 16; ++e) own[e * 64 + lane] = __builtin_ldexp(own[e * 64 + lane], down(e));
        take();
    }
    if (!sweep_32(v) && lane == 0) *p.flag = 1;
    double* const to = p.diag + (then * kSet + slot_i) * kTile;
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int e = 0; e < 4; ++e) to[(16 * (w >> 1) + k + 4 * e) * kB + 16 * (w & 1) + c] = -v[w >> 1][w & 1][e];
    if (far) {
#pragma unroll 1
        for (int e = 0; e < 16; ++e) {
            double* const x = to + (16 * (e >> 3) + k + 4 * (e & 3)) * kB + 16 * (e >> 2 & 1) + c;
            *x = __builtin_ldexp(*x, down(e));
        }
    }
}

}  // namespace

void launch_coarse_inverse(const InversePlan& P, double* work, int* tables, const double* rho, const double* m,
                           const int n[3], const int per[3], const double cd[3], int face_rule, double* out, int* flag,
                           hipStream_t s) {
    const int64_t tiles = (int64_t)P.blocks * (P.blocks + 1) / 2;
    InverseArgs a{};
    a.blocks = tables;
    a.sets = a.blocks + 2 * P.blocks;
    a.perm = a.sets + P.steps * kSet;
    a.nonzero = tables + P.tables.size();
    a.tiles = work;
    a.panels = a.tiles + tiles * kTile;
    a.diag = a.panels + 2 * kSet * (int64_t)P.blocks * kTile;
    a.nb = P.blocks;
    a.n = P.n;
    a.step = -1;
    a.rho = rho;
    a.m = m;
    a.nx = n[0];
    a.ny = n[1];
    a.nz = n[2];
    a.px = per[0] && n[0] > 1;  // one cell has no wrap face
    a.py = per[1] && n[1] > 1;
    a.pz = per[2] && n[2] > 1;
    a.cx = cd[0];
    a.cy = cd[1];
    a.cz = cd[2];
    a.face_rule = face_rule;
    a.out = out;
    a.flag = flag;
    const dim3 grid((unsigned)tiles), block(256);
    hipLaunchKernelGGL(k_inverse_step<STEP_FIRST>, grid, block, 0, s, a);
    for (a.step = 0; a.step + 1 < P.steps; ++a.step) hipLaunchKernelGGL(k_inverse_step<STEP_INNER>, grid, block, 0, s, a);
    hipLaunchKernelGGL(k_inverse_step<STEP_LAST>, grid, block, 0, s, a);
}

}  // namespace hp
