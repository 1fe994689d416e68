// hp_small.hip -- V-cycles of small levels, and whole CG solves of small grids, in one launch.
//
// On a level of a few thousand cells a kernel takes 2.5-5 us whatever it does: its launch, its first
// loads, the write-back at its end; and a V-cycle runs six of them per level. Here one workgroup of
// 512 threads holds such a level and all below it: the vectors that neighbours read lie in LDS, what
// only the cell itself needs (weights, diagonal, residual, q) in registers of the thread that owns
// it, and a phase ends with a workgroup barrier. A half sweep of 4096 cells takes about half a
// microsecond so, bound by the six LDS reads per cell.
//
// The coarsest solve, a product with a dense inverse of up to 2 MB (or more, where odd sizes stop the
// coarsening), is more than one CU should stream. Helper workgroups of the same launch share it: every
// workgroup registers as it starts; the first is the owner and waits a bounded time for the others, then
// closes the registration, and those that come later leave at once. Nothing ever waits for a
// workgroup that has not started, so a launch makes progress whatever else occupies the GPU, and no
// value depends on how many helpers came. The right-hand side and the solution pass between the
// workgroups as relaxed agent-scope atomics: such a store goes through to the memory that all XCDs see,
// such a load takes no stale line from a cache of the CU or the XCD; each wave waits for its own stores
// (vmcnt 0) before its workgroup adds to the counter that the others poll, so the barrier needs no
// cache write-back or invalidation (1.0 us against 2 with agent-scope fences).
//
// A persistent team of up to 256 workgroups over whole levels was measured too: 3.3 us per phase
// with 16 workgroups and 5-7 with 256, no better than the launches it replaced.
#include "hp_device.h"
#include "hp_internal.h"
#include "hp_small.h"

#include <algorithm>
#include <cmath>

namespace hp {

namespace {

constexpr int kTT = kSmallThreads;
constexpr int kTW = kTT / 64;            // waves per workgroup
constexpr int kJoinPolls = 64;           // how long the owner waits for helpers

template <typename T>
__device__ __forceinline__ T ld(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum over a wave, the same in every lane: within rows of 16 by register permutes, then the four
// rows' sums (the cross-lane shuffle through LDS takes six times as long)
template <int CTRL>
__device__ __forceinline__ double permuted(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0u, (unsigned)u, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0u, (unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double wave_total(double v) {
    v += permuted<0xB1>(v);   // lanes 1 0 3 2 of each four
    v += permuted<0x4E>(v);   // lanes 2 3 0 1
    v += permuted<0x141>(v);  // the eight of a half row, mirrored
    v += permuted<0x140>(v);  // the row, mirrored
    return (of_lane(v, 0) + of_lane(v, 16)) + (of_lane(v, 32) + of_lane(v, 48));
}

struct Member {
    SmallState* t;
    int rank, size;      // of this workgroup among those of the launch, and how many there are
    unsigned target;     // what the counter reaches at the next barrier
    int polls;           // at most so many a barrier
    int lost;            // a barrier ran out of them

    // every member's stores before the barrier are visible to every member's loads after it
    __device__ __forceinline__ void barrier() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (size > 1 && !lost) {
            __shared__ int ok;
            if (threadIdx.x == 0) {
                target += size;
                __hip_atomic_fetch_add(&t->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                int n = 0;
                while ((int)(ld(&t->arrived) - target) < 0 && ++n < polls) {}
                ok = n < polls;
            }
            __syncthreads();
            lost |= !ok;
        }
    }
};

// Sum over the workgroup, the same in every thread; sums is an LDS array of kTW (free again after the
// next workgroup barrier).
__device__ __forceinline__ double group_total(double v, double* sums) {
    v = wave_total(v);
    if ((threadIdx.x & 63) == 0) sums[threadIdx.x >> 6] = v;
    __syncthreads();
    static_assert(kTW == 8, "half a row of lanes");
    double s = sums[threadIdx.x & 7];
    s += permuted<0xB1>(s);
    s += permuted<0x4E>(s);
    s += permuted<0x141>(s);
    return of_lane(s, 0);
}

// ---- one cell of a level ----

// h / d for 0 <= h < 2^22 with inv = 1 / d rounded: (h + 1/2) / d is at least 1 / (2 d) away from an
// integer, and the product's error is below that
__device__ __forceinline__ int quotient(int h, float inv) { return (int)(((float)h + 0.5f) * inv); }

// A cell's storage position (natural or red-black split order) and its neighbours', x-, x+, y-, y+,
// z-, z+. Behind a face that does not exist stands the cell itself.
struct Cell {
    int i, j, k, a;
    int at[6];
    bool lo[3];  // whether the low faces exist
    // item h of colour c: x pairs, fastest in x (i may fall outside an odd axis)
    __device__ __forceinline__ Cell(const SmallLevel& L, int h, int c) {
        const int row = quotient(h, L.inv_hx);
        k = quotient(row, L.inv_ny);
        j = row - k * L.g.ny;
        const int t = h - row * L.hx, par = (c + j + k) & 1;
        i = 2 * t + par;
        a = row * L.g.nx + (L.g.split ? c * L.hx + t : i);
    }
    __device__ __forceinline__ void look_round(const SmallLevel& L) {
        const Geo<double>& g = L.g;
        // the cell (split order: its x partner, of the other colour) from which the others are offsets
        const int o = g.split ? a + ((i + j + k) & 1 ? -L.hx : L.hx) : a;
        const int xl = g.split ? (i & 1) - 1 : -1, xu = g.split ? (i & 1) : 1;
        const int xw = (g.split ? L.hx : g.nx) - 1;  // from one end of a row to the other
        const int sy = g.nx, sz = g.nx * g.ny;
        lo[0] = i > 0 || g.px;
        lo[1] = j > 0 || g.py;
        lo[2] = k > 0 || g.pz;
        at[0] = i > 0 ? o + xl : g.px ? o + xw : a;
        at[1] = i < g.nx - 1 ? o + xu : g.px ? o - xw : a;
        at[2] = j > 0 ? o - sy : g.py ? o + (g.ny - 1) * sy : a;
        at[3] = j < g.ny - 1 ? o + sy : g.py ? o - (g.ny - 1) * sy : a;
        at[4] = k > 0 ? o - sz : g.pz ? o + (g.nz - 1) * sz : a;
        at[5] = k < g.nz - 1 ? o + sz : g.pz ? o - (g.nz - 1) * sz : a;
    }
    // face weights: the high faces' stand at the cell, the low faces' at the neighbour below
    __device__ __forceinline__ void weights(const SmallLevel& L, double* w) const {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double* wd = L.w + (int64_t)d * L.n;
            const double v = wd[at[2 * d]];
            w[2 * d + 1] = wd[a];
            w[2 * d] = lo[d] ? v : 0.0;
        }
    }
};

// f(cell, colour) for the cells of colour c of a level
template <typename F>
__device__ __forceinline__ void for_cells(const SmallLevel& L, int c, F&& f) {
    for (int h = threadIdx.x; h < L.items; h += kTT) {
        Cell e(L, h, c);
        if (e.i < L.g.nx) f(e);
    }
}

// storage position from a cell's row (its first position), x index and colour
__device__ __forceinline__ int in_row(const SmallLevel& L, int row, int i, int c) {
    return row + (L.g.split ? c * L.hx + (i >> 1) : i);
}

// rc = R t on the next level, reading the red cells only
__device__ __forceinline__ void restrict_red(const SmallLevel& L, const SmallLevel& C, const double* t, double* rc) {
    const bool fx = L.coarsened[0];
    for (int h = threadIdx.x; h < C.n; h += kTT) {
        const int row = quotient(h, C.inv_nx), I = h - row * C.g.nx, K = quotient(row, C.inv_ny), J = row - K * C.g.ny;
        int ix[4], iy[4], iz[4];
        float wx[4], wy[4], wz[4];
        restrict_taps(I, L.g.nx, fx, L.periodic[0], ix, wx);
        restrict_taps(J, L.g.ny, L.coarsened[1], L.periodic[1], iy, wy);
        restrict_taps(K, L.g.nz, L.coarsened[2], L.periodic[2], iz, wz);
        // Of the four taps in x of a row two are red: 1 and 3 (even i) or 0 and 2 (odd i). A tap that
        // does not exist has weight 0 and reads the parent's child of the same colour; on an axis
        // that is not coarsened the one tap counts where it is red.
        // (scalars: as arrays their choice by parity is an index, and they end up in memory)
        auto weight = [&](int o, int q) { return fx ? wx[2 * q + 1 - o] : (q == 0 && (I & 1) == o ? 1.0f : 0.0f); };
        auto place = [&](int o, int q, float w) {
            const int i = fx ? (w != 0.0f ? ix[2 * q + 1 - o] : 2 * I + o) : (I & ~1) + o;
            return in_row(L, 0, min(i, L.g.nx - 1), 0);
        };
        const float we0 = weight(0, 0), we1 = weight(0, 1), wo0 = weight(1, 0), wo1 = weight(1, 1);
        const int pe0 = place(0, 0, we0), pe1 = place(0, 1, we1), po0 = place(1, 0, wo0), po1 = place(1, 1, wo1);
        double acc = 0.0;
#pragma unroll 1
        for (int c = 0; c < (L.coarsened[2] ? 4 : 1); ++c) {  // (rolled up: unrolled its values spill the cells' registers)
            const int zc = c == 0 ? iz[0] : c == 1 ? iz[1] : c == 2 ? iz[2] : iz[3];
            const float wc = c == 0 ? wz[0] : c == 1 ? wz[1] : c == 2 ? wz[2] : wz[3];
            auto row_sum = [&](int yb) {
                const bool odd = (yb + zc) & 1;
                const double* line = t + (yb + L.g.ny * zc) * L.g.nx;
                const double v0 = line[odd ? po0 : pe0], v1 = line[odd ? po1 : pe1];
                const float w0 = odd ? wo0 : we0, w1 = odd ? wo1 : we1;
                // (a weight of 0 may stand on a position that holds no residual)
                return (w0 != 0.0f ? w0 * v0 : 0.0) + (w1 != 0.0f ? w1 * v1 : 0.0);
            };
            double accy = wy[0] * row_sum(iy[0]);
            if (L.coarsened[1]) accy += wy[1] * row_sum(iy[1]) + wy[2] * row_sum(iy[2]) + wy[3] * row_sum(iy[3]);
            acc += wc * accy;
        }
        rc[in_row(C, row * C.g.nx, I, (I + J + K) & 1)] = acc;
    }
}

// z += P e on red cells (the black half sweep that follows overwrites the black ones)
__device__ __forceinline__ void prolong_red(const SmallLevel& L, const SmallLevel& C, const double* ec, double* z) {
    for_cells(L, 0, [&](Cell& e) {
        int ix[2], iy[2], iz[2];
        float wx[2], wy[2], wz[2];
        prolong_taps(e.i, C.g.nx, L.coarsened[0], L.periodic[0], ix, wx);
        prolong_taps(e.j, C.g.ny, L.coarsened[1], L.periodic[1], iy, wy);
        prolong_taps(e.k, C.g.nz, L.coarsened[2], L.periodic[2], iz, wz);
        // the x sum of one coarse row
        auto row_sum = [&](int yb, int zc) {
            const int row = (yb + C.g.ny * zc) * C.g.nx;
            return wx[0] * ec[in_row(C, row, ix[0], (ix[0] + yb + zc) & 1)] +
                   wx[1] * ec[in_row(C, row, ix[1], (ix[1] + yb + zc) & 1)];
        };
        auto plane_sum = [&](int zc) {
            double s = wy[0] * row_sum(iy[0], zc);
            if (L.coarsened[1]) s += wy[1] * row_sum(iy[1], zc);
            return s;
        };
        double acc = wz[0] * plane_sum(iz[0]);
        if (L.coarsened[2]) acc += wz[1] * plane_sum(iz[1]);
        z[e.a] += acc;
    });
}

// 512 columns from c0 of two rows of the coarsest inverse, held by a wave (zero past the last)
struct Rows {
    double v[2][8];
    __device__ __forceinline__ void load(const double* ainv, int nc, int row, int c0) {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int c = c0 + lane + 64 * u;
                const double x = ainv[(int64_t)min(row + q, nc - 1) * nc + min(c, nc - 1)];
                v[q][u] = c < nc ? x : 0.0;
            }
    }
};

// Rows 2 (W rank + w), .. of z = A_c^-1 b by the W waves of each of `size` workgroups, two rows a
// wave at a time; b(c) and put(row, value). HELD: the first two rows' first columns are in `held`.
template <bool HELD, typename B, typename P>
__device__ __forceinline__ void coarse_rows(const double* ainv, int nc, int rank, int size, const Rows& held, B&& b, P&& put) {
    const int lane = threadIdx.x & 63;
    const int first = 2 * (rank * kTW + (int)(threadIdx.x >> 6)), step = 2 * size * kTW;
    auto add = [&](const Rows& r, int c0, double* acc) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int c = c0 + lane + 64 * u;
            const double x = b(min(c, nc - 1));
            acc[0] += r.v[0][u] * x;
            acc[1] += r.v[1][u] * x;
        }
    };
    for (int row = first; row < nc; row += step) {
        double acc[2] = {0.0, 0.0};
        const bool have = HELD && row == first;
        if (have) add(held, 0, acc);
        for (int c0 = have ? 512 : 0; c0 < nc; c0 += 512) {
            Rows r;
            r.load(ainv, nc, row, c0);
            add(r, c0, acc);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const double s = wave_total(acc[q]);
            if (lane == 0 && row + q < nc) put(row + q, s);
        }
    }
}

// memory that no kernel writes while this one runs: read through the scalar cache
typedef __attribute__((address_space(4))) const char* constant_t;

// natural-order position of a cell from its storage position
__device__ __forceinline__ int natural(const SmallLevel& L, int a) {
    if (!L.g.split) return a;
    const int row = quotient(a, L.inv_nx), k = quotient(row, L.inv_ny), j = row - k * L.g.ny;
    const int s = a - row * L.g.nx, c = s >= L.hx;
    return row * L.g.nx + 2 * (s - c * L.hx) + ((c + j + k) & 1);
}

// The owner's program: one V-cycle on the args' first level, or (CG) a whole solve: input checks, the first
// residual, the iterations, the true residual and further rounds from it. U: items of each colour per thread
// on that level.
template <int U, bool CG>
__device__ __forceinline__ void own(Member& me, const SmallArgs& args, double* lds, double* sums) {
    const SmallTable* A = (const SmallTable*)(constant_t)args.table;
    const int last = A->levels - 1, nu_pre = args.nu_pre, nu_post = args.nu_post;
    const SmallCG& C = args.cg;
    const SmallLevel L0 = A->lv[0];
    const int nc = A->nc;
    // LDS: p and q (CG), then z and t of the first level, then r, z and t of the others (the coarsest has
    // no t)
    double* const p0 = lds;
    double* const q0 = lds + L0.n;
    double* const z0 = CG ? lds + 2 * L0.n : lds;
    double* const t0 = z0 + L0.n;
    double* const below = t0 + L0.n;
    auto level_r = [&](const SmallLevel& L) { return below + L.lds; };

    // own cells of the first level: position, neighbours (two 16-bit positions to a word), weights,
    // 1 / diagonal, residual
    struct Own {
        int a;
        unsigned at[3];
        double w[6], dinv, r;
        // (the empty asm keeps what is derived from the packed positions inside the iteration: the
        // compiler hoists every unpacked address out of it otherwise, and spills)
        __device__ __forceinline__ int self() const {
            int v = a;
            asm volatile("" : "+v"(v));
            return v;
        }
        // sum of w (v[neighbour] - c)
        __device__ __forceinline__ double gather(const double* v, double c) const {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                unsigned p = at[q];
                asm volatile("" : "+v"(p));
                s += w[2 * q] * (v[p & 0xffffu] - c);
                s += w[2 * q + 1] * (v[p >> 16] - c);
            }
            return s;
        }
    };
    Own e[2][U];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            Own& o = e[c][u];
            const int h = (int)threadIdx.x + kTT * u;
            Cell cell(L0, min(h, L0.items - 1), c);
            const bool in = h < L0.items && cell.i < L0.g.nx;
            if (cell.i >= L0.g.nx) cell = Cell(L0, 0, 0);
            cell.look_round(L0);
            o.a = in ? cell.a : -1;
#pragma unroll
            for (int q = 0; q < 3; ++q) o.at[q] = (unsigned)cell.at[2 * q] | (unsigned)cell.at[2 * q + 1] << 16;
            cell.weights(L0, o.w);
            o.dinv = L0.dinv[cell.a];
            o.r = CG ? 0.0 : args.r[cell.a];
        }
    // f(own cell) for the cells of colour c
    auto mine = [&](int c, auto&& f) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (e[c][u].a >= 0) f(e[c][u]);
    };
    auto sweep0 = [&](int c) {
        mine(c, [&](Own& o) { z0[o.self()] = (o.r + o.gather(z0, 0.0)) * o.dinv; });
        __syncthreads();
    };

    int it = 0, code = SMALL_MORE, rounds = 0;
    double rz = 0.0, rr = 0.0, alpha = 0.0, beta = 0.0, bb = 0.0, target = 0.0;
    // r = b - A x with ||r||^2, x through p's place in LDS; with_b: also ||b||^2, and whether an entry of
    // either is not finite
    auto true_residual = [&](bool with_b, bool& finite) {
        double v = 0.0, vb = 0.0, bad = 0.0;
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 2; ++c)
            mine(c, [&](Own& o) {
                const int a = o.self();
                p0[a] = C.x[natural(L0, a)];
            });
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 2; ++c)
            mine(c, [&](Own& o) {
                const int a = o.self();
                const double x = p0[a], b = C.b[natural(L0, a)];
                o.r = b - (L0.m[a] * x - o.gather(p0, x));
                v += o.r * o.r;
                vb += b * b;
                if (!(b - b == 0.0) || !(x - x == 0.0)) bad = 1.0;
            });
        const double s = group_total(v, sums);
        if (with_b) {
            __syncthreads();
            bb = group_total(vb, sums);
            __syncthreads();
            finite = group_total(bad, sums) == 0.0;
        }
        __syncthreads();  // sums and p are free again
        return s;
    };
    if constexpr (CG) {
        bool finite = true;
        rr = true_residual(true, finite);
        target = C.tol * sqrt(bb);
        if (!finite) {
            code = SMALL_INPUT;
        } else if (bb == 0.0) {
            code = SMALL_CONVERGED;
            rr = 0.0;
#pragma unroll
            for (int c = 0; c < 2; ++c) mine(c, [&](Own& o) { C.x[natural(L0, o.self())] = 0.0; });
        } else if (sqrt(rr) <= target) {
            code = SMALL_CONVERGED;
        }
    }
    bool first = true;
    while (code == SMALL_MORE) {
        // zero-guess pre-smoothing, further sweeps, residual of the red cells, restriction
        // (the black cells are cleared: behind a face that does not exist they read themselves, times 0)
        mine(0, [&](Own& o) { z0[o.self()] = o.r * o.dinv; });
        mine(1, [&](Own& o) { z0[o.self()] = 0.0; });
        __syncthreads();
        sweep0(1);
        for (int s = 1; s < nu_pre; ++s) {
            sweep0(0);
            sweep0(1);
        }
        mine(0, [&](Own& o) {
            // after a zero-guess pre-smoothing r - m z - sum w z = 0 on the red cells
            const int a = o.self();
            if (nu_pre > 1) {
                const double z = z0[a];
                t0[a] = o.r - L0.m[a] * z + o.gather(z0, z);
            } else {
                t0[a] = o.gather(z0, 0.0);
            }
        });
        __syncthreads();
        for (int l = 0; l < last; ++l) {
            const SmallLevel L = A->lv[l], N = A->lv[l + 1];
            double* const r = level_r(L);
            double* const z = r + L.n;
            double* const t = z + L.n;
            if (l > 0) {
                for_cells(L, 0, [&](Cell& c) { z[c.a] = r[c.a] * L.dinv[c.a]; });
                for_cells(L, 1, [&](Cell& c) { z[c.a] = 0.0; });
                __syncthreads();
                for (int s = 0; s < 2 * nu_pre - 1; ++s) {
                    for_cells(L, 1 ^ (s & 1), [&](Cell& c) {
                        double w[6], v = r[c.a];
                        c.look_round(L);
                        c.weights(L, w);
#pragma unroll
                        for (int q = 0; q < 6; ++q) v += w[q] * z[c.at[q]];
                        z[c.a] = v * L.dinv[c.a];
                    });
                    __syncthreads();
                }
                for_cells(L, 0, [&](Cell& c) {
                    double w[6];
                    c.look_round(L);
                    c.weights(L, w);
                    const double zc = nu_pre > 1 ? z[c.a] : 0.0;
                    double v = nu_pre > 1 ? r[c.a] - L.m[c.a] * zc : 0.0;
#pragma unroll
                    for (int q = 0; q < 6; ++q) v += w[q] * (z[c.at[q]] - zc);
                    t[c.a] = v;
                });
                __syncthreads();
            }
            restrict_red(L, N, l == 0 ? t0 : t, level_r(N));
            __syncthreads();
        }
        {
            // coarsest solve: by the helpers, by way of memory, or alone from LDS
            double* const r = level_r(A->lv[last]);
            double* const z = r + nc;
            if (me.size > 1) {
                for (int c = threadIdx.x; c < nc; c += kTT) st(args.exchange + c, r[c]);
                me.barrier();
                me.barrier();
                for (int c = threadIdx.x; c < nc; c += kTT) z[c] = ld(args.exchange + nc + c);
            } else {
                coarse_rows<false>(A->ainv, nc, 0, 1, Rows{}, [&](int c) { return r[c]; },
                                   [&](int row, double v) { z[row] = v; });
            }
            __syncthreads();
        }
        for (int l = last - 1; l >= 0; --l) {
            const SmallLevel L = A->lv[l], N = A->lv[l + 1];
            double* const r = level_r(L);
            double* const z = l == 0 ? z0 : r + L.n;
            prolong_red(L, N, level_r(N) + N.n, z);
            __syncthreads();
            if (l > 0)
                for (int s = 0; s < 2 * nu_post; ++s) {
                    for_cells(L, 1 ^ (s & 1), [&](Cell& c) {
                        double w[6], v = r[c.a];
                        c.look_round(L);
                        c.weights(L, w);
#pragma unroll
                        for (int q = 0; q < 6; ++q) v += w[q] * z[c.at[q]];
                        z[c.a] = v * L.dinv[c.a];
                    });
                    __syncthreads();
                }
        }
        for (int s = 0; s < nu_post; ++s) {
            sweep0(1);
            sweep0(0);
        }
        if constexpr (!CG) {
#pragma unroll
            for (int c = 0; c < 2; ++c) mine(c, [&](Own& o) { args.z[o.a] = me.lost ? __builtin_nan("") : z0[o.a]; });
            break;
        } else {
            double v = 0.0;
#pragma unroll
            for (int c = 0; c < 2; ++c) mine(c, [&](Own& o) { v += o.r * z0[o.self()]; });
            const double next = group_total(v, sums);
            beta = next / rz;
            rz = next;
            // x += alpha p, p = z + beta p
            const double al = alpha, be = beta;
#pragma unroll
            for (int c = 0; c < 2; ++c)
                mine(c, [&](Own& o) {
                    const int a = o.self();
                    double pv = z0[a];
                    if (!first) {
                        const double old = p0[a];
                        C.x[natural(L0, a)] += al * old;
                        pv += be * old;
                    }
                    p0[a] = pv;
                });
            first = false;
            __syncthreads();
            // q = A p, <p, q>
            v = 0.0;
#pragma unroll
            for (int c = 0; c < 2; ++c)
                mine(c, [&](Own& o) {
                    const int a = o.self();
                    const double pv = p0[a], s = L0.m[a] * pv - o.gather(p0, pv);
                    q0[a] = s;
                    v += pv * s;
                });
            const double pq = group_total(v, sums);
            const bool sound = pq > 0.0 && pq < INFINITY;
            alpha = sound ? rz / pq : 0.0;
            const double a2 = alpha;
            __syncthreads();  // sums are free again
            v = 0.0;
#pragma unroll
            for (int c = 0; c < 2; ++c)
                mine(c, [&](Own& o) {
                    o.r -= a2 * q0[o.self()];
                    v += o.r * o.r;
                });
            rr = group_total(v, sums);
            ++it;
            if (!sound) code = SMALL_BREAKDOWN;
            else if (!(rr < INFINITY)) code = SMALL_NAN;
            else if (sqrt(rr) <= target) code = SMALL_CONVERGED;
            else if (it >= C.budget) code = SMALL_BUDGET;
            if (me.lost) code = SMALL_LOST;
            if (code == SMALL_CONVERGED || code == SMALL_BUDGET) {
                // the update of x that is still due
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    mine(c, [&](Own& o) {
                        const int a = o.self();
                        C.x[natural(L0, a)] += a2 * p0[a];
                    });
                bool finite;
                rr = true_residual(false, finite);
                if (code == SMALL_CONVERGED && !(sqrt(rr) <= target)) {
                    // from the true residual again
                    ++rounds;
                    first = true;
                    code = it < C.budget ? SMALL_MORE : SMALL_BUDGET;
                }
            }
        }
    }
    if constexpr (CG) {
        if (threadIdx.x == 0) {
            C.result->rr = rr;
            C.result->bb = bb;
            C.result->iterations = it;
            C.result->rounds = rounds;
            C.result->code = code;
            st(&me.t->done, 1u);  // before the barrier that the helpers wait at
        }
        if (me.size > 1) me.barrier();
    } else {
        if (me.lost && threadIdx.x == 0) args.scal[S_FLAG] = FLAG_LOST;
    }
}

// A helper's program: its rows of every coarsest solve until the owner is done.
template <bool CG>
__device__ __forceinline__ void help(Member& me, const SmallArgs& args) {
    const SmallTable* A = (const SmallTable*)(constant_t)args.table;
    const int nc = A->nc;
    Rows held;
    held.load(A->ainv, nc, 2 * ((me.rank - 1) * kTW + (int)(threadIdx.x >> 6)), 0);
    while (true) {
        me.barrier();
        if (me.lost || (CG && ld(&me.t->done))) break;
        coarse_rows<true>(A->ainv, nc, me.rank - 1, me.size - 1, held, [&](int c) { return ld(args.exchange + c); },
                          [&](int row, double v) { st(args.exchange + nc + row, v); });
        me.barrier();
        if (!CG || me.lost) break;
    }
}

template <int U, bool CG>
__global__ __launch_bounds__(kTT) void k_small(SmallArgs args) {
    extern __shared__ double dynamic_lds[];
    __shared__ double sums[kTW];
    __shared__ int s_rank, s_size;
    SmallState* const t = args.state;
    if (threadIdx.x == 0) {
        const unsigned want = gridDim.x, closed = 0x10000u;
        int rank = 0, size = 1;
        if (want > 1) {
            const unsigned r = __hip_atomic_fetch_add(&t->joined, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            size = 0;
            if (r == 0) {
                for (int n = 0; n < kJoinPolls && ld(&t->joined) < want; ++n) {}
                size = (int)(__hip_atomic_fetch_or(&t->joined, closed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & (closed - 1));
                st(&t->size, (unsigned)size);
            } else if (r < closed) {
                // registered before the closing: the owner runs and will say the size
                for (int n = 0; n < kBarrierPolls && size == 0; ++n) size = (int)ld(&t->size);
            }
            rank = r < closed && size > 0 ? (int)r : -1;
        }
        s_rank = rank;
        s_size = size;
    }
    __syncthreads();
    Member me{t, s_rank, s_size, 0u, args.polls, 0};
    if (me.rank == 0)
        own<U, CG>(me, args, dynamic_lds, sums);
    else if (me.rank > 0)
        help<CG>(me, args);
    // the last workgroup to leave clears the state for the next launch
    __syncthreads();
    if (threadIdx.x == 0 && (gridDim.x == 1 || __hip_atomic_fetch_add(&t->left, 1u, __ATOMIC_RELAXED,
                                                                      __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1)) {
        st(&t->joined, 0u);
        st(&t->size, 0u);
        st(&t->arrived, 0u);
        st(&t->done, 0u);
        st(&t->left, 0u);
    }
}

}  // namespace

static void (*small_kernel(bool whole_cg, int per_thread))(SmallArgs) {
    if (per_thread <= 1) return whole_cg ? k_small<1, true> : k_small<1, false>;
    if (per_thread <= 2) return whole_cg ? k_small<2, true> : k_small<2, false>;
    return whole_cg ? k_small<4, true> : k_small<4, false>;
}

hipError_t prepare_small(const SmallShape& sh) {
    // more LDS than the default 64 KB has to be asked for
    hipError_t e = hipSuccess;
    for (bool cg : {false, true})
        if (e == hipSuccess && (!cg || sh.lds_cg))
            e = hipFuncSetAttribute((const void*)small_kernel(cg, sh.per_thread),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kSmallLds);
    return e;
}

void launch_small(const SmallArgs& a, bool whole_cg, const SmallShape& sh, hipStream_t s) {
    hipLaunchKernelGGL(small_kernel(whole_cg, sh.per_thread), dim3(sh.groups), dim3(kTT),
                       (whole_cg ? sh.lds_cg : sh.lds_cycle) * sizeof(double), s, a);
}

// The table, and of every cell of its levels (blockIdx.y) the inverse diagonals, as k_jacobi_diag computes
// them, and the weights of its high faces (0 where there is none). One launch for all these levels
// where k_jacobi_diag takes one each.
template <int FR>
__global__ __launch_bounds__(256) void k_small_setup(SmallTable a, SmallTable* table) {
    const SmallTable* A = (const SmallTable*)(constant_t)__builtin_amdgcn_kernarg_segment_ptr();
    const int l = blockIdx.y;
    const SmallLevel L = A->lv[l];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        table->lv[l] = L;
        if (l == 0) {
            table->ainv = A->ainv;
            table->levels = A->levels;
            table->nc = A->nc;
        }
    }
    for (int h = blockIdx.x * 256 + threadIdx.x; h < 2 * L.items; h += gridDim.x * 256) {
        const int c = h >= L.items;
        Cell e(L, c ? h - L.items : h, c);
        if (e.i >= L.g.nx) continue;
        e.look_round(L);
        const bool up[3] = {e.i < L.g.nx - 1 || L.g.px, e.j < L.g.ny - 1 || L.g.py, e.k < L.g.nz - 1 || L.g.pz};
        const double f[3] = {L.g.cx, L.g.cy, L.g.cz}, ra = L.rho[e.a], ma = L.m[e.a];
        const float ra32 = (float)ra;
        double d = ma;
        float d32 = (float)ma;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const bool face = q & 1 ? up[q >> 1] : e.lo[q >> 1];
            const double rb = L.rho[e.at[q]], kappa = face_kappa<FR>(ra, rb);
            d += (face ? f[q >> 1] : 0.0) * kappa;
            d32 += (face ? L.c32[q >> 1] : 0.0f) * face_kappa<FR>(ra32, (float)rb);
            if ((q & 1) && L.w) L.w[(int64_t)(q >> 1) * L.n + e.a] = face ? f[q >> 1] * kappa : 0.0;
        }
        L.dinv[e.a] = 1.0 / d;
        if (L.dinv32) L.dinv32[e.a] = 1.0f / d32;
    }
}

void launch_small_setup(const SmallTable& a, int face_rule, SmallTable* table, hipStream_t s) {
    const dim3 grid((unsigned)std::min((2 * a.lv[0].items + 255) / 256, 512), (unsigned)a.levels);
    WITH_FACE_RULE(face_rule, hipLaunchKernelGGL((k_small_setup<FRV>), grid, dim3(256), 0, s, a, table));
}

}  // namespace hp
