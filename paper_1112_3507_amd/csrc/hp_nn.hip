// hp_nn.hip -- the learned warm start / preconditioner: a small 3D U-Net in BF16 on the gfx950
// matrix cores (v_mfma_f32_16x16x32_bf16, FP32 accumulation), with hand-written forward,
// backward-data, backward-weight, pooling, head, loss and Adam kernels.
//
// Network (levels n, n/2, n/4; channels 16/32/64; 3x3x3 convolutions with periodic padding in
// x and y and zero padding in z, like the solver's boundaries):
//   e1 = relu(conv(relu(conv(in, 4->16)), 16->16))
//   e2 = relu(conv(relu(conv(pool(e1), 16->32)), 32->32))
//   e3 = relu(conv(relu(conv(pool(e2), 32->64)), 64->64))
//   d2 = relu(conv(relu(conv([up(e3), e2], 96->32)), 32->32))
//   d1 = relu(conv(relu(conv([up(d2), e1], 48->16)), 16->16))
//   y  = d1 . w_out + b_out
// pool = 2x2x2 mean, up = nearest 2x copy, [.,.] = channel concatenation (never materialised:
// the convolution reads the two tensors, and the upsampled one at half the coordinates).
//
// Layout: activations channels-last ([voxel][channel], x fastest) in bfloat16, gradients in
// FP32. Parameters are one flat FP32 vector: per convolution W[o][tap][c] then b[o], then
// w_out[16], b_out; taps t = (dz+1)*9 + (dy+1)*3 + (dx+1).
//
// Convolution as a GEMM on the matrix cores: D[o][v] = sum_k W[o][k] X[k][v] with k = (tap, c).
// A 256-thread workgroup owns a 16 x 4 x (4 SPW) brick of output voxels; the input brick with its
// one-voxel halo is staged in LDS one channel chunk at a time (each thread loading whole halo
// voxels at indices fixed for the launch); every wave64 owns SPW z-slices of the brick (four
// 16-voxel rows each). With one 16-channel output tile the weights of the chunk are staged in
// LDS and held in registers, and the products run input row by input row, each B fragment read
// once and fed to every output row it reaches (up to 9 products per LDS read); with several
// tiles each K step of 32 feeds one MFMA per tile and row. ReLU, the bfloat16 rounding and (in
// inference) the network head run in the epilogue. The backward-data pass is the same kernel with the weights
// flipped in space and transposed in channels; the backward-weight pass contracts over voxels
// with both operands transposed through LDS.
#include "hp.h"
#include "hp_internal.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

namespace hpnn {

typedef unsigned short bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BX = 16, BY = 4, BZ = 4;                 // output brick
constexpr int HX = BX + 2, HY = BY + 2, HZ = BZ + 2;  // input brick with halo
constexpr int HV = HX * HY * HZ;                       // 648 halo voxels
constexpr int NCONV = 10;
constexpr int CIN[NCONV] = {4, 16, 16, 32, 32, 64, 96, 32, 48, 16};
constexpr int COUT[NCONV] = {16, 16, 32, 32, 64, 64, 32, 32, 16, 16};
constexpr int HEAD = 16;

__host__ __device__ inline int cin_pad(int l) { return CIN[l] < 8 ? 8 : CIN[l]; }

__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float((unsigned)h << 16); }
// round to nearest even
__device__ __forceinline__ bf16_t f2bf(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

__device__ __forceinline__ bf16x8 as_bf8(uint4 u) { return __builtin_bit_cast(bf16x8, u); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
// two floats to two bfloat16 (round to nearest even) in one word, low half first: one
// v_cvt_pk_bf16_f32 on gfx950
__device__ __forceinline__ unsigned pack_bf2(float lo, float hi) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// ------------------------------------------------------------------------------------------
// convolution forward (also backward-data with transformed weights)

struct ConvArgs {
    const bf16_t* a;  // first input tensor (ca channels), half resolution if a_up
    int ca, a_up;
    const bf16_t* b;  // second input tensor (cb channels), full resolution
    int cb;
    const bf16_t* w;  // [cout][27 * (ca + cb)]
    const float* bias;
    void* out;        // [voxel][cout], bf16 or f32
    int cout;
    int nx, ny, nz;
    int relu;
    // non-null (one output tile only): the network head is applied in the epilogue and out is
    // y[voxel] (FP32) = sum_c bf16(act[voxel][c]) head[c] + head[16]; act itself is not stored
    const float* head;
    // non-null (one output tile, two z-slices per wave, bf16 output): the 2x2x2 mean of the
    // stored activation is written here as well ([coarse voxel][16], grid sizes halved)
    bf16_t* pool_out;
    // backward-data with the ReLU mask of the layer before it (OUT_GRAD, OUT_CONCAT): that layer's
    // stored activation, and the masked gradient before its rounding (for the bias gradient's sums)
    const bf16_t* mask = nullptr;
    float* full = nullptr;
    float* skip = nullptr;  // OUT_CONCAT: gradient of the skip channels [voxel][cout - 16 CU], FP32
};

// What a convolution stores: the (ReLU'd) activation in bfloat16; plain FP32; the gradient at the
// output of the layer before it, masked by that layer's ReLU, in bfloat16; or, for an input that is
// [upsampled, skip], the gradient of the upsampled part summed over the 2x2x2 children and masked
// like that at the coarse voxels, and the skip part in FP32. The masked forms write 6 bytes per
// value (2, and 4 for the bias sums) where an FP32 gradient, its split and a masking pass moved 22.
enum { OUT_ACT = 0, OUT_F32 = 1, OUT_GRAD = 2, OUT_CONCAT = 3 };

// SPW z-slices per wave: the output brick is 16 x 4 x (4 SPW) voxels.
template <int CT, int G, int SPW, int OUT>
__global__ __launch_bounds__(256) void k_conv_fwd(ConvArgs p) {
    constexpr int CC = 8 * G;                  // channels per LDS chunk
    constexpr int FZ = 4 * SPW, FHZ = FZ + 2, FHV = HX * HY * FHZ;
    constexpr int NV = (FHV + 255) / 256;      // halo voxels per thread (G 16-byte loads each)
    constexpr int NSTEPS = (27 * CC + 31) / 32;
    // one output tile (16 channels): its weights of the chunk are staged in LDS too
    constexpr bool WL = (CT == 1);
    constexpr int NWL = WL ? 16 * 27 * G : 0;  // 16-byte weight groups of the chunk
    constexpr int NUW = (NWL + 255) / 256;
    // LDS layout: the halo brick as G planes [8-channel group][halo voxel], so the 16 lanes that
    // read one B fragment row touch 16 consecutive 16-byte words; the weight rows at an odd
    // stride of 16-byte words for the same reason on the A fragment
    constexpr int WS = (27 * G) | 1;
    __shared__ uint4 lds[FHV * G + (WL ? 16 * WS : 0)];
    const int cin = p.ca + p.cb;
    const int bxn = (p.nx + BX - 1) / BX, byn = (p.ny + BY - 1) / BY;
    const int bid = blockIdx.x;
    const int x0 = (bid % bxn) * BX;
    const int y0 = ((bid / bxn) % byn) * BY;
    const int z0 = (bid / (bxn * byn)) * FZ;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, grp = lane >> 4;
    const int anx = p.a_up ? p.nx >> 1 : p.nx, any = p.a_up ? p.ny >> 1 : p.ny;
    const int Ktot = 27 * cin;

    // The thread's halo voxels (hv = tid + 256 i): their voxel index in the full-resolution
    // tensor b and in tensor a (half resolution when upsampled), -1 outside the grid (zero
    // padding in z; a brick wider than the grid reaches past the periodic image in x or y,
    // and those voxels only feed outputs outside the grid). Fixed for the whole launch.
    int vb[NV], va[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int hv = tid + 256 * i;
        const int hx = hv % HX, hy = (hv / HX) % HY, hz = hv / (HX * HY);
        int gx = x0 + hx - 1, gy = y0 + hy - 1;
        const int gz = z0 + hz - 1;
        gx = gx < 0 ? gx + p.nx : (gx >= p.nx ? gx - p.nx : gx);
        gy = gy < 0 ? gy + p.ny : (gy >= p.ny ? gy - p.ny : gy);
        const bool in = hv < FHV && gz >= 0 && gz < p.nz && gx >= 0 && gx < p.nx && gy >= 0 && gy < p.ny;
        vb[i] = in ? (gz * p.ny + gy) * p.nx + gx : -1;
        va[i] = !in ? -1 : (p.a_up ? ((gz >> 1) * any + (gy >> 1)) * anx + (gx >> 1) : vb[i]);
    }
    // accumulators start from the bias: this lane's outputs are channels ct*16 + 4 grp + e
    f32x4 acc[4 * SPW][CT];  // row r of slice sl at 4 sl + r
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        f32x4 b0 = {0.f, 0.f, 0.f, 0.f};
        if (p.bias) {
#pragma unroll
            for (int e = 0; e < 4; ++e) b0[e] = p.bias[ct * 16 + 4 * grp + e];
        }
#pragma unroll
        for (int r = 0; r < 4 * SPW; ++r) acc[r][ct] = b0;
    }
    // weight fragment of K step s: 8 consecutive k of output row ct*16 + li
    auto wload = [&](int c0, int s, uint4* w) {
        const int kk = s * 32 + grp * 8;
        const int tap = kk / CC, c = kk - tap * CC;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
            w[ct] = tap < 27 ? *(const uint4*)(p.w + (int64_t)(ct * 16 + li) * Ktot + tap * cin + c0 + c)
                             : uint4{0u, 0u, 0u, 0u};
    };

    for (int c0 = 0; c0 < cin; c0 += CC) {
        // stage the chunk: all loads of a thread in flight before its LDS stores; a thread takes
        // whole halo voxels (the chunk's CC channels are G consecutive 16-byte words in memory)
        const bool from_a = c0 < p.ca;
        const bf16_t* base = from_a ? p.a + c0 : p.b + (c0 - p.ca);
        const int cstride = from_a ? p.ca : p.cb;
        uint4 v[NV][G];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            // outside the grid: a harmless load of voxel 0, replaced by zeros
            const int idx = from_a ? va[i] : vb[i];
            const uint4* src = (const uint4*)(base + (int64_t)(idx < 0 ? 0 : idx) * cstride);
#pragma unroll
            for (int q = 0; q < G; ++q) {
                const uint4 t = src[q];
                v[i][q] = idx >= 0 ? t : uint4{0u, 0u, 0u, 0u};
            }
        }
        uint4 wcur[CT], wnext[CT];
        uint4 wv[NUW > 0 ? NUW : 1];
        if (WL) {
            // weight row o, tap, 8-channel group of the chunk -> lds[FHV G + o WS + tap G + group]
#pragma unroll
            for (int i = 0; i < NUW; ++i) {
                const int u = tid + 256 * i;
                wv[i] = uint4{0u, 0u, 0u, 0u};
                if ((i + 1) * 256 <= NWL || u < NWL) {
                    const int o = u / (27 * G), kq = u - o * (27 * G);
                    const int tap = kq / G, c8 = kq - tap * G;
                    wv[i] = *(const uint4*)(p.w + (int64_t)o * Ktot + tap * cin + c0 + c8 * 8);
                }
            }
        } else {
            wload(c0, 0, wcur);
        }
        __syncthreads();  // the previous chunk's reads of lds are done
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int hv = tid + 256 * i;
            if ((i + 1) * 256 <= FHV || hv < FHV) {
#pragma unroll
                for (int q = 0; q < G; ++q) lds[q * FHV + hv] = v[i][q];
            }
        }
        if (WL) {
#pragma unroll
            for (int i = 0; i < NUW; ++i) {
                const int u = tid + 256 * i;
                if ((i + 1) * 256 <= NWL || u < NWL) lds[FHV * G + (u / (27 * G)) * WS + u % (27 * G)] = wv[i];
            }
        }
        __syncthreads();
        if constexpr (WL) {
            // One output tile: the products are taken input row by input row, so that each B
            // fragment read from LDS feeds every output row that needs it (up to 9). A K step holds
            // TPS taps of one (dz, dy) pair, neighbouring in dx, times the CC channels of the
            // chunk; its A fragments (weights) stay in registers for the whole chunk. Taps past
            // dx = 2 have zero weights (a quarter or a third of the products when TPS > 1).
            constexpr int TPS = 32 / CC;             // taps per K step (1, 2 or 4)
            constexpr int NT = (3 + TPS - 1) / TPS;  // K steps per (dz, dy)
            const int tin = (grp * 8) / CC, cg = ((grp * 8) % CC) >> 3;
            bf16x8 aw[9][NT];
#pragma unroll
            for (int q = 0; q < 9; ++q)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int dx = t * TPS + tin;
                    const uint4 w = lds[FHV * G + li * WS + (q * 3 + (dx < 3 ? dx : 2)) * G + cg];
                    aw[q][t] = as_bf8(dx < 3 ? w : uint4{0u, 0u, 0u, 0u});
                }
#pragma unroll
            for (int iz = 0; iz < SPW + 2; ++iz)
#pragma unroll
                for (int iy = 0; iy < HY; ++iy)
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        // past dx = 2 the A side is zero; B reads the dx = 2 voxel (finite)
                        const int dx = t * TPS + tin;
                        const int hv = ((wave * SPW + iz) * HY + iy) * HX + li + (dx < 3 ? dx : 2);
                        const bf16x8 bf = as_bf8(lds[cg * FHV + hv]);
#pragma unroll
                        for (int dz = 0; dz < 3; ++dz)
#pragma unroll
                            for (int dy = 0; dy < 3; ++dy) {
                                const int sl = iz - dz, r = iy - dy;
                                if (sl < 0 || sl >= SPW || r < 0 || r >= 4) continue;
                                acc[sl * 4 + r][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    aw[dz * 3 + dy][t], bf, acc[sl * 4 + r][0], 0, 0, 0);
                            }
                    }
        } else {
            // several output tiles: K step by K step, each B fragment feeding CT products
#pragma unroll 2
            for (int s = 0; s < NSTEPS; ++s) {
                // next step's weights in flight while this step's products run
                if (s + 1 < NSTEPS) wload(c0, s + 1, wnext);
                const int kk = s * 32 + grp * 8;
                const int tap = kk / CC, c = kk - tap * CC;
                const bool kv = tap < 27;
                const int dz = tap / 9, dy = (tap / 3) % 3, dx = tap % 3;
                bf16x8 af[CT];
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) af[ct] = as_bf8(wcur[ct]);
#pragma unroll
                for (int sr = 0; sr < 4 * SPW; ++sr) {
                    const int sl = sr >> 2, r = sr & 3;
                    uint4 xv = {0u, 0u, 0u, 0u};
                    if (kv) {
                        const int hv = ((wave * SPW + sl + dz) * HY + (r + dy)) * HX + (li + dx);
                        xv = lds[(c >> 3) * FHV + hv];
                    }
                    const bf16x8 bf = as_bf8(xv);
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
                        acc[sr][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ct], bf, acc[sr][ct], 0, 0, 0);
                }
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) wcur[ct] = wnext[ct];
            }
        }
    }
    // epilogue: this lane holds D[o = ct*16 + 4*grp + e][voxel li of row r of slice sl] (bias
    // included); a brick inside the grid needs no bounds checks
    const bool full = x0 + BX <= p.nx && y0 + BY <= p.ny && z0 + FZ <= p.nz;
    const int gx = x0 + li;
    constexpr int CU = OUT == OUT_CONCAT ? 2 * CT / 3 : 0;   // output tiles of the upsampled part
    // v masked by the activation at `at` (4 channels), stored as bfloat16 and in full
    auto mask_store = [&](f32x4 v, int64_t at) {
        const uint2 a = *(const uint2*)(p.mask + at);
        const unsigned on[4] = {a.x << 16, a.x & 0xffff0000u, a.y << 16, a.y & 0xffff0000u};
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(on[e]) > 0.f ? v[e] : 0.f;
        *(f32x4*)(p.full + at) = v;
        *(uint2*)((bf16_t*)p.out + at) = uint2{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
    };
    if constexpr (OUT == OUT_CONCAT) {
        // The children of a coarse voxel sit in two lanes (x), two rows (y) and two waves (z, handed
        // over through LDS); they are added one after the other, x fastest.
        static_assert(2 * 4 * CU * 64 <= FHV * G, "in the place of the staged brick");
        __syncthreads();
        f32x4* odd = (f32x4*)lds + (wave >> 1) * (4 * CU * 64);
        if (wave & 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int ct = 0; ct < CU; ++ct) odd[(r * CU + ct) * 64 + lane] = acc[r][ct];
        }
        __syncthreads();
        if (!(wave & 1)) {
            const int gz = z0 + wave;
#pragma unroll
            for (int yp = 0; yp < 2; ++yp) {
                const int gy = y0 + 2 * yp;
                const bool in = !(li & 1) && gx < p.nx && gy < p.ny && gz < p.nz;
                const int64_t vox = ((int64_t)(gz >> 1) * (p.ny >> 1) + (gy >> 1)) * (p.nx >> 1) + (gx >> 1);
#pragma unroll
                for (int ct = 0; ct < CU; ++ct) {
                    f32x4 s = acc[2 * yp][ct];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        s[e] += __shfl_xor(acc[2 * yp][ct][e], 1, 64);
                        s[e] += acc[2 * yp + 1][ct][e];
                        s[e] += __shfl_xor(acc[2 * yp + 1][ct][e], 1, 64);
                    }
#pragma unroll
                    for (int y = 0; y < 2; ++y)
#pragma unroll
                        for (int x = 0; x < 2; ++x) s += odd[((2 * yp + y) * CU + ct) * 64 + (lane ^ x)];
                    if (in) mask_store(s, vox * (16 * CU) + ct * 16 + 4 * grp);
                }
            }
        }
    }
    constexpr bool POOL = (CT == 1 && SPW == 2 && OUT == OUT_ACT);
    uint2 stored[POOL ? 4 * SPW : 1];  // the bfloat16 pairs written for each row (pooling)
#pragma unroll
    for (int sr = 0; sr < (POOL ? 4 * SPW : 1); ++sr) stored[sr] = uint2{0u, 0u};
#pragma unroll
    for (int sr = 0; sr < 4 * SPW; ++sr) {
        const int gz = z0 + wave * SPW + (sr >> 2), gy = y0 + (sr & 3);
        if (!full && (gx >= p.nx || gy >= p.ny || gz >= p.nz)) continue;
        const int64_t vox = ((int64_t)gz * p.ny + gy) * p.nx + gx;
#pragma unroll
        for (int ct = CU; ct < CT; ++ct) {
            const int o = ct * 16 + 4 * grp;
            if constexpr (OUT == OUT_CONCAT) {
                *(f32x4*)(p.skip + vox * (16 * (CT - CU)) + (o - 16 * CU)) = acc[sr][ct];
                continue;
            }
            if constexpr (OUT == OUT_GRAD) {
                mask_store(acc[sr][ct], vox * p.cout + o);
                continue;
            }
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = p.relu ? fmaxf(acc[sr][ct][e], 0.f) : acc[sr][ct][e];
            if (CT == 1 && p.head) {
                // the activation as it would be stored (bfloat16), dotted with the head weights;
                // the four lanes of a voxel hold channels 4 grp .. 4 grp + 3
                const unsigned q0 = pack_bf2(v[0], v[1]), q1 = pack_bf2(v[2], v[3]);
                float part = __uint_as_float(q0 << 16) * p.head[o] + __uint_as_float(q0 & 0xffff0000u) * p.head[o + 1] +
                             __uint_as_float(q1 << 16) * p.head[o + 2] + __uint_as_float(q1 & 0xffff0000u) * p.head[o + 3];
                part += __shfl_xor(part, 16, 64);
                part += __shfl_xor(part, 32, 64);
                if (grp == 0) ((float*)p.out)[vox] = part + p.head[HEAD];
                continue;
            }
            if (OUT == OUT_F32) {
                *(float4*)((float*)p.out + vox * p.cout + o) = make_float4(v[0], v[1], v[2], v[3]);
            } else {
                uint2 pk;
                pk.x = pack_bf2(v[0], v[1]);
                pk.y = pack_bf2(v[2], v[3]);
                *(uint2*)((bf16_t*)p.out + vox * p.cout + o) = pk;
                if constexpr (POOL) stored[sr] = pk;
            }
        }
    }
    if constexpr (POOL) {
        if (p.pool_out) {
            // 2x2x2 mean of the stored activation: the wave holds two z-slices and four y rows, and
            // the x pair sits in lanes li, li + 1. The eight values of each channel are summed in
            // z, y, x order (x fastest) in FP32, then halved three times and rounded.
            const int cx = p.nx >> 1, cy = p.ny >> 1;
            const int X = gx >> 1, Z = (z0 + wave * SPW) >> 1;
#pragma unroll
            for (int yp = 0; yp < 2; ++yp) {
                float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int zc = 0; zc < 2; ++zc)
#pragma unroll
                    for (int yc = 0; yc < 2; ++yc) {
                        const uint2 own = stored[zc * 4 + 2 * yp + yc];
                        const uint2 nxt = uint2{(unsigned)__shfl_down((int)own.x, 1, 64),
                                                (unsigned)__shfl_down((int)own.y, 1, 64)};
                        const unsigned w[2][2] = {{own.x, own.y}, {nxt.x, nxt.y}};
#pragma unroll
                        for (int xc = 0; xc < 2; ++xc) {
                            sum[0] += __uint_as_float(w[xc][0] << 16);
                            sum[1] += __uint_as_float(w[xc][0] & 0xffff0000u);
                            sum[2] += __uint_as_float(w[xc][1] << 16);
                            sum[3] += __uint_as_float(w[xc][1] & 0xffff0000u);
                        }
                    }
                const int Y = (y0 >> 1) + yp;
                if (!(li & 1) && gx < p.nx && 2 * Y < p.ny && 2 * Z < p.nz) {
                    uint2 pk;
                    pk.x = pack_bf2(sum[0] * 0.125f, sum[1] * 0.125f);
                    pk.y = pack_bf2(sum[2] * 0.125f, sum[3] * 0.125f);
                    *(uint2*)(p.pool_out + (((int64_t)Z * cy + Y) * cx + X) * 16 + 4 * grp) = pk;
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// backward weights: dW[o][t][c] = sum_v g[v][o] x[v + d_t][c], a contraction over voxels, in kBwdWParts
// partial sums over every kBwdWParts-th brick of 16 x 4 x 4 voxels. The order of every sum is fixed: brick by
// brick, its rows in y pairs, one matrix product of 32 voxels for each (lane group g of the product: voxels
// 8 g .. 8 g + 7 of the pair). Training keeps its weights for long, and they must not move with the launch
// shape: a gradient that differs in its last bit flips a bfloat16 rounding now and then, and a step
// later the gradients are 1e-4 apart.
//
// A workgroup owns 16 output and 16 input channels of one partial sum. Its first three waves multiply: wave w the nine
// taps of x offset w, walking the input's row pairs, each B fragment read once for every product it has a
// part in (30 fragments for 72 products). The other kLoaders threads bring the bricks: loads two bricks
// ahead in registers, into one of two LDS bricks as they lie in memory ([voxel][16 channels], 16-byte
// stores) while the other is multiplied, one barrier per brick; the LDS transposed read
// (ds_read_b64_tr_b16) hands each lane four voxels of one channel. A workgroup has up to 1 / 96 of the bricks one
// after the other, so a brick's time counts: 1.4 us at 128^3, bound by the loaders (120 us for a 16 -> 16 layer,
// 176 for 48 -> 16); 1.7 with the same waves loading and multiplying in turn, and 10 (870 us for the layer)
// with 2-byte transposes written to LDS. More partial sums would give shorter chains (512 of them: 44 us), but
// other sums.

struct BwdWArgs {
    const bf16_t* g;  // [voxel][cout] gradient at the convolution output (after the ReLU mask)
    int cout;
    const bf16_t* a;  // conv input tensors as in ConvArgs
    int ca, a_up;
    const bf16_t* b;
    int cb;
    float* partial;   // [gridDim.x][cin_chunks][cout][27][16]
    int nx, ny, nz;
};

constexpr int kBwdWParts = 96;
constexpr int kMultipliers = 192, kLoaders = 320;  // threads

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

// MFMA fragment (lane li: channel li; K = eight x positions from the lane's word p on) from
// [voxel][16 channels] in LDS
__device__ __forceinline__ bf16x8 frag_tr(const uint2* p) {
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p + 16));
    typedef short i16x8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

__global__ __launch_bounds__(kMultipliers + kLoaders, 1) void k_conv_bwd_w(BwdWArgs p) {
    constexpr int XW = 2 * HV, GW = 2 * BX * BY * BZ;  // 16-byte words of the halo brick and of g's
    constexpr int NX = (XW + kLoaders - 1) / kLoaders, NG = (GW + kLoaders - 1) / kLoaders;
    // (every loader stores all its words: what is past the brick goes to the padding)
    constexpr int XP = NX * kLoaders, GP = NG * kLoaders;
    __shared__ uint4 lds[2][XP + GP];
    const int cin = p.ca + p.cb;
    const int c0 = blockIdx.y * 16, o0 = blockIdx.z * 16;
    const int tid = (int)threadIdx.x - kMultipliers, lane = threadIdx.x & 63, dx = threadIdx.x >> 6;
    const int li = lane & 15, grp = lane >> 4;
    const int bxn = (p.nx + BX - 1) / BX, byn = (p.ny + BY - 1) / BY, bzn = (p.nz + BZ - 1) / BZ;
    const int nbricks = bxn * byn * bzn;
    const bool from_a = c0 < p.ca;
    // Byte offsets of this thread's words from the first voxel of a brick's halo (of an
    // inner brick; an upsampled input's voxels have half the coordinates) and of the brick.
    const int xc = from_a ? p.ca : p.cb, xs = from_a && p.a_up ? 1 : 0, xnx = p.nx >> xs, xny = p.ny >> xs;
    const char* const xbase = (const char*)(from_a ? p.a + c0 : p.b + (c0 - p.ca));
    const char* const gbase = (const char*)(p.g + o0);
    // which half of its voxel's channels a thread takes is fixed; the first layer has no second half
    const int half = (tid & 1) * 8;
    const bool there = c0 + half < cin;
    int64_t xoff[NX], goff[NG];
    unsigned hpos[NX], gpos[NG];  // and the coordinates, 8 bits each
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int hv = min(tid + kLoaders * i, XW - 1) >> 1, hx = hv % HX, hy = (hv / HX) % HY, hz = hv / (HX * HY);
        // (an inner brick starts at even coordinates: its halo's first voxel is at -1, of which the half is -1)
        const int x = xs ? (hx + 1) >> 1 : hx, y = xs ? (hy + 1) >> 1 : hy, z = xs ? (hz + 1) >> 1 : hz;
        xoff[i] = (int64_t)((z * xny + y) * xnx + x) * (xc * 2) + (there ? half * 2 : 0);
        hpos[i] = hx | hy << 8 | hz << 16;
    }
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        const int v = min(tid + kLoaders * i, GW - 1) >> 1, vx = v % BX, vy = (v / BX) % BY, vz = v / (BX * BY);
        goff[i] = (int64_t)((vz * p.ny + vy) * p.nx + vx) * (p.cout * 2) + half * 2;
        gpos[i] = vx | vy << 8 | vz << 16;
    }

    struct Stage {
        uint4 x[NX], g[NG];
        unsigned in;  // which of them lie inside, one bit each
    };
    constexpr unsigned kAll = (1u << (NX + NG)) - 1;
    // Where this workgroup's next 64 bricks lie, one to a lane (the divisions and products of one brick alone
    // would take longer than its matrix products): its coordinates, the voxels that the offsets count
    // from (-1 where the brick isn't an inner one).
    const int step = gridDim.x;
    int bx, by, bz, xat, gat;
    auto plan = [&](int k) {
        const int b = min((int)blockIdx.x + (k + lane) * step, nbricks - 1), row = b / bxn;
        bx = (b - row * bxn) * BX;
        bz = row / byn * BZ;
        by = (row - row / byn * byn) * BY;
        const bool inner = bx > 0 && bx + BX < p.nx && by > 0 && by + BY < p.ny && bz > 0 && bz + BZ < p.nz;
        xat = inner ? (((bz - 1) >> xs) * xny + ((by - 1) >> xs)) * xnx + ((bx - 1) >> xs) : -1;
        gat = (bz * p.ny + by) * p.nx + bx;
    };
    // (the loads are the same instructions for every brick, and for none past the last: only then can the
    // wait for one stage's leave the next one's in flight)
    auto fetch = [&](int k, Stage& st) {
        if ((k & 63) == 0) plan(k);
        int xv = __builtin_amdgcn_readlane(xat, k & 63), gv = __builtin_amdgcn_readlane(gat, k & 63);
        int64_t xo[NX], go[NG];
        unsigned in = kAll;
        if (xv >= 0) {
#pragma unroll
            for (int i = 0; i < NX; ++i) xo[i] = xoff[i];
#pragma unroll
            for (int i = 0; i < NG; ++i) go[i] = goff[i];
        } else {
            const int x0 = __builtin_amdgcn_readlane(bx, k & 63), y0 = __builtin_amdgcn_readlane(by, k & 63),
                      z0 = __builtin_amdgcn_readlane(bz, k & 63);
            xv = gv = 0;
            in = 0u;
#pragma unroll
            for (int i = 0; i < NX; ++i) {
                int gx = x0 + (int)(hpos[i] & 255u) - 1, gy = y0 + (int)(hpos[i] >> 8 & 255u) - 1;
                const int gz = z0 + (int)(hpos[i] >> 16) - 1;
                gx = gx < 0 ? gx + p.nx : (gx >= p.nx ? gx - p.nx : gx);
                gy = gy < 0 ? gy + p.ny : (gy >= p.ny ? gy - p.ny : gy);
                // past the periodic image (a brick wider than the grid): zero, as its gradient is
                const bool ok = (gz >= 0) & (gz < p.nz) & (gx >= 0) & (gx < p.nx) & (gy >= 0) & (gy < p.ny);
                in |= ok ? 1u << i : 0u;
                const int v = ok ? ((gz >> xs) * xny + (gy >> xs)) * xnx + (gx >> xs) : 0;
                xo[i] = (int64_t)v * (xc * 2) + (there ? half * 2 : 0);
            }
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                const int gx = x0 + (int)(gpos[i] & 255u), gy = y0 + (int)(gpos[i] >> 8 & 255u), gz = z0 + (int)(gpos[i] >> 16);
                const bool ok = (gx < p.nx) & (gy < p.ny) & (gz < p.nz);
                in |= ok ? 1u << (NX + i) : 0u;
                go[i] = (int64_t)(ok ? (gz * p.ny + gy) * p.nx + gx : 0) * (p.cout * 2) + half * 2;
            }
        }
        if (!there) in &= ~((1u << NX) - 1);
        st.in = (int)blockIdx.x + k * step < nbricks ? in : 0u;
        const char* const xfrom = xbase + (int64_t)xv * (xc * 2);
        const char* const gfrom = gbase + (int64_t)gv * (p.cout * 2);
#pragma unroll
        for (int i = 0; i < NX; ++i) st.x[i] = *(const uint4*)(xfrom + xo[i]);
#pragma unroll
        for (int i = 0; i < NG; ++i) st.g[i] = *(const uint4*)(gfrom + go[i]);
    };
    auto store = [&](const Stage& st, uint4* to) {
        auto put = [&](int at, const uint4& v, int bit) {
            const unsigned m = 0u - (st.in >> bit & 1u);
            to[at] = uint4{v.x & m, v.y & m, v.z & m, v.w & m};
        };
#pragma unroll
        for (int i = 0; i < NX; ++i) put(tid + kLoaders * i, st.x[i], i);
#pragma unroll
        for (int i = 0; i < NG; ++i) put(XP + tid + kLoaders * i, st.g[i], NX + i);
    };
    // consecutive workgroups take consecutive bricks in turn, so that those running together
    // share halo lines in the caches; two a turn, a brick of zeros past an odd last one
    const int mine = (nbricks - (int)blockIdx.x + step - 1) / step;
    if (tid >= 0) {
        Stage st[2];
        fetch(0, st[0]);
        fetch(1, st[1]);
        store(st[0], lds[0]);
        fetch(2, st[0]);
        __syncthreads();
        for (int k = 0; k < mine; k += 2)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                store(st[1 - q], lds[1 - q]);
                fetch(k + q + 3, st[1 - q]);
                __syncthreads();
            }
        return;
    }

    f32x4 acc[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    // this lane's word of the transposed reads: of the row pair's row grp / 2, the voxel 8 (grp % 2) + li / 4,
    // channels 4 (li % 4) ...
    const int at = (8 * (grp & 1) + (li >> 2)) * 4 + (li & 3);
    auto multiply = [&](const uint4* from) {
        const uint2* gw = (const uint2*)(from + XP) + (grp >> 1) * (BX * 4) + at;
        const uint2* xw = (const uint2*)from + (grp >> 1) * (HX * 4) + dx * 4 + at;
        bf16x8 af[2 * BZ];
#pragma unroll
        for (int q = 0; q < 2 * BZ; ++q) af[q] = frag_tr(gw + q * 2 * BX * 4);
#pragma unroll
        for (int iz = 0; iz < HZ; ++iz)
#pragma unroll
            for (int iy = 0; iy < HY - 1; ++iy) {
                const bf16x8 bf = frag_tr(xw + (iz * HY + iy) * HX * 4);
#pragma unroll
                for (int dz = 0; dz < 3; ++dz)
#pragma unroll
                    for (int dy = 0; dy < 3; ++dy) {
                        const int z = iz - dz, y = iy - dy;
                        if (z < 0 || z >= BZ || (y != 0 && y != 2)) continue;
                        acc[dz * 3 + dy] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[2 * z + y / 2], bf, acc[dz * 3 + dy], 0, 0, 0);
                    }
            }
    };
    __syncthreads();
    for (int k = 0; k < mine; k += 2) {
        multiply(lds[0]);
        __syncthreads();
        multiply(lds[1]);
        __syncthreads();
    }
    // the lane holds D[o = 4 grp + e][c = li] of its taps
    float* out = p.partial + (((int64_t)blockIdx.x * gridDim.y + blockIdx.y) * p.cout + o0) * (27 * 16);
#pragma unroll
    for (int q = 0; q < 9; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) out[((int64_t)(4 * grp + e) * 27 + 3 * q + dx) * 16 + li] = acc[q][e];
}

// sum the per-workgroup partials in a fixed order into the flat gradient W[o][t][c] (c < creal):
// 16 weights per workgroup, 16 threads for each (part q goes to thread q % 16), in FP64
__global__ __launch_bounds__(256) void k_reduce_dw(const float* __restrict__ partial, int nparts, int nchunks, int cout,
                                                   int creal, float* __restrict__ gw) {
    __shared__ double sm[16][17];
    const int w = threadIdx.x & 15, lane = threadIdx.x >> 4;
    const int idx = blockIdx.x * 16 + w;  // over cout * 27 * creal
    const int n = cout * 27 * creal;
    const int id = idx < n ? idx : 0;
    const int c = id % creal, t = (id / creal) % 27, o = id / (creal * 27);
    const float* at = partial + ((int64_t)(c / 16) * cout * 27 + (int64_t)o * 27 + t) * 16 + c % 16;
    const int64_t stride = (int64_t)nchunks * cout * 27 * 16;
    double s = 0.0;
#pragma unroll 8
    for (int q = lane; q < nparts; q += 16) s += at[q * stride];
    sm[w][lane] = s;
    __syncthreads();
    if (lane == 0 && idx < n) {
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < 16; ++q) v += sm[w][q];
        gw[idx] = (float)v;
    }
}

// ------------------------------------------------------------------------------------------
// elementwise and small kernels

// network input: [b/s, log rho, log c2, p_prev/s, 0, 0, 0, 0] in bf16; s = sqrt(scal[0])
// (c2 may be null: then log c2 = -log(rho m) from the mass term m = 1/(rho c2))
// Position of natural-order cell v in the red-black split storage of an nx x ny x nz level (each x
// row holds its red cells, then its black cells; nx even): where the solver keeps its finest-level
// vectors.
__device__ __forceinline__ int64_t split_pos(int64_t v, int nx, int ny) {
    const int64_t row = v / nx;
    const int i = (int)(v - row * nx);
    const int j = (int)(row % ny);
    const int64_t k = row / ny;
    const int c = (int)((i + j + k) & 1);
    return row * nx + c * (nx >> 1) + (i >> 1);
}

// b and pprev in natural order or (split != 0) in the split storage of the nx x ny grid; rho,
// c2 and m always in natural order
__global__ void k_features(const double* __restrict__ b, const double* __restrict__ rho,
                           const double* __restrict__ c2, const double* __restrict__ m,
                           const double* __restrict__ pprev, const double* __restrict__ ss,
                           bf16_t* __restrict__ out, int64_t n, int split, int nx, int ny) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const int64_t vb = split ? split_pos(v, nx, ny) : v;
    const double inv = 1.0 / ss[1];
    const double lc2 = c2 ? log(c2[v]) : -log(rho[v] * m[v]);
    uint4 pk;
    pk.x = (unsigned)f2bf((float)(b[vb] * inv)) | ((unsigned)f2bf((float)log(rho[v])) << 16);
    pk.y = (unsigned)f2bf((float)lc2) | ((unsigned)f2bf((float)(pprev ? pprev[vb] * inv : 0.0)) << 16);
    pk.z = 0u;
    pk.w = 0u;
    *(uint4*)(out + v * 8) = pk;
}

// scale: ss[0] = sum b^2 (from a reduction), ss[1] = sqrt(mean b^2) (1 when b = 0)
__global__ void k_scale(double* ss, double n) {
    const double m = ss[0] / n;
    ss[1] = m > 0.0 ? sqrt(m) : 1.0;
}

__global__ void k_sumsq_partial(const double* __restrict__ b, int64_t n, double* partial) {
    double acc = 0.0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        acc += b[v] * b[v];
    __shared__ double ws[4];
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = ws[0] + ws[1] + ws[2] + ws[3];
}

__global__ void k_sum_partials(const double* partial, int n, double* out) {
    double acc = 0.0;
    for (int q = threadIdx.x; q < n; q += blockDim.x) acc += partial[q];
    __shared__ double ws[4];
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) *out = ws[0] + ws[1] + ws[2] + ws[3];
}

// 2x2x2 mean (bf16 in/out), coarse dims (cx, cy, cz), c channels (a multiple of 8): one thread
// per coarse voxel and 8-channel group, 16-byte loads
__global__ void k_pool(const bf16_t* __restrict__ in, bf16_t* __restrict__ out, int cx, int cy,
                       int cz, int c) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int cg = c >> 3;
    const int64_t total = (int64_t)cx * cy * cz * cg;
    if (idx >= total) return;
    const int g = (int)(idx % cg);
    const int64_t v = idx / cg;
    const int x = (int)(v % cx), y = (int)((v / cx) % cy), z = (int)(v / ((int64_t)cx * cy));
    const int fx = 2 * cx, fy = 2 * cy;
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int64_t fv = ((int64_t)(2 * z + (q >> 2)) * fy + (2 * y + ((q >> 1) & 1))) * fx + (2 * x + (q & 1));
        const uint4 w = *(const uint4*)(in + fv * c + 8 * g);
        const unsigned u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[2 * e] += __uint_as_float(u[e] << 16);
            s[2 * e + 1] += __uint_as_float(u[e] & 0xffff0000u);
        }
    }
    uint4 r;
    r.x = pack_bf2(s[0] * 0.125f, s[1] * 0.125f);
    r.y = pack_bf2(s[2] * 0.125f, s[3] * 0.125f);
    r.z = pack_bf2(s[4] * 0.125f, s[5] * 0.125f);
    r.w = pack_bf2(s[6] * 0.125f, s[7] * 0.125f);
    *(uint4*)(out + v * c + 8 * g) = r;
}

// Channel sums (bias and head gradients). Like the weights' sums theirs keep one order whatever the launch: FP32
// sums over groups of 64 consecutive voxels, voxel j of every 256 / C together first, then j = 0, 1, ..; FP64
// over the groups. A wave takes a group, lane (j, q) channels 4 q .. 4 q + 3.
constexpr int kSumVox = 4 * 64;  // voxels per workgroup

// the group's sums of channel `lane` from the lanes' own sums; `ws`: 64 values of LDS for this wave
template <int C>
__device__ __forceinline__ float group_sum(float4 own, float4* ws) {
    const int lane = threadIdx.x & 63;
    ws[lane] = own;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    float s = 0.f;
    if (lane < C)
#pragma unroll
        for (int j = 0; j < 256 / C; ++j) s += ((const float*)ws)[j * C + lane];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return s;
}

// the workgroup's sums: partial[block][C] from each wave's sum of channel `lane`
template <int C>
__device__ __forceinline__ void block_sums(double total, double* __restrict__ partial) {
    __shared__ double sums[4][64];
    sums[threadIdx.x >> 6][threadIdx.x & 63] = total;
    __syncthreads();
    if (threadIdx.x < C)
        partial[(int64_t)blockIdx.x * C + threadIdx.x] =
            (sums[0][threadIdx.x] + sums[1][threadIdx.x]) + (sums[2][threadIdx.x] + sums[3][threadIdx.x]);
}

// Channel sums of g[v][C].
template <int C>
__global__ __launch_bounds__(256) void k_channel_sums(const float* __restrict__ g, int64_t nv, double* __restrict__ partial) {
    __shared__ float4 ws[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t v0 = (int64_t)blockIdx.x * kSumVox + wave * 64 + lane / (C / 4);
    float4 own = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < C / 4; ++i) {
        const int64_t v = v0 + i * (256 / C);
        if (v < nv) {
            const float4 t = *(const float4*)(g + v * C + 4 * (lane % (C / 4)));
            own.x += t.x;
            own.y += t.y;
            own.z += t.z;
            own.w += t.w;
        }
    }
    block_sums<C>(group_sum<C>(own, ws[wave]), partial);
}

// Gradient at a skip connection's activation, g[v][C] + gpool[v/2][C] / 8 (the 2x2x2 pooling's
// gradient), masked by the activation and rounded to bfloat16 (the operand of the backward
// convolutions), with the channel sums of the masked value. Bound by its memory traffic (53 us at
// 128^3 x 16, 5.3 TB/s).
template <int C>
__global__ __launch_bounds__(256) void k_relu_bwd_pool(const float* __restrict__ g, const float* __restrict__ gpool,
                                                       const bf16_t* __restrict__ act, bf16_t* __restrict__ gp, int nx,
                                                       int ny, int64_t nv, double* __restrict__ partial) {
    __shared__ float4 ws[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, ch = 4 * (lane % (C / 4));
    const int cx = nx >> 1, cy = ny >> 1;
    const int64_t v0 = (int64_t)blockIdx.x * kSumVox + wave * 64 + lane / (C / 4);
    float4 own = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < C / 4; ++i) {
        const int64_t v = v0 + i * (256 / C);
        if (v < nv) {
            // (fewer than 2^31 voxels)
            const int x = (int)v % nx, row = (int)v / nx, y = row % ny, z = row / ny;
            const int64_t cv = ((int64_t)(z >> 1) * cy + (y >> 1)) * cx + (x >> 1);
            const float4 a = *(const float4*)(g + v * C + ch), b = *(const float4*)(gpool + cv * C + ch);
            const uint2 w = *(const uint2*)(act + v * C + ch);
            const float4 t = {__uint_as_float(w.x << 16) > 0.f ? a.x + b.x * 0.125f : 0.f,
                              __uint_as_float(w.x & 0xffff0000u) > 0.f ? a.y + b.y * 0.125f : 0.f,
                              __uint_as_float(w.y << 16) > 0.f ? a.z + b.z * 0.125f : 0.f,
                              __uint_as_float(w.y & 0xffff0000u) > 0.f ? a.w + b.w * 0.125f : 0.f};
            own.x += t.x;
            own.y += t.y;
            own.z += t.z;
            own.w += t.w;
            *(uint2*)(gp + v * C + ch) = uint2{pack_bf2(t.x, t.y), pack_bf2(t.z, t.w)};
        }
    }
    block_sums<C>(group_sum<C>(own, ws[wave]), partial);
}

// column sums of partial[nrows][stride], columns c0 + blockIdx.x: one workgroup per column,
// fixed-order tree
__global__ __launch_bounds__(256) void k_reduce_cols(const double* __restrict__ partial, int nrows, int stride, int c0,
                                                     float* __restrict__ out) {
    __shared__ double sm[256];
    const int ch = blockIdx.x, tid = threadIdx.x;
    double s = 0.0;
#pragma unroll 8
    for (int q = tid; q < nrows; q += 256) s += partial[(int64_t)q * stride + c0 + ch];
    sm[tid] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) sm[tid] += sm[tid + w];
        __syncthreads();
    }
    if (tid == 0) out[ch] = (float)sm[0];
}

// head: y[v] = sum_c d1[v][c] w[c] + b
__global__ void k_head(const bf16_t* __restrict__ d1, const float* __restrict__ wb, float* __restrict__ y,
                       int64_t nv) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nv) return;
    float s = wb[HEAD];
#pragma unroll
    for (int c = 0; c < HEAD; ++c) s += bf2f(d1[v * HEAD + c]) * wb[c];
    y[v] = s;
}

// loss = mean (y - t)^2 ; gy = 2 (y - t) / n ; block partial sums of the squared error
__global__ void k_loss(const float* __restrict__ y, const float* __restrict__ t, float* __restrict__ gy,
                       int64_t n, double* __restrict__ partial) {
    double acc = 0.0;
    const double inv = 2.0 / (double)n;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const double d = (double)y[v] - (double)t[v];
        acc += d * d;
        gy[v] = (float)(d * inv);
    }
    __shared__ double ws[4];
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = ws[0] + ws[1] + ws[2] + ws[3];
}

// Head backward with the last layer's ReLU: gp[v][c] = bf16(gy[v] w[c] where d1[v][c] > 0, else 0);
// partial[block][0..15] = sum gy d1, [16] = sum gy, [17..32] = sum of the masked gradient before its rounding (the last
// layer's bias gradient). The head's sums keep an order too: FP32 over 256 consecutive voxels, voxels t, t + 64,
// .. together first, then t = 0, 1, ..; so thread (t, q) takes those voxels, channels 4 q .. 4 q + 3, and the bias
// sums' groups of 64 (see group_sum) go through LDS. kHeadVox voxels per workgroup.
constexpr int kHeadVox = 1024, kHeadCols = 2 * HEAD + 1;

__global__ __launch_bounds__(256) void k_head_bwd(const float* __restrict__ gy, const bf16_t* __restrict__ d1,
                                                  const float* __restrict__ wb, bf16_t* __restrict__ gp, int64_t nv,
                                                  double* __restrict__ partial) {
    __shared__ float4 masked[256][4];   // [voxel][q]
    __shared__ float4 heads[64][4];     // [t][q]: sum of gy d1
    __shared__ float ones[64];          // [t]: sum of gy
    const int tid = threadIdx.x, t = tid >> 2, q = tid & 3, lane = tid & 63, wave = tid >> 6;
    const float w[4] = {wb[4 * q], wb[4 * q + 1], wb[4 * q + 2], wb[4 * q + 3]};
    double total = 0.0, bias = 0.0;  // of column tid, and of the wave's bias sum of channel `lane`
    for (int64_t v0 = (int64_t)blockIdx.x * kHeadVox; v0 < min(nv, ((int64_t)blockIdx.x + 1) * kHeadVox); v0 += 256) {
        float hs[4] = {0.f, 0.f, 0.f, 0.f}, gs = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t v = v0 + 64 * k + t;
            float m[4] = {0.f, 0.f, 0.f, 0.f};
            if (v < nv) {
                const float g = gy[v];
                const uint2 a = *(const uint2*)(d1 + v * HEAD + 4 * q);
                const float d[4] = {__uint_as_float(a.x << 16), __uint_as_float(a.x & 0xffff0000u),
                                    __uint_as_float(a.y << 16), __uint_as_float(a.y & 0xffff0000u)};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    m[e] = d[e] > 0.f ? g * w[e] : 0.f;
                    hs[e] = __builtin_fmaf(g, d[e], hs[e]);
                }
                gs += g;
                *(uint2*)(gp + v * HEAD + 4 * q) = uint2{pack_bf2(m[0], m[1]), pack_bf2(m[2], m[3])};
            }
            masked[64 * k + t][q] = make_float4(m[0], m[1], m[2], m[3]);
        }
        heads[t][q] = make_float4(hs[0], hs[1], hs[2], hs[3]);
        if (q == 0) ones[t] = gs;
        __syncthreads();
        // the wave's group of 64 voxels: lane (j, q) takes j, j + 16, ..
        float4 own = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 m = masked[64 * wave + 16 * i + (lane >> 2)][lane & 3];
            own.x += m.x;
            own.y += m.y;
            own.z += m.z;
            own.w += m.w;
        }
        bias += group_sum<HEAD>(own, &masked[64 * wave][0]);
        if (tid <= HEAD) {
            float s = 0.f;
#pragma unroll 16
            for (int i = 0; i < 64; ++i) s += tid < HEAD ? ((const float*)&heads[i][0])[tid] : ones[i];
            total += s;
        }
        __syncthreads();
    }
    __shared__ double sums[4][HEAD];
    if (lane < HEAD) sums[wave][lane] = bias;
    __syncthreads();
    double* const row = partial + (int64_t)blockIdx.x * kHeadCols;
    if (tid <= HEAD) row[tid] = total;
    if (tid < HEAD) row[HEAD + 1 + tid] = (sums[0][tid] + sums[1][tid]) + (sums[2][tid] + sums[3][tid]);
}

// x_out = scale * y (scale = s * out_scale), FP64 output
// x (natural order, or split storage with split != 0) = s * out_scale * y
__global__ void k_output(const float* __restrict__ y, const double* __restrict__ ss, double oscale,
                         double* __restrict__ x, int64_t n, int split, int nx, int ny) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n) x[split ? split_pos(v, nx, ny) : v] = (double)y[v] * ss[1] * oscale;
}

__global__ void k_output_minus(const float* __restrict__ y, const double* __restrict__ ss, double oscale,
                               const double* __restrict__ x, double* __restrict__ d, int64_t n) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n) d[v] = (double)y[v] * ss[1] * oscale - x[v];
}

__global__ void k_scaled_grad(const double* __restrict__ q, const double* __restrict__ ss, double oscale,
                              double coef, float* __restrict__ gy, int64_t n) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n) gy[v] = (float)(coef * ss[1] * oscale * q[v]);
}

// target in network units: t = x / (s * out_scale)
__global__ void k_target(const double* __restrict__ x, const double* __restrict__ ss, double oscale,
                         float* __restrict__ t, int64_t n) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n) t[v] = (float)(x[v] / (ss[1] * oscale));
}

// FP32 master parameters -> bf16 forward weights [o][27*cinp] (zero padded channels) and
// backward-data weights [c][27*o] (flipped taps, transposed channels)
__global__ void k_pack(const float* __restrict__ w, int cin, int cinp, int cout,
                       bf16_t* __restrict__ wf, bf16_t* __restrict__ wbk) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;  // over cout * 27 * cinp
    if (idx >= cout * 27 * cinp) return;
    const int c = idx % cinp, t = (idx / cinp) % 27, o = idx / (cinp * 27);
    const float val = c < cin ? w[((int64_t)o * 27 + t) * cin + c] : 0.f;
    const bf16_t h = f2bf(val);
    wf[idx] = h;
    if (c < cin) wbk[((int64_t)c * 27 + (26 - t)) * cout + o] = h;
}

// Adam (Kingma and Ba) with bias correction, FP32 state
__global__ void k_adam(float* __restrict__ th, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int64_t n, float lr, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = 0.9f * m[i] + 0.1f * gi;
    const float vi = 0.999f * v[i] + 0.001f * gi * gi;
    m[i] = mi;
    v[i] = vi;
    th[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
}

__global__ void k_zero_f32(float* x, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = 0.f;
}

// ------------------------------------------------------------------------------------------
// host side

inline unsigned nblk(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

struct Level {
    int nx, ny, nz;
    int64_t nv;
};

}  // namespace hpnn

using namespace hpnn;

constexpr int kGradBufs = 4, kSides = 2;
// Fewest voxels for weight gradients on streams of their own: the events take the host 50 us a step, and below it is the
// host that a step waits for (32 x 64 x 32: 690 us with them, 655 without; 64^3: 750 and 803).
constexpr int64_t kBesideVoxels = 1 << 17;

struct hp_net {
    hipStream_t stream = nullptr;
    Level lv[3];
    int training = 0;
    int64_t nparam = 0;
    int64_t woff[NCONV], boff[NCONV], hoff = 0;  // parameter offsets
    float *theta = nullptr, *grad = nullptr, *m = nullptr, *v = nullptr;
    bf16_t *wf[NCONV] = {}, *wbk[NCONV] = {};
    // activations (bf16): input, conv outputs, pools
    bf16_t* x0 = nullptr;
    bf16_t* act[NCONV] = {};
    bf16_t *p1 = nullptr, *p2 = nullptr;
    float* y = nullptr;
    // training buffers
    float *t = nullptr, *gy = nullptr;
    // masked gradients (bf16) at the layers' outputs, taken in turn: the layer's own in gbuf[cur]. The weight
    // gradients read them on streams of their own, taken in turn, too.
    bf16_t* gbuf[kGradBufs] = {};
    int cur = 0;
    bool beside = false;  // whether they do; two buffers and one wpart otherwise
    hipStream_t side[kSides] = {};
    int turn = 0;
    hipEvent_t ready = nullptr, read[kGradBufs] = {};  // a gradient is written; gbuf[q] has been read
    hipEvent_t test_event = nullptr;                   // (hp_test_nn_beside)
    bool reading[kGradBufs] = {};                      // read[q] has been recorded in this pass
    float *gskip0 = nullptr, *gskip1 = nullptr;  // gradients of e1 and e2 through their skip connections
    float *gp1 = nullptr, *gp2 = nullptr;        // gradients of the pooled tensors
    float* wpart[kSides] = {};  // backward-weight partials
    int64_t wpart_cap = 0;
    double* cpart = nullptr;  // column partials (bias / head)
    float* gfull = nullptr;   // a masked gradient before its rounding (see ConvArgs::full)
    int64_t cpart_cap = 0;
    double* ss = nullptr;     // [sum b^2, s, loss]
    double* dpart = nullptr;
    double out_scale = 1.0;
    int step = 0;
    std::vector<void*> allocs;
};

namespace {

thread_local std::string g_nn_err;

int nfail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_nn_err = buf;
    return code;
}

template <typename T>
int nalloc(hp_net* N, T** p, int64_t n) {
    void* q = nullptr;
    if (hipMalloc(&q, (size_t)std::max<int64_t>(n, 1) * sizeof(T)) != hipSuccess)
        return nfail(HP_ENOMEM, "network workspace allocation of %lld elements failed", (long long)n);
    N->allocs.push_back(q);
    *p = (T*)q;
    return HP_OK;
}

int level_of_conv(int l) {
    static const int lvl[NCONV] = {0, 0, 1, 1, 2, 2, 1, 1, 0, 0};
    return lvl[l];
}

int check() {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return nfail(HP_EHIP, "kernel launch failed: %s", hipGetErrorString(e));
    return HP_OK;
}

// Workgroups of layer l's convolution with `cin` input and `cout` output channels. Two z-slices per
// wave for the 16-channel outputs (more products per staged brick; four were slower: the larger
// brick leaves room for fewer workgroups per CU).
int conv_groups(int cin) { return (cin % 32 == 0) ? 4 : ((cin % 16 == 0) ? 2 : 1); }  // 16-byte groups per chunk voxel
int conv_slices(int cin, int cout) { return (cout == 16 && conv_groups(cin) <= 2) ? 2 : 1; }
unsigned conv_blocks(const Level& L, int cin, int cout) {
    const int fz = 4 * conv_slices(cin, cout);
    return (unsigned)(((L.nx + BX - 1) / BX) * ((L.ny + BY - 1) / BY) * ((L.nz + fz - 1) / fz));
}

template <int CT, int G, int SPW, int OUT>
void conv_start(hp_net* N, const ConvArgs& p, unsigned blocks) {
    hipLaunchKernelGGL((k_conv_fwd<CT, G, SPW, OUT>), dim3(blocks), dim3(256), 0, N->stream, p);
}

// Forward convolution of layer l; with `pool` (16-channel outputs) the launch also writes the 2x2x2
// mean there.
void conv_launch(hp_net* N, int l, const bf16_t* a, int ca, int a_up, const bf16_t* b, int cb,
                 const bf16_t* w, const float* bias, void* out, int cout, const float* head, bf16_t* pool) {
    const Level& L = N->lv[level_of_conv(l)];
    ConvArgs p{a, ca, a_up, b, cb, w, bias, out, cout, L.nx, L.ny, L.nz, 1, head, pool};
    const int cin = ca + cb, g = conv_groups(cin);
    const unsigned blocks = conv_blocks(L, cin, cout);
    switch (cout / 16) {
        case 1:
            if (g == 2) conv_start<1, 2, 2, OUT_ACT>(N, p, blocks);
            else conv_start<1, 1, 2, OUT_ACT>(N, p, blocks);
            break;
        case 2:
            if (g == 4) conv_start<2, 4, 1, OUT_ACT>(N, p, blocks);
            else conv_start<2, 2, 1, OUT_ACT>(N, p, blocks);
            break;
        default: conv_start<4, 4, 1, OUT_ACT>(N, p, blocks); break;
    }
}

// Backward-data convolution of layer l: its masked gradient with the flipped, transposed
// weights. The gradient of its input goes, masked by the ReLU of the layer before it, to `next` and
// gfull (layers 9, 7, 5, 3, 1), for the concatenated inputs of layers 8 and 6 only the upsampled
// part with the skip part in `f32`, and plainly to `f32` for the pooled inputs of layers 4 and 2.
void conv_backward_data(hp_net* N, int l, bf16_t* next, float* f32) {
    const Level& L = N->lv[level_of_conv(l)];
    const unsigned blocks = conv_blocks(L, COUT[l], CIN[l]);
    ConvArgs p{N->gbuf[N->cur], COUT[l], 0, nullptr, 0, N->wbk[l], nullptr, next, CIN[l], L.nx, L.ny, L.nz, 0, nullptr,
               nullptr};
    p.full = N->gfull;
    p.mask = l > 0 ? N->act[l - 1] : nullptr;
    switch (l) {
        case 9:
        case 1: conv_start<1, 2, 2, OUT_GRAD>(N, p, blocks); break;
        case 7:
        case 3: conv_start<2, 4, 1, OUT_GRAD>(N, p, blocks); break;
        case 5: conv_start<4, 4, 1, OUT_GRAD>(N, p, blocks); break;
        case 8:
            p.skip = f32;
            conv_start<3, 2, 1, OUT_CONCAT>(N, p, blocks);
            break;
        case 6:
            p.skip = f32;
            conv_start<6, 4, 1, OUT_CONCAT>(N, p, blocks);
            break;
        case 4:
            p.out = f32;
            conv_start<2, 4, 1, OUT_F32>(N, p, blocks);
            break;
        default:  // 2
            p.out = f32;
            conv_start<1, 4, 1, OUT_F32>(N, p, blocks);
            break;
    }
}

// conv input tensors of layer l in the forward pass
struct ConvIn {
    const bf16_t* a;
    int ca, a_up;
    const bf16_t* b;
    int cb;
};

ConvIn conv_inputs(hp_net* N, int l) {
    switch (l) {
        case 0: return {N->x0, 8, 0, nullptr, 0};
        case 1: return {N->act[0], 16, 0, nullptr, 0};
        case 2: return {N->p1, 16, 0, nullptr, 0};
        case 3: return {N->act[2], 32, 0, nullptr, 0};
        case 4: return {N->p2, 32, 0, nullptr, 0};
        case 5: return {N->act[4], 64, 0, nullptr, 0};
        case 6: return {N->act[5], 64, 1, N->act[3], 32};
        case 7: return {N->act[6], 32, 0, nullptr, 0};
        case 8: return {N->act[7], 32, 1, N->act[1], 16};
        default: return {N->act[8], 16, 0, nullptr, 0};
    }
}

int pack_weights(hp_net* N) {
    for (int l = 0; l < NCONV; ++l) {
        const int n = COUT[l] * 27 * cin_pad(l);
        hipLaunchKernelGGL(k_pack, dim3(nblk(n)), dim3(256), 0, N->stream, N->theta + N->woff[l],
                           CIN[l], cin_pad(l), COUT[l], N->wf[l], N->wbk[l]);
    }
    return check();
}

int forward_net(hp_net* N) {
    for (int l = 0; l < NCONV; ++l) {
        if (l == 4) {
            const Level& L = N->lv[2];
            hipLaunchKernelGGL(k_pool, dim3(nblk(L.nv * 4)), dim3(256), 0, N->stream, N->act[3], N->p2,
                               L.nx, L.ny, L.nz, 32);
        }
        ConvIn in = conv_inputs(N, l);
        // without training the last layer's activation is only needed by the head, which then
        // runs in that convolution's epilogue
        const bool fuse_head = l == NCONV - 1 && !N->training;
        // layer 1 pools in its epilogue
        conv_launch(N, l, in.a, in.ca, in.a_up, in.b, in.cb, N->wf[l], N->theta + N->boff[l],
                    fuse_head ? (void*)N->y : (void*)N->act[l], COUT[l], fuse_head ? N->theta + N->hoff : nullptr,
                    l == 1 ? N->p1 : nullptr);
    }
    if (N->training) {
        const Level& L = N->lv[0];
        hipLaunchKernelGGL(k_head, dim3(nblk(L.nv)), dim3(256), 0, N->stream, N->act[9],
                           N->theta + N->hoff, N->y, L.nv);
    }
    return check();
}

int rhs_scale(hp_net* N, const double* b) {
    const int64_t n = N->lv[0].nv;
    const int nb = 1024;
    hipLaunchKernelGGL(k_sumsq_partial, dim3(nb), dim3(256), 0, N->stream, b, n, N->dpart);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, N->stream, N->dpart, nb, N->ss);
    hipLaunchKernelGGL(k_scale, dim3(1), dim3(1), 0, N->stream, N->ss, (double)n);
    return check();
}

// Orders between the network's stream and those of the weight gradients. Without one, what follows would race: a pass in
// which one fails launches nothing more (see backward_net).
int record(hipEvent_t e, hipStream_t s) { return hipEventRecord(e, s) == hipSuccess ? HP_OK : nfail(HP_EHIP, "event record failed"); }
int wait_for(hipStream_t s, hipEvent_t e) { return hipStreamWaitEvent(s, e, 0) == hipSuccess ? HP_OK : nfail(HP_EHIP, "event wait failed"); }

// The buffer *q for the next masked gradient, once nothing reads it any more.
int next_gradient(hp_net* N, int* q) {
    *q = (N->cur + 1) % (N->beside ? kGradBufs : 2);
    return N->reading[*q] ? wait_for(N->stream, N->read[*q]) : HP_OK;
}

// Weight gradient of layer l from its masked output gradient, beside what follows on the network's stream: its
// workgroups are few (96 at 16 -> 16 channels) and each brick waits for the one before. A step at 128^3
// takes 1941 us so, 2238 in one stream (2105 with one stream for them and three buffers).
int weight_gradient(hp_net* N, int l) {
    hipStream_t side = N->stream;
    int rc;
    if (N->beside) {
        N->turn = (N->turn + 1) % kSides;
        side = N->side[N->turn];
        if ((rc = record(N->ready, N->stream)) || (rc = wait_for(side, N->ready))) return rc;
    }
    const Level& L = N->lv[level_of_conv(l)];
    const int co = COUT[l];
    ConvIn in = conv_inputs(N, l);
    // channel chunks of 16 (the first layer's 8 padded channels read as 8 + 8 zeros)
    const int chunks = (cin_pad(l) + 15) / 16;
    const int nbr = ((L.nx + BX - 1) / BX) * ((L.ny + BY - 1) / BY) * ((L.nz + BZ - 1) / BZ);
    const int parts = std::min(nbr, kBwdWParts);
    BwdWArgs bw{N->gbuf[N->cur], co, in.a, in.ca, in.a_up, in.b, in.cb, N->wpart[N->turn], L.nx, L.ny, L.nz};
    hipLaunchKernelGGL(k_conv_bwd_w, dim3(parts, chunks, co / 16), dim3(kMultipliers + kLoaders), 0, side, bw);
    const int n = co * 27 * CIN[l];
    hipLaunchKernelGGL(k_reduce_dw, dim3(nblk(n, 16)), dim3(256), 0, side, N->wpart[N->turn], parts, chunks, co, CIN[l],
                       N->grad + N->woff[l]);
    if (!N->beside) return HP_OK;
    N->reading[N->cur] = true;
    return record(N->read[N->cur], side);
}

// out[0..c) = column sums of cpart[rows][stride] from column c0 on
void column_sums(hp_net* N, int rows, int stride, int c0, int c, float* out) {
    hipLaunchKernelGGL(k_reduce_cols, dim3(c), dim3(256), 0, N->stream, N->cpart, rows, stride, c0, out);
}

// Backward of layer l from its masked output gradient: its weight gradient, and the
// gradient of its input (see conv_backward_data). Where that is the masked gradient of layer
// l - 1's output, it becomes the current one and that layer's bias gradient is formed.
int backward_conv(hp_net* N, int l, float* f32 = nullptr) {
    int rc = weight_gradient(N, l);
    if (rc || l == 0) return rc;
    const bool pooled = l == 4 || l == 2;
    int q = N->cur;
    if (!pooled && (rc = next_gradient(N, &q))) return rc;
    conv_backward_data(N, l, pooled ? nullptr : N->gbuf[q], f32);
    if (pooled) return HP_OK;
    const int64_t nv = N->lv[level_of_conv(l - 1)].nv;
    const unsigned rows = nblk(nv, kSumVox);
    const int c = COUT[l - 1];
    switch (c) {
        case 16: hipLaunchKernelGGL(k_channel_sums<16>, dim3(rows), dim3(256), 0, N->stream, N->gfull, nv, N->cpart); break;
        case 32: hipLaunchKernelGGL(k_channel_sums<32>, dim3(rows), dim3(256), 0, N->stream, N->gfull, nv, N->cpart); break;
        default: hipLaunchKernelGGL(k_channel_sums<64>, dim3(rows), dim3(256), 0, N->stream, N->gfull, nv, N->cpart); break;
    }
    column_sums(N, (int)rows, c, 0, c, N->grad + N->boff[l - 1]);
    N->cur = q;
    return HP_OK;
}

// Masked gradient of the skip activation of layer l (1 or 3), now the current one, and its bias gradient.
int backward_skip(hp_net* N, int l, const float* g, const float* gpool) {
    const Level& L = N->lv[level_of_conv(l)];
    const unsigned rows = nblk(L.nv, kSumVox);
    auto kernel = l == 1 ? k_relu_bwd_pool<16> : k_relu_bwd_pool<32>;
    int q;
    if (int rc = next_gradient(N, &q)) return rc;
    N->cur = q;
    hipLaunchKernelGGL(kernel, dim3(rows), dim3(256), 0, N->stream, g, gpool, N->act[l], N->gbuf[N->cur], L.nx, L.ny, L.nv,
                       N->cpart);
    column_sums(N, (int)rows, COUT[l], 0, COUT[l], N->grad + N->boff[l]);
    return HP_OK;
}

}  // namespace

// =============================================================================================
// C ABI of the network

extern "C" {

const char* hp_nn_last_error(void) { return g_nn_err.c_str(); }

long long hp_nn_num_params(void) {
    long long n = 0;
    for (int l = 0; l < NCONV; ++l) n += 27LL * CIN[l] * COUT[l] + COUT[l];
    return n + HEAD + 1;
}

void hp_nn_free(hp_net* N) {
    if (!N) return;
    if (N->stream) (void)hipStreamSynchronize(N->stream);
    else (void)hipDeviceSynchronize();
    for (hipStream_t t : N->side)
        if (t) {
            (void)hipStreamSynchronize(t);
            (void)hipStreamDestroy(t);
        }
    if (N->ready) (void)hipEventDestroy(N->ready);
    if (N->test_event) (void)hipEventDestroy(N->test_event);
    for (hipEvent_t e : N->read)
        if (e) (void)hipEventDestroy(e);
    for (void* p : N->allocs) (void)hipFree(p);
    delete N;
}

int hp_nn_create(int nx, int ny, int nz, int training, hp_net** out) {
    g_nn_err.clear();
    if (!out) return nfail(HP_EINVAL, "out must be non-null");
    *out = nullptr;
    if (nx < 4 || ny < 4 || nz < 4 || nx % 4 || ny % 4 || nz % 4)
        return nfail(HP_EINVAL, "network grid sizes must be multiples of 4 (got %d x %d x %d)", nx, ny, nz);
    // the convolutions index voxels with 32-bit integers
    if ((int64_t)nx * ny * nz >= ((int64_t)1 << 31))
        return nfail(HP_EINVAL, "network grid of %d x %d x %d cells exceeds 2^31 - 1 cells", nx, ny, nz);
    hp_net* N = new hp_net();
    N->training = training ? 1 : 0;
    for (int q = 0; q < 3; ++q) {
        N->lv[q].nx = nx >> q;
        N->lv[q].ny = ny >> q;
        N->lv[q].nz = nz >> q;
        N->lv[q].nv = (int64_t)(nx >> q) * (ny >> q) * (nz >> q);
    }
    int64_t off = 0;
    for (int l = 0; l < NCONV; ++l) {
        N->woff[l] = off;
        off += 27LL * CIN[l] * COUT[l];
        N->boff[l] = off;
        off += COUT[l];
    }
    N->hoff = off;
    N->nparam = off + HEAD + 1;
    int rc = HP_OK;
    auto bail = [&](int code) {
        hp_nn_free(N);
        return code;
    };
    if ((rc = nalloc(N, &N->theta, N->nparam))) return bail(rc);
    for (int l = 0; l < NCONV; ++l) {
        if ((rc = nalloc(N, &N->wf[l], (int64_t)COUT[l] * 27 * cin_pad(l))) ||
            (rc = nalloc(N, &N->wbk[l], (int64_t)COUT[l] * 27 * cin_pad(l))))
            return bail(rc);
        if ((rc = nalloc(N, &N->act[l], N->lv[level_of_conv(l)].nv * COUT[l]))) return bail(rc);
    }
    const int64_t V = N->lv[0].nv;
    if ((rc = nalloc(N, &N->x0, V * 8)) || (rc = nalloc(N, &N->p1, N->lv[1].nv * 16)) ||
        (rc = nalloc(N, &N->p2, N->lv[2].nv * 32)) || (rc = nalloc(N, &N->y, V)) ||
        (rc = nalloc(N, &N->ss, 4)) || (rc = nalloc(N, &N->dpart, 1024)))
        return bail(rc);
    if (N->training) {
        if ((rc = nalloc(N, &N->grad, N->nparam)) || (rc = nalloc(N, &N->m, N->nparam)) ||
            (rc = nalloc(N, &N->v, N->nparam)) || (rc = nalloc(N, &N->t, V)) || (rc = nalloc(N, &N->gy, V)))
            return bail(rc);
        const int64_t most = std::max(V * 16, N->lv[1].nv * 32);
        N->beside = V >= kBesideVoxels;
        for (int q = 0; q < (N->beside ? kGradBufs : 2); ++q)
            if ((rc = nalloc(N, &N->gbuf[q], most))) return bail(rc);
        if (N->beside) {
            bool made = hipEventCreateWithFlags(&N->ready, hipEventDisableTiming) == hipSuccess;
            for (hipStream_t& t : N->side) made = made && hipStreamCreateWithFlags(&t, hipStreamNonBlocking) == hipSuccess;
            for (hipEvent_t& e : N->read) made = made && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
            if (!made) return bail(nfail(HP_EHIP, "stream or event creation failed"));
        }
        if ((rc = nalloc(N, &N->gfull, most)) ||
            (rc = nalloc(N, &N->gskip0, V * 16)) || (rc = nalloc(N, &N->gskip1, N->lv[1].nv * 32)) ||
            (rc = nalloc(N, &N->gp1, N->lv[1].nv * 16)) || (rc = nalloc(N, &N->gp2, N->lv[2].nv * 32)))
            return bail(rc);
        for (int l = 0; l < NCONV; ++l)
            N->wpart_cap = std::max(N->wpart_cap, (int64_t)kBwdWParts * ((cin_pad(l) + 15) / 16) * COUT[l] * 27 * 16);
        // channel-sum rows of the head and of the layers
        N->cpart_cap = (int64_t)nblk(V, kHeadVox) * kHeadCols;
        for (int l = 0; l < NCONV; ++l)
            N->cpart_cap = std::max(N->cpart_cap, (int64_t)nblk(N->lv[level_of_conv(l)].nv, kSumVox) * COUT[l]);
        if ((rc = nalloc(N, &N->wpart[0], N->wpart_cap)) || (N->beside && (rc = nalloc(N, &N->wpart[1], N->wpart_cap))) ||
            (rc = nalloc(N, &N->cpart, N->cpart_cap)))
            return bail(rc);
        hipLaunchKernelGGL(k_zero_f32, dim3(nblk(N->nparam)), dim3(256), 0, 0, N->m, N->nparam);
        hipLaunchKernelGGL(k_zero_f32, dim3(nblk(N->nparam)), dim3(256), 0, 0, N->v, N->nparam);
    }
    hipLaunchKernelGGL(k_zero_f32, dim3(nblk(N->nparam)), dim3(256), 0, 0, N->theta, N->nparam);
    if ((rc = check())) return bail(rc);
    if (hipDeviceSynchronize() != hipSuccess) return bail(nfail(HP_EHIP, "device synchronisation failed"));
    *out = N;
    return HP_OK;
}

int hp_nn_set_stream(hp_net* N, void* stream) {
    if (!N) return nfail(HP_EINVAL, "null network");
    N->stream = (hipStream_t)stream;
    return HP_OK;
}

int hp_nn_set_params(hp_net* N, const float* params) {
    if (!N || !params) return nfail(HP_EINVAL, "null argument");
    if (hipMemcpyAsync(N->theta, params, N->nparam * sizeof(float), hipMemcpyDeviceToDevice, N->stream) != hipSuccess)
        return nfail(HP_EHIP, "parameter copy failed");
    return pack_weights(N);
}

int hp_nn_get_params(hp_net* N, float* params) {
    if (!N || !params) return nfail(HP_EINVAL, "null argument");
    if (hipMemcpyAsync(params, N->theta, N->nparam * sizeof(float), hipMemcpyDeviceToDevice, N->stream) != hipSuccess)
        return nfail(HP_EHIP, "parameter copy failed");
    return HP_OK;
}

int hp_nn_get_grad(hp_net* N, float* grad) {
    if (!N || !grad || !N->training) return nfail(HP_EINVAL, "null argument or not a training network");
    if (hipMemcpyAsync(grad, N->grad, N->nparam * sizeof(float), hipMemcpyDeviceToDevice, N->stream) != hipSuccess)
        return nfail(HP_EHIP, "gradient copy failed");
    return HP_OK;
}

static const char kCkptMagic[8] = {'H', 'P', 'N', 'E', 'T', '0', '1', '\0'};

int hp_nn_save(hp_net* N, const char* path) {
    g_nn_err.clear();
    if (!N || !path) return nfail(HP_EINVAL, "null argument");
    std::vector<float> host((size_t)N->nparam);
    if (hipMemcpyAsync(host.data(), N->theta, N->nparam * sizeof(float), hipMemcpyDeviceToHost, N->stream) !=
            hipSuccess ||
        hipStreamSynchronize(N->stream) != hipSuccess)
        return nfail(HP_EHIP, "parameter copy failed");
    FILE* f = std::fopen(path, "wb");
    if (!f) return nfail(HP_EIO, "cannot open %s for writing", path);
    const int64_t count = N->nparam;
    const double scale = N->out_scale;
    bool ok = std::fwrite(kCkptMagic, 1, 8, f) == 8 && std::fwrite(&count, sizeof count, 1, f) == 1 &&
              std::fwrite(&scale, sizeof scale, 1, f) == 1 &&
              std::fwrite(host.data(), sizeof(float), host.size(), f) == host.size();
    ok = (std::fclose(f) == 0) && ok;
    return ok ? HP_OK : nfail(HP_EIO, "cannot write %s", path);
}

int hp_nn_load(hp_net* N, const char* path) {
    g_nn_err.clear();
    if (!N || !path) return nfail(HP_EINVAL, "null argument");
    FILE* f = std::fopen(path, "rb");
    if (!f) return nfail(HP_EIO, "cannot open %s", path);
    char magic[8];
    int64_t count = -1;
    double scale = 0.0;
    bool ok = std::fread(magic, 1, 8, f) == 8 && std::memcmp(magic, kCkptMagic, 8) == 0 &&
              std::fread(&count, sizeof count, 1, f) == 1 && std::fread(&scale, sizeof scale, 1, f) == 1;
    if (!ok || count != N->nparam) {
        std::fclose(f);
        return nfail(HP_EIO, "%s is not a checkpoint of this network (%lld parameters expected)", path,
                     (long long)N->nparam);
    }
    std::vector<float> host((size_t)count);
    ok = std::fread(host.data(), sizeof(float), host.size(), f) == host.size();
    std::fclose(f);
    if (!ok) return nfail(HP_EIO, "%s is truncated", path);
    if (!(scale > 0.0) || !std::isfinite(scale)) return nfail(HP_EIO, "%s holds an invalid output scale", path);
    if (hipMemcpyAsync(N->theta, host.data(), host.size() * sizeof(float), hipMemcpyHostToDevice, N->stream) !=
            hipSuccess ||
        hipStreamSynchronize(N->stream) != hipSuccess)
        return nfail(HP_EHIP, "parameter copy failed");
    N->out_scale = scale;
    return pack_weights(N);
}

int hp_nn_set_output_scale(hp_net* N, double s) {
    if (!N || !(s > 0.0) || !std::isfinite(s)) return nfail(HP_EINVAL, "output scale must be positive");
    N->out_scale = s;
    return HP_OK;
}

// raw network: input features [voxel][8] bf16 -> y [voxel] FP32
int hp_nn_forward_raw(hp_net* N, const unsigned short* in, float* y) {
    if (!N || !in || !y) return nfail(HP_EINVAL, "null argument");
    if (hipMemcpyAsync(N->x0, in, N->lv[0].nv * 8 * sizeof(bf16_t), hipMemcpyDeviceToDevice, N->stream) != hipSuccess)
        return nfail(HP_EHIP, "input copy failed");
    int rc = forward_net(N);
    if (rc) return rc;
    if (hipMemcpyAsync(y, N->y, N->lv[0].nv * sizeof(float), hipMemcpyDeviceToDevice, N->stream) != hipSuccess)
        return nfail(HP_EHIP, "output copy failed");
    return HP_OK;
}

// backward pass from the output gradient in gy (FP32, network units) to the parameter gradient
int backward_net(hp_net* N) {
    N->cur = 0;
    for (bool& r : N->reading) r = false;
    const int64_t V = N->lv[0].nv;
    // head, and the masked gradient of the last layer's output
    const unsigned rows = nblk(V, kHeadVox);
    hipLaunchKernelGGL(k_head_bwd, dim3(rows), dim3(256), 0, N->stream, N->gy, N->act[9], N->theta + N->hoff, N->gbuf[0],
                       V, N->cpart);
    column_sums(N, (int)rows, kHeadCols, 0, HEAD + 1, N->grad + N->hoff);
    column_sums(N, (int)rows, kHeadCols, HEAD + 1, HEAD, N->grad + N->boff[9]);
    // decoder and encoder in reverse
    auto layers = [&]() -> int {
        int rc;
        if ((rc = backward_conv(N, 9))) return rc;
        if ((rc = backward_conv(N, 8, N->gskip0))) return rc;  // [up(act7), act1]
        if ((rc = backward_conv(N, 7))) return rc;
        if ((rc = backward_conv(N, 6, N->gskip1))) return rc;  // [up(act5), act3]
        if ((rc = backward_conv(N, 5))) return rc;
        if ((rc = backward_conv(N, 4, N->gp2))) return rc;
        if ((rc = backward_skip(N, 3, N->gskip1, N->gp2))) return rc;
        if ((rc = backward_conv(N, 3))) return rc;
        if ((rc = backward_conv(N, 2, N->gp1))) return rc;
        if ((rc = backward_skip(N, 1, N->gskip0, N->gp1))) return rc;
        if ((rc = backward_conv(N, 1))) return rc;
        if ((rc = backward_conv(N, 0))) return rc;
        // what follows stands behind the weight gradients, too
        for (hipStream_t t : N->side)
            if (N->beside && ((rc = record(N->ready, t)) || (rc = wait_for(N->stream, N->ready)))) return rc;
        return HP_OK;
    };
    if (const int rc = layers()) {
        for (hipStream_t t : N->side)
            if (N->beside) (void)hipStreamSynchronize(t);
        (void)hipGetLastError();  // reported by rc
        return rc;
    }
    return check();
}

// mean squared error loss and gradient for the input already in x0 and the target in t
int loss_grad(hp_net* N, double* loss) {
    const int64_t V = N->lv[0].nv;
    int rc = forward_net(N);
    if (rc) return rc;
    const int nb = 1024;
    hipLaunchKernelGGL(k_loss, dim3(nb), dim3(256), 0, N->stream, N->y, N->t, N->gy, V, N->dpart);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, N->stream, N->dpart, nb, N->ss + 2);
    if ((rc = backward_net(N))) return rc;
    if (loss) {
        double h[4];
        if (hipMemcpyAsync(h, N->ss, 4 * sizeof(double), hipMemcpyDeviceToHost, N->stream) != hipSuccess ||
            hipStreamSynchronize(N->stream) != hipSuccess)
            return nfail(HP_EHIP, "loss copy failed");
        *loss = h[2] / (double)V;
    }
    return HP_OK;
}

int adam(hp_net* N, float lr) {
    N->step++;
    const float c1 = 1.0f - powf(0.9f, (float)N->step);
    const float c2 = 1.0f - powf(0.999f, (float)N->step);
    hipLaunchKernelGGL(k_adam, dim3(nblk(N->nparam)), dim3(256), 0, N->stream, N->theta, N->grad, N->m,
                       N->v, N->nparam, lr, c1, c2);
    return pack_weights(N);
}

// network input from (b, rho, c2 or m, p_prev): scale, features into x0
int features(hp_net* N, const double* b, const double* rho, const double* c2, const double* m,
             const double* pprev, int split = 0) {
    int rc = rhs_scale(N, b);
    if (rc) return rc;
    const Level& L = N->lv[0];
    hipLaunchKernelGGL(k_features, dim3(nblk(L.nv)), dim3(256), 0, N->stream, b, rho, c2, m, pprev, N->ss,
                       N->x0, L.nv, split, L.nx, L.ny);
    return check();
}

}  // namespace

extern "C" {

// raw loss and gradient: input features [voxel][8] bf16 and target [voxel] FP32 (network
// units); the gradient goes to the network's gradient buffer (hp_nn_get_grad)
int hp_nn_loss_grad_raw(hp_net* N, const unsigned short* in, const float* target, double* loss) {
    if (!N || !in || !target || !N->training) return nfail(HP_EINVAL, "null argument or not a training network");
    const int64_t V = N->lv[0].nv;
    if (hipMemcpyAsync(N->x0, in, V * 8 * sizeof(bf16_t), hipMemcpyDeviceToDevice, N->stream) != hipSuccess ||
        hipMemcpyAsync(N->t, target, V * sizeof(float), hipMemcpyDeviceToDevice, N->stream) != hipSuccess)
        return nfail(HP_EHIP, "input copy failed");
    return loss_grad(N, loss);
}

// Not part of the interface, for tests. how = 0: the weight gradients of a network that has streams for them run on its own
// stream; 1: on those streams (as it is created); 2: the same with an event that can't be recorded. Between passes
// only; returns whether the network has such streams.
int hp_test_nn_beside(hp_net* N, int how) {
    if (!N->side[0]) return 0;
    if (!N->ready) std::swap(N->ready, N->test_event);
    if (how == 2) std::swap(N->ready, N->test_event);
    N->beside = how != 0;
    return 1;
}

int hp_nn_adam(hp_net* N, float lr) {
    if (!N || !N->training) return nfail(HP_EINVAL, "not a training network");
    if (!(lr > 0.f)) return nfail(HP_EINVAL, "learning rate must be positive");
    return adam(N, lr);
}

int hp_nn_forward(hp_net* N, const double* b, const double* rho, const double* c2,
                  const double* p_prev, double* x) {
    if (!N || !b || !rho || !c2 || !x) return nfail(HP_EINVAL, "null argument");
    int rc = features(N, b, rho, c2, nullptr, p_prev);
    if (rc) return rc;
    if ((rc = forward_net(N))) return rc;
    const int64_t V = N->lv[0].nv;
    hipLaunchKernelGGL(k_output, dim3(nblk(V)), dim3(256), 0, N->stream, N->y, N->ss, N->out_scale, x, V, 0,
                       N->lv[0].nx, N->lv[0].ny);
    return check();
}

int hp_nn_train_step(hp_net* N, const double* b, const double* rho, const double* c2,
                     const double* p_prev, const double* x_target, float lr, double* loss) {
    if (!N || !b || !rho || !c2 || !x_target || !N->training)
        return nfail(HP_EINVAL, "null argument or not a training network");
    if (!(lr > 0.f)) return nfail(HP_EINVAL, "learning rate must be positive");
    int rc = features(N, b, rho, c2, nullptr, p_prev);
    if (rc) return rc;
    const int64_t V = N->lv[0].nv;
    hipLaunchKernelGGL(k_target, dim3(nblk(V)), dim3(256), 0, N->stream, x_target, N->ss, N->out_scale,
                       N->t, V);
    if ((rc = loss_grad(N, loss))) return rc;
    return adam(N, lr);
}

}  // extern "C"

// ---- used by the solver's learned mode (hp_solver.hip) ----
namespace hp {
int nn_grid(const hp_net* N, int* nx, int* ny, int* nz) {
    *nx = N->lv[0].nx;
    *ny = N->lv[0].ny;
    *nz = N->lv[0].nz;
    return HP_OK;
}
// z = s * out_scale * net(r / s, log rho, -log(rho m), p_prev / s), s = RMS(r)
int nn_apply(hp_net* N, hipStream_t stream, const double* r, const double* rho, const double* m,
             const double* pprev, double* z, int split) {
    N->stream = stream;
    int rc = features(N, r, rho, nullptr, m, pprev, split);
    if (rc) return rc;
    if ((rc = forward_net(N))) return rc;
    const Level& L = N->lv[0];
    hipLaunchKernelGGL(k_output, dim3(nblk(L.nv)), dim3(256), 0, N->stream, N->y, N->ss, N->out_scale, z, L.nv,
                       split, L.nx, L.ny);
    return check();
}
const char* nn_error() { return g_nn_err.c_str(); }

int nn_train_forward(hp_net* N, hipStream_t stream, const double* b, const double* rho,
                     const double* m, const double* pprev) {
    if (!N->training) return nfail(HP_EINVAL, "not a training network");
    N->stream = stream;
    int rc = features(N, b, rho, nullptr, m, pprev);
    if (rc) return rc;
    return forward_net(N);
}

// d = s * out_scale * y - x (physical units, FP64)
int nn_output_minus(hp_net* N, const double* x, double* d) {
    const int64_t V = N->lv[0].nv;
    hipLaunchKernelGGL(k_output_minus, dim3(nblk(V)), dim3(256), 0, N->stream, N->y, N->ss, N->out_scale,
                       x, d, V);
    return check();
}

// gy = coef * s * out_scale * q  (chain rule from physical to network units), then backward + Adam
int nn_train_backward(hp_net* N, const double* q, double coef, float lr) {
    const int64_t V = N->lv[0].nv;
    hipLaunchKernelGGL(k_scaled_grad, dim3(nblk(V)), dim3(256), 0, N->stream, q, N->ss, N->out_scale, coef,
                       N->gy, V);
    int rc = backward_net(N);
    if (rc) return rc;
    return adam(N, lr);
}
}  // namespace hp
