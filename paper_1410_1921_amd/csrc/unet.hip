// Layers of the warm-start U-Net: 3x3x3 convolution (forward, input gradient, weight
// gradient) as implicit GEMMs on the bf16 matrix cores, 2x2x2 mean pooling, nearest
// upsampling, the ReLU gradient, the 1x1x1 output head with its masked squared-error
// loss, Adam, and the conversions between the solver's fields and network tensors.
//
// Tensors are channels-last bf16: element (voxel v, channel c) at v * cs + c, with v =
// x + nx (y + ny z); a view is a pointer to its first channel plus the channel stride cs,
// so the [skip, upsampled] concatenation of a decoder input is two views of one buffer.
// Weights are [27][cout][cin], tap t = 9 (dz + 1) + 3 (dy + 1) + (dx + 1); products
// accumulate in binary32.
#include <algorithm>
#include <type_traits>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <initializer_list>

#include "../../include/lbm_nn.h"
#include "lbm_internal.h"

namespace lbm {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// binary32 -> bfloat16, round to nearest even (finite inputs)
__device__ inline uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// D = A B + C for 16x16 tiles, K = 16.  Lane l = 16 q + r holds A[m = r][k = 4q .. 4q+3],
// B[k = 4q .. 4q+3][n = r] and D[m = 4q .. 4q+3][n = r].
__device__ inline f32x4 mfma16(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// The same with K = 32: lanes hold k = 8 q .. 8 q + 7.
__device__ inline f32x4 mfma32(bf16x8 a, bf16x8 b, f32x4 c) {
    typedef __bf16 v8 __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8, a), __builtin_bit_cast(v8, b), c, 0, 0, 0);
}
__device__ inline bf16x8 join(bf16x4 a, bf16x4 b) {
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

struct NnGrid {
    int nx, ny, nz;
    int64_t nvox;
};

__device__ inline void tap_offset(int t, int flip, int &dx, int &dy, int &dz) {
    dz = t / 9 - 1;
    dy = (t / 3) % 3 - 1;
    dx = t % 3 - 1;
    if (flip) {
        dx = -dx;
        dy = -dy;
        dz = -dz;
    }
}

// y[v][c] = act(bias[c] + sum_t sum_k x[v + d_t][k] w[t][c][k]) for NB blocks of 16
// output channels; d_t negated with flip.  One wave per 16 consecutive voxels.
template <int NB>
__global__ __launch_bounds__(256) void k_conv3d(NnGrid g, const uint16_t *__restrict__ x, int x_cs,
                                                int cin, const uint16_t *__restrict__ w,
                                                const float *__restrict__ bias,
                                                uint16_t *__restrict__ y, int y_cs, int relu,
                                                int flip) {
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int64_t m0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
    if (m0 >= g.nvox) return;  // uniform per wave; nvox is a multiple of 16
    const int64_t va = m0 + r;
    const int ax = (int)(va % g.nx), ay = (int)((va / g.nx) % g.ny), az = (int)(va / ((int64_t)g.nx * g.ny));
    const int cout = NB * 16;
    f32x4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; nb++) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int t = 0; t < 27; t++) {
        int dx, dy, dz;
        tap_offset(t, flip, dx, dy, dz);
        const int sx = ax + dx, sy = ay + dy, sz = az + dz;
        const bool ok = sx >= 0 && sx < g.nx && sy >= 0 && sy < g.ny && sz >= 0 && sz < g.nz;
        const int64_t sv = ok ? ((int64_t)sz * g.ny + sy) * g.nx + sx : 0;
        const uint16_t *xp = x + sv * x_cs + 4 * q;
        const uint16_t *wp = w + ((int64_t)t * cout + r) * cin + 4 * q;
        for (int kc = 0; kc < cin; kc += 16) {
            const bf16x4 a = ok ? *reinterpret_cast<const bf16x4 *>(xp + kc) : bf16x4{0, 0, 0, 0};
#pragma unroll
            for (int nb = 0; nb < NB; nb++) {
                const bf16x4 b = *reinterpret_cast<const bf16x4 *>(wp + (int64_t)nb * 16 * cin + kc);
                acc[nb] = mfma16(a, b, acc[nb]);
            }
        }
    }
#pragma unroll
    for (int nb = 0; nb < NB; nb++) {
        const int c = nb * 16 + r;
        const float bc = bias ? bias[c] : 0.f;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float v = acc[nb][j] + bc;
            if (relu) v = v > 0.f ? v : 0.f;
            y[(m0 + 4 * q + j) * y_cs + c] = f2bf(v);
        }
    }
}

// The same convolution on grids whose three sizes are multiples of 4: a workgroup of
// WX x WY x WZ = 4 waves, one block of 16 output channels, and a brick of 4 WX x 4 WY x
// PZ WZ voxels, of which each wave holds a column of PZ planes of 4 x 4.  Per block of 16
// input channels the workgroup copies its halo of x (zero outside the grid) and the block's
// 27 x 16 x 16 weights into LDS, with 16-byte loads issued during the previous block's
// products.
//
// What would bound it is the LDS operand read: 8 bytes a lane are 4 cycles of the unit that
// four matrix cores share, a product 16 cycles of one of them.  So a wave keeps the 27
// weights in registers and walks the input planes of its column in the order of the taps'
// z: each of a plane's nine shifted operands is read once and multiplied into the three
// output planes it touches, 9 (PZ + 2) reads for 27 PZ products.  The reads are free of
// conflicts: the four channel quads lie in planes of their own, 8 bytes a voxel, rows padded
// to 12 voxels, which puts the 16 voxels of a tile into 16 different pairs of banks.  The
// weights are the A operand, so that a lane ends with four channels of one voxel and writes
// them with one 8-byte store.  Every output adds its products in one order, whatever the
// brick: input block, then tap.
//
// Measured, a wave per 4 x 4 x 4 brick that read both operands for every product before:
// 96^3 x 16 -> 16 channels 50.8 -> 31 us, 96^3 x 48 -> 16 137 -> 65, 48^3 x 96 -> 32 83 -> 35,
// 24^3 x 192 -> 64 73 -> 24, 12^3 x 128 -> 128 46 -> 12; 390 to 560 of the 1260 TFLOP/s of the
// 16 x 16 x 16 products on the 96^3 levels, the matrix cores busy half of the time: what is
// left is a workgroup's start, when halo and weights are on their way while only one other
// workgroup of the compute unit works.
typedef uint32_t u32x4a8 __attribute__((ext_vector_type(4), aligned(8)));  // 16 bytes at 8
template <int WX, int WY, int WZ, int PZ, bool FLIP>
__global__ __launch_bounds__(256) void k_conv3d_bricks(NnGrid g, const uint16_t *__restrict__ x, int x_cs,
                                                       int cin, const uint16_t *__restrict__ w,
                                                       int cout, const float *__restrict__ bias,
                                                       uint16_t *__restrict__ y, int y_cs, int relu) {
    constexpr int TX = 4 * WX, TY = 4 * WY, TZ = PZ * WZ;
    constexpr int HX = TX + 2, HY = TY + 2, HZ = TZ + 2, RS = 12;  // halo; row stride in voxels
    constexpr int QS = RS * HY * HZ;                               // voxels of a quad plane
    constexpr int NCP = HX * HY * 2, PP = 256 / NCP;  // 16-byte chunks of a halo plane; planes at once
    constexpr int PER = (HZ + PP - 1) / PP;
    constexpr int NWT = 27 * 32, WPER = (NWT + 255) / 256;         // 16-byte chunks of the weights
    static_assert(WX * WY * WZ == 4 && TX <= 8, "four waves, rows of at most 10 voxels");
    __shared__ __align__(16) uint16_t sx[4 * QS * 4];       // [quad][voxel][4 channels]
    __shared__ __align__(16) uint16_t sw[27 * 4 * 16 * 4];  // [tap][quad][out channel][4 channels]
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bx = (g.nx + TX - 1) / TX, by = (g.ny + TY - 1) / TY;
    const int b = (int)xcd_block(blockIdx.x, gridDim.x / kXcd), c0 = (int)blockIdx.y * 16;
    if (b >= bx * by * ((g.nz + TZ - 1) / TZ)) return;
    const int x0 = TX * (b % bx), y0 = TY * ((b / bx) % by), z0 = TZ * (b / (bx * by));
    // the thread's chunks of the halo: one place in the plane, half (8 channels) of its 16, in
    // the planes hz, hz + PP, ..
    const int hc = tid % NCP, hz = tid / NCP, hx = (hc >> 1) % HX, hy = (hc >> 1) / HX;
    const int sxv = x0 - 1 + hx, syv = y0 - 1 + hy, szv = z0 - 1 + hz;
    const bool inside = hz < PP && sxv >= 0 && sxv < g.nx && syv >= 0 && syv < g.ny;
    // addresses as one scalar base per load and one lane offset for all of them: in 32 bits
    // where a thread stays in one plane (10 rows of a tensor: lbm_nn_conv3d sees to the limit)
    typedef typename std::conditional<PP == 1, uint32_t, int64_t>::type LaneOff;
    const int64_t plane = (int64_t)g.nx * g.ny * x_cs;
    const uint16_t *const src = x + (z0 - 1) * plane + ((int64_t)(y0 - 1) * g.nx + x0 - 1) * x_cs;
    const LaneOff so = (LaneOff)((PP == 1 ? 0 : hz * plane) + ((int64_t)hy * g.nx + hx) * x_cs + 8 * (hc & 1));
    const uint32_t wo = (uint32_t)(((tid >> 5) * cout + ((tid >> 1) & 15)) * cin + 8 * (tid & 1));
    uint16_t *const dst = sx + (2 * (hc & 1) * QS + (hz * HY + hy) * RS + hx) * 4;
    uint4 pre[PER];
    u32x4a8 wpre[WPER];
    auto load_block = [&](int kc) {
#pragma unroll
        for (int k = 0; k < PER; k++) {
            const int vz = szv + PP * k;
            pre[k] = uint4{0u, 0u, 0u, 0u};
            if (inside && hz + PP * k < HZ && vz >= 0 && vz < g.nz)
                pre[k] = *reinterpret_cast<const uint4 *>(src + PP * k * plane + kc + so);
        }
#pragma unroll
        for (int k = 0; k < WPER; k++) {
            if (tid + 256 * k < NWT)  // 8 taps at once; out channel, half
                wpre[k] = *reinterpret_cast<const u32x4a8 *>(w + ((int64_t)8 * k * cout + c0) * cin + kc + wo);
        }
    };
    auto store_block = [&]() {
#pragma unroll
        for (int k = 0; k < PER; k++) {
            if (hz < PP && hz + PP * k < HZ) {
                uint16_t *d = dst + PP * k * HY * RS * 4;
                *reinterpret_cast<uint2 *>(d) = uint2{pre[k].x, pre[k].y};
                *reinterpret_cast<uint2 *>(d + 4 * QS) = uint2{pre[k].z, pre[k].w};
            }
        }
#pragma unroll
        for (int k = 0; k < WPER; k++) {
            const int c = tid + 256 * k;
            if (c < NWT) {
                uint16_t *d = sw + (((c >> 5) * 4 + 2 * (c & 1)) * 16 + ((c >> 1) & 15)) * 4;
                *reinterpret_cast<uint2 *>(d) = uint2{wpre[k].x, wpre[k].y};
                *reinterpret_cast<uint2 *>(d + 64) = uint2{wpre[k].z, wpre[k].w};
            }
        }
    };
    const int tx = wave % WX, ty = (wave / WX) % WY, tz = wave / (WX * WY) * PZ;
    // element offset in sx of the lane's voxel of the column's lowest input plane, quad q
    const int base = (q * QS + (tz * HY + ty * 4 + (r >> 2) + 1) * RS + tx * 4 + (r & 3) + 1) * 4;
    f32x4 acc[PZ];
#pragma unroll
    for (int p = 0; p < PZ; p++) acc[p] = f32x4{0.f, 0.f, 0.f, 0.f};
    load_block(0);
    for (int kc = 0; kc < cin; kc += 16) {
        if (kc) __syncthreads();  // the previous channel block's operands are read
        store_block();
        __syncthreads();
        if (kc + 16 < cin) load_block(kc + 16);
        bf16x4 wv[27];  // A[m = r][k = 4 q .. 4 q + 3]
#pragma unroll
        for (int t = 0; t < 27; t++) wv[t] = *reinterpret_cast<const bf16x4 *>(sw + (t * 64 + lane) * 4);
#pragma unroll
        for (int i = 0; i < PZ + 2; i++) {  // input planes, upwards, or downwards for the mirrored taps
            const int h = FLIP ? PZ + 1 - i : i;
            bf16x4 av[9];  // B[k = 4 q .. 4 q + 3][n = r]
#pragma unroll
            for (int u = 0; u < 9; u++) {
                const int off = (FLIP ? -1 : 1) * (u % 3 - 1 + RS * (u / 3 - 1));
                av[u] = *reinterpret_cast<const bf16x4 *>(sx + base + (h * HY * RS + off) * 4);
            }
#pragma unroll
            for (int u = 0; u < 9; u++)
#pragma unroll
                for (int dz = 0; dz < 3; dz++) {
                    const int p = FLIP ? h + dz - 2 : h - dz;  // the output plane of tap dz
                    if (p >= 0 && p < PZ) acc[p] = mfma16(wv[dz * 9 + u], av[u], acc[p]);
                }
        }
    }
    // D[m = 4 q + j][n = r]: output channel c0 + 4 q + j, voxel (r & 3, r >> 2) of the plane
    const int vx = x0 + tx * 4, vy = y0 + ty * 4;
    if (vx >= g.nx || vy >= g.ny) return;
    const bool wide = y_cs % 4 == 0 && reinterpret_cast<uintptr_t>(y) % 8 == 0;
    const uint32_t yo = (uint32_t)(((r >> 2) * g.nx + (r & 3)) * y_cs + 4 * q);
    float bc[4];
#pragma unroll
    for (int j = 0; j < 4; j++) bc[j] = bias ? bias[c0 + 4 * q + j] : 0.f;
#pragma unroll
    for (int p = 0; p < PZ; p++) {
        const int vz = z0 + tz + p;
        if (vz >= g.nz) break;
        uint32_t o[2];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            float v = acc[p][j] + bc[j];
            if (relu) v = v > 0.f ? v : 0.f;
            const uint32_t h = f2bf(v);
            o[j >> 1] = j & 1 ? o[j >> 1] | h << 16 : h;
        }
        uint16_t *d = y + (((int64_t)vz * g.ny + vy) * g.nx + vx) * y_cs + c0 + yo;
        if (wide) {
            *reinterpret_cast<uint2 *>(d) = uint2{o[0], o[1]};
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++) d[j] = (uint16_t)(o[j >> 1] >> (j & 1) * 16);
        }
    }
}

// Partial weight gradients over one chunk of voxels for tap t = blockIdx.y and output
// block cb = blockIdx.z: part[chunk][t][co][ci] = sum_v g[v][co] x[v + d_t][ci] for
// NBI blocks of 16 input channels; the centre tap also forms part_b[chunk][co] = sum_v
// g[v][co].  One wave per block.
template <int NBI>
__global__ __launch_bounds__(64) void k_conv3d_wgrad(NnGrid g, const uint16_t *__restrict__ x,
                                                     int x_cs, const uint16_t *__restrict__ gy,
                                                     int g_cs, int cout, int64_t chunk,
                                                     float *__restrict__ part,
                                                     float *__restrict__ part_b) {
    const int lane = threadIdx.x, r = lane & 15, q = lane >> 4;
    const int64_t ch = blockIdx.x;
    const int t = blockIdx.y, cb = blockIdx.z;
    const int cin = NBI * 16;
    int dx, dy, dz;
    tap_offset(t, 0, dx, dy, dz);
    const int64_t v_lo = ch * chunk, v_hi = v_lo + chunk < g.nvox ? v_lo + chunk : g.nvox;
    f32x4 acc[NBI];
#pragma unroll
    for (int ib = 0; ib < NBI; ib++) acc[ib] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 accb = f32x4{0.f, 0.f, 0.f, 0.f};
    const short one = (short)0x3f80;  // bfloat16 1.0
    const bf16x4 ones = bf16x4{one, one, one, one};
    for (int64_t v0 = v_lo; v0 < v_hi; v0 += 16) {
        bf16x4 a;
        int64_t src[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int64_t v = v0 + 4 * q + j;
            a[j] = (short)gy[v * g_cs + cb * 16 + r];
            const int vx = (int)(v % g.nx), vy = (int)((v / g.nx) % g.ny), vz = (int)(v / ((int64_t)g.nx * g.ny));
            const int sx = vx + dx, sy = vy + dy, sz = vz + dz;
            src[j] = sx >= 0 && sx < g.nx && sy >= 0 && sy < g.ny && sz >= 0 && sz < g.nz
                         ? ((int64_t)sz * g.ny + sy) * g.nx + sx
                         : -1;
        }
#pragma unroll
        for (int ib = 0; ib < NBI; ib++) {
            bf16x4 b;
#pragma unroll
            for (int j = 0; j < 4; j++) b[j] = src[j] >= 0 ? (short)x[src[j] * x_cs + ib * 16 + r] : (short)0;
            acc[ib] = mfma16(a, b, acc[ib]);
        }
        if (t == 13) accb = mfma16(a, ones, accb);
    }
#pragma unroll
    for (int ib = 0; ib < NBI; ib++)
#pragma unroll
        for (int j = 0; j < 4; j++)
            part[((ch * 27 + t) * cout + cb * 16 + 4 * q + j) * cin + ib * 16 + r] = acc[ib][j];
    if (t == 13 && r == 0)
#pragma unroll
        for (int j = 0; j < 4; j++) part_b[ch * cout + cb * 16 + 4 * q + j] = accb[j];
}

// Four values of one channel at four consecutive voxels, out of LDS rows of 16 channels: the
// 16 lanes of a group read a 4 x 16 block, 8 bytes each in memory order, and lane r receives
// its column r.
__device__ __forceinline__ bf16x4 read_column4(const uint16_t *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) bf16x4 *)p);
}

// The same weight gradient on grids whose three sizes are multiples of 4: a workgroup of four
// waves owns one chunk of bricks of 8 x 8 x 4 voxels (blockIdx.x), one block of 16 output
// channels and one of 16 input channels (blockIdx.y), and all 27 taps; each wave takes a
// column of 4 x 4 x 4 of every brick (none where the brick is cut by the grid's upper x or y
// side).  The brick's gy and the halo of x around it (zero outside the grid) are loaded
// during the previous brick's products and go to LDS as they lie in memory, 16 channels a
// voxel.
//
// A product sums over K = 32 voxels, two z planes of a column, so both operands run across
// voxels: read_column4 turns them on their way out of LDS (2-byte reads, four for every
// operand, were what this took its time for).  Per (dx, dy) the six input planes are read
// once and used for all three dz, 54 reads for 54 products of 16 cycles.  The four waves'
// sums are added through LDS at the end, in one order, so that a workgroup writes one partial
// row.
//
// Measured with the sum of the rows, a wave per 4 x 4 x 4 brick with K = 16 before: 96^3 x 16 ->
// 16 channels 101 -> 33 us, 96^3 x 48 -> 16 182 -> 94, 48^3 x 96 -> 32 88 -> 36, 24^3 x 192 -> 64
// 83 -> 33, 12^3 x 128 -> 128 92 -> 24.  Vector work beside the products (addresses, registers
// moved for the overlapping pairs of planes) and the staging are what is left; the products
// alone would take 5 us of the first.
__global__ __launch_bounds__(256, 2) void k_conv3d_wgrad_bricks(NnGrid g, const uint16_t *__restrict__ x,
                                                                int x_cs, int cin,
                                                                const uint16_t *__restrict__ gy,
                                                                int g_cs, int cout, int bricks, int nb,
                                                                float *__restrict__ part,
                                                                float *__restrict__ part_b) {
    constexpr int H = 10, HN = H * H * 6;            // halo voxels in x and y, in all
    constexpr int NCP = 2 * H * H;                   // 16-byte chunks of a halo plane
    constexpr int SUM = 28 * 256;                    // a wave's sums: 27 taps and gy's own
    __shared__ __align__(16) float lds[2 * SUM];
    uint16_t *const sx = reinterpret_cast<uint16_t *>(lds), *const sg = sx + HN * 16;
    static_assert((HN + 256) * 16 * 2 <= 2 * SUM * 4, "halo and gy lie in the sums' memory");
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wx = wave & 1, wy = wave >> 1;
    const int64_t ch = blockIdx.x;
    const int ncb = cout / 16;
    const int cb = (int)blockIdx.y % ncb, ib = (int)blockIdx.y / ncb;
    const int bx = (g.nx + 7) / 8, by = (g.ny + 7) / 8;
    const int b_lo = (int)ch * bricks, b_hi = b_lo + bricks < nb ? b_lo + bricks : nb;
    // the thread's chunks: half (8 channels) of one voxel of a plane, in each plane of the halo
    // and in every other plane of gy
    const int hc = tid % NCP, hx = (hc >> 1) % H - 1, hy = (hc >> 1) / H - 1;
    const int gxv = (tid >> 1) & 7, gyv = (tid >> 4) & 7, gzv = tid >> 7;
    const int64_t xplane = (int64_t)g.nx * g.ny * x_cs, gplane = (int64_t)g.nx * g.ny * g_cs;
    const uint16_t *const xs = x + ((int64_t)hy * g.nx + hx) * x_cs + ib * 16 + 8 * (hc & 1);
    const uint16_t *const gs = gy + gzv * gplane + ((int64_t)gyv * g.nx + gxv) * g_cs + cb * 16 + 8 * (tid & 1);
    uint4 px[6], pg[2];
    auto load_brick = [&](int x0, int y0, int z0) {
        const int64_t o = ((int64_t)z0 * g.ny + y0) * g.nx + x0;  // the brick's first voxel
        const bool in_g = x0 + gxv < g.nx && y0 + gyv < g.ny;
        const bool in_x = tid < NCP && x0 + hx >= 0 && x0 + hx < g.nx && y0 + hy >= 0 && y0 + hy < g.ny;
#pragma unroll
        for (int k = 0; k < 2; k++) pg[k] = uint4{0u, 0u, 0u, 0u};
        if (in_g)
#pragma unroll
            for (int k = 0; k < 2; k++)
                pg[k] = *reinterpret_cast<const uint4 *>(gs + o * g_cs + 2 * k * gplane);
#pragma unroll
        for (int k = 0; k < 6; k++) px[k] = uint4{0u, 0u, 0u, 0u};
        if (in_x) {
#pragma unroll
            for (int k = 0; k < 6; k++)
                if (z0 - 1 + k >= 0 && z0 - 1 + k < g.nz)
                    px[k] = *reinterpret_cast<const uint4 *>(xs + o * x_cs + (k - 1) * xplane);
        }
    };
    f32x4 acc[28];
#pragma unroll
    for (int t = 0; t < 28; t++) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const short one = (short)0x3f80;  // bfloat16 1.0
    const bf16x8 ones = bf16x8{one, one, one, one, one, one, one, one};
    // lane's address inside a 4 x 16 block: voxel r / 4 of the row, channels 4 (r % 4) ..
    const uint16_t *const ga = sg + ((wy * 4 + q) * 8 + wx * 4 + (r >> 2)) * 16 + 4 * (r & 3);
    const uint16_t *const xa = sx + ((wy * 4 + q + 1) * H + wx * 4 + (r >> 2) + 1) * 16 + 4 * (r & 3);
    int x0 = 8 * (b_lo % bx), y0 = 8 * ((b_lo / bx) % by), z0 = 4 * (b_lo / (bx * by));
    load_brick(x0, y0, z0);
    for (int b = b_lo; b < b_hi; b++) {
        const bool column = x0 + 4 * wx < g.nx && y0 + 4 * wy < g.ny;
        __syncthreads();  // the previous brick's operands are read
#pragma unroll
        for (int k = 0; k < 2; k++) *reinterpret_cast<uint4 *>(sg + (tid + 256 * k) * 8) = pg[k];
#pragma unroll
        for (int k = 0; k < 6; k++)
            if (tid < NCP) *reinterpret_cast<uint4 *>(sx + (tid + NCP * k) * 8) = px[k];
        __syncthreads();
        x0 += 8;
        if (x0 >= g.nx) x0 = 0, y0 += 8;
        if (y0 >= g.ny) y0 = 0, z0 += 4;
        if (b + 1 < b_hi) load_brick(x0, y0, z0);
        if (!column) continue;
        // A[m = output channel r][k = 8 q + 4 e + j] = gy at voxel (j, q) of plane 2 i + e
        bf16x8 a[2];
#pragma unroll
        for (int i = 0; i < 2; i++)
            a[i] = join(read_column4(ga + 2 * i * 64 * 16), read_column4(ga + (2 * i + 1) * 64 * 16));
        if (ib == 0)
#pragma unroll
            for (int i = 0; i < 2; i++) acc[27] = mfma32(a[i], ones, acc[27]);
#pragma unroll
        for (int u = 0; u < 9; u++) {
            // B[k][n = input channel r] = x at that voxel + (dx, dy, dz)
            bf16x4 bv[6];
#pragma unroll
            for (int h = 0; h < 6; h++)
                bv[h] = read_column4(xa + (h * H * H + (u / 3 - 1) * H + u % 3 - 1) * 16);
#pragma unroll
            for (int i = 0; i < 2; i++)
#pragma unroll
                for (int dz = 0; dz < 3; dz++)
                    acc[dz * 9 + u] = mfma32(a[i], join(bv[2 * i + dz], bv[2 * i + dz + 1]), acc[dz * 9 + u]);
        }
    }
    // the four waves' sums: waves 2 and 3 to 0 and 1, then 1 to 0
#pragma unroll
    for (int half = 2; half >= 1; half >>= 1) {
        __syncthreads();
        float *const m = lds + (wave & (half - 1)) * SUM + 4 * lane;
        if (wave >= half && wave < 2 * half)
#pragma unroll
            for (int t = 0; t < 28; t++) *reinterpret_cast<f32x4 *>(m + t * 256) = acc[t];
        __syncthreads();
        if (wave < half)
#pragma unroll
            for (int t = 0; t < 28; t++) acc[t] += *reinterpret_cast<const f32x4 *>(m + t * 256);
    }
    if (wave) return;
#pragma unroll
    for (int t = 0; t < 27; t++)
#pragma unroll
        for (int j = 0; j < 4; j++)
            part[((ch * 27 + t) * cout + cb * 16 + 4 * q + j) * cin + ib * 16 + r] = acc[t][j];
    if (ib == 0 && r == 0)
#pragma unroll
        for (int j = 0; j < 4; j++) part_b[ch * cout + cb * 16 + 4 * q + j] = acc[27][j];
}

// out[i] (+)= sum_c part[c * count + i] over c = 0 .. nparts - 1 for i < count, and the same
// of part_b into out_b for the n_b outputs of the bias, which the blocks from nblk on work
// (none: n_b = 0), in a fixed order: G threads per four outputs each sum one contiguous
// G-th of the partials in order, then the G sums are added in order.  Count and n_b are
// multiples of 16, so a group of four is whole; it is read with 16 bytes a lane.
template <int G>
__global__ __launch_bounds__(256) void k_sum_parts(const float *__restrict__ part, int64_t nparts,
                                                   int64_t count, float *__restrict__ out,
                                                   const float *__restrict__ part_b, int n_b,
                                                   float *__restrict__ out_b, unsigned nblk,
                                                   int accumulate) {
    constexpr int O = 256 / G;
    __shared__ f32x4 lds[G][O + 1];
    unsigned blk = blockIdx.x;
    if (blk >= nblk) blk -= nblk, part = part_b, count = n_b, out = out_b;
    const int o = threadIdx.x % O, gr = threadIdx.x / O;
    const int64_t i = ((int64_t)blk * O + o) * 4;
    const int64_t per = (nparts + G - 1) / G;
    const int64_t c0 = gr * per, c1 = c0 + per < nparts ? c0 + per : nparts;
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
    if (i < count)
#pragma unroll 4
        for (int64_t c = c0; c < c1; c++) s += *reinterpret_cast<const f32x4 *>(part + c * count + i);
    lds[gr][o] = s;
    __syncthreads();
    if (gr == 0 && i < count) {
        f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < G; k++) t += lds[k][o];
#pragma unroll
        for (int j = 0; j < 4; j++) out[i + j] = accumulate ? out[i + j] + t[j] : t[j];
    }
}

// wt[t][ci][co] = w[t][co][ci] (bf16), the weights of the input-gradient convolution.
__global__ __launch_bounds__(256) void k_transpose_w(const uint16_t *__restrict__ w, int cout,
                                                     int cin, uint16_t *__restrict__ wt) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t n = (int64_t)27 * cout * cin;
    if (i >= n) return;
    const int64_t t = i / ((int64_t)cout * cin), rem = i % ((int64_t)cout * cin);
    const int co = (int)(rem / cin), ci = (int)(rem % cin);
    wt[(t * cin + ci) * cout + co] = w[i];
}

// The elementwise layers take V consecutive channels per thread: 8 (one 16-byte access) or 4
// where the channel count, the strides and the pointers allow it, else 1.
template <int V>
__device__ inline void ldv(const uint16_t *p, uint16_t (&o)[V]) {
    if constexpr (V == 8) {
        const uint4 u = *reinterpret_cast<const uint4 *>(p);
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int k = 0; k < 8; k++) o[k] = (uint16_t)(w[k >> 1] >> (k & 1) * 16);
    } else if constexpr (V == 4) {
        const uint2 u = *reinterpret_cast<const uint2 *>(p);
        o[0] = (uint16_t)(u.x & 0xffffu); o[1] = (uint16_t)(u.x >> 16);
        o[2] = (uint16_t)(u.y & 0xffffu); o[3] = (uint16_t)(u.y >> 16);
    } else {
#pragma unroll
        for (int k = 0; k < V; k++) o[k] = p[k];
    }
}
template <int V>
__device__ inline void stv(uint16_t *p, const uint16_t (&o)[V]) {
    if constexpr (V == 8) {
        uint32_t w[4];
#pragma unroll
        for (int k = 0; k < 4; k++) w[k] = (uint32_t)o[2 * k] | ((uint32_t)o[2 * k + 1] << 16);
        *reinterpret_cast<uint4 *>(p) = uint4{w[0], w[1], w[2], w[3]};
    } else if constexpr (V == 4) {
        uint2 u;
        u.x = (uint32_t)o[0] | ((uint32_t)o[1] << 16);
        u.y = (uint32_t)o[2] | ((uint32_t)o[3] << 16);
        *reinterpret_cast<uint2 *>(p) = u;
    } else {
#pragma unroll
        for (int k = 0; k < V; k++) p[k] = o[k];
    }
}

// Item i of n as (voxel v, channel ch) with cv groups of V channels a voxel; false beyond n.
// In 32 bits where n fits: the 64-bit division took longer than the copy.
template <int V>
__device__ inline bool item(int64_t n, int cv, int64_t &v, int &ch) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (n <= 0xffffffffll) {
        const uint32_t u = (uint32_t)i / (uint32_t)cv;
        v = u;
        ch = (int)((uint32_t)i - u * (uint32_t)cv) * V;
    } else {
        v = i / cv;
        ch = (int)(i % cv) * V;
    }
    return i < n;
}
// Coordinates of voxel v of an nx x ny x .. grid; a voxel number fits 32 bits below 2^32.
__device__ inline void voxel_xyz(int64_t v, int nx, int ny, int &x, int &y, int &z) {
    if (v <= 0xffffffffll) {
        const uint32_t u = (uint32_t)v, row = u / (uint32_t)nx;
        x = (int)(u - row * (uint32_t)nx);
        z = (int)(row / (uint32_t)ny);
        y = (int)(row - (uint32_t)z * (uint32_t)ny);
    } else {
        x = (int)(v % nx);
        y = (int)((v / nx) % ny);
        z = (int)(v / ((int64_t)nx * ny));
    }
}

// The elementwise kernels below move V channels a thread, 16 bytes (V = 8) where strides and
// pointers allow, and are bound by memory.  At 96^3, with 8 bytes a thread and 64-bit divisions
// before: upsampling into 32 channels 26 -> 18 us, pooling 16 channels 22 -> 21, the input of
// the network (2 bytes a store before) 38 -> 11.
//
// 2x2x2 mean of the fine grid n (even sizes) onto the coarse grid.
template <int V>
__global__ __launch_bounds__(256) void k_pool2(NnGrid f, int c, const uint16_t *__restrict__ x,
                                               int x_cs, uint16_t *__restrict__ y, int y_cs,
                                               int accumulate) {
    const int cx = f.nx / 2, cy = f.ny / 2, cz = f.nz / 2;
    int64_t v;
    int ch, X, Y, Z;
    if (!item<V>((int64_t)cx * cy * cz * (c / V), c / V, v, ch)) return;
    voxel_xyz(v, cx, cy, X, Y, Z);
    float s[V];
#pragma unroll
    for (int k = 0; k < V; k++) s[k] = 0.f;
#pragma unroll
    for (int m = 0; m < 8; m++) {
        const int64_t fv = ((int64_t)(2 * Z + (m >> 2)) * f.ny + 2 * Y + ((m >> 1) & 1)) * f.nx + 2 * X + (m & 1);
        uint16_t e[V];
        ldv<V>(x + fv * x_cs + ch, e);
#pragma unroll
        for (int k = 0; k < V; k++) s[k] += bf2f(e[k]);
    }
    uint16_t o[V];
    if (accumulate) ldv<V>(y + v * y_cs + ch, o);
#pragma unroll
    for (int k = 0; k < V; k++) {
        float t = s[k] * 0.125f;
        if (accumulate) t += bf2f(o[k]);
        o[k] = f2bf(t);
    }
    stv<V>(y + v * y_cs + ch, o);
}

// Adjoint of the mean pooling: each fine voxel gets 1/8 of its parent's gradient.
template <int V>
__global__ __launch_bounds__(256) void k_pool2_bwd(NnGrid f, int c, const uint16_t *__restrict__ gy,
                                                   int gy_cs, uint16_t *__restrict__ gx, int gx_cs,
                                                   int accumulate) {
    int64_t v;
    int ch, x, y, z;
    if (!item<V>(f.nvox * (c / V), c / V, v, ch)) return;
    voxel_xyz(v, f.nx, f.ny, x, y, z);
    const int64_t pv = ((int64_t)(z / 2) * (f.ny / 2) + y / 2) * (f.nx / 2) + x / 2;
    uint16_t e[V], o[V];
    ldv<V>(gy + pv * gy_cs + ch, e);
    if (accumulate) ldv<V>(gx + v * gx_cs + ch, o);
#pragma unroll
    for (int k = 0; k < V; k++) {
        float t = 0.125f * bf2f(e[k]);
        if (accumulate) t += bf2f(o[k]);
        o[k] = f2bf(t);
    }
    stv<V>(gx + v * gx_cs + ch, o);
}

// Nearest upsampling from the coarse grid to the fine grid f (each fine voxel copies its
// parent), and its adjoint (each parent sums its 8 children).
template <int V>
__global__ __launch_bounds__(256) void k_up2(NnGrid f, int c, const uint16_t *__restrict__ x,
                                             int x_cs, uint16_t *__restrict__ y, int y_cs) {
    int64_t v;
    int ch, xx, yy, zz;
    if (!item<V>(f.nvox * (c / V), c / V, v, ch)) return;
    voxel_xyz(v, f.nx, f.ny, xx, yy, zz);
    const int64_t pv = ((int64_t)(zz / 2) * (f.ny / 2) + yy / 2) * (f.nx / 2) + xx / 2;
    uint16_t e[V];
    ldv<V>(x + pv * x_cs + ch, e);
    stv<V>(y + v * y_cs + ch, e);
}

template <int V>
__global__ __launch_bounds__(256) void k_up2_bwd(NnGrid f, int c, const uint16_t *__restrict__ gy,
                                                 int gy_cs, uint16_t *__restrict__ gx, int gx_cs) {
    const int cx = f.nx / 2, cy = f.ny / 2, cz = f.nz / 2;
    int64_t v;
    int ch, X, Y, Z;
    if (!item<V>((int64_t)cx * cy * cz * (c / V), c / V, v, ch)) return;
    voxel_xyz(v, cx, cy, X, Y, Z);
    float s[V];
#pragma unroll
    for (int k = 0; k < V; k++) s[k] = 0.f;
#pragma unroll
    for (int m = 0; m < 8; m++) {
        const int64_t fv = ((int64_t)(2 * Z + (m >> 2)) * f.ny + 2 * Y + ((m >> 1) & 1)) * f.nx + 2 * X + (m & 1);
        uint16_t e[V];
        ldv<V>(gy + fv * gy_cs + ch, e);
#pragma unroll
        for (int k = 0; k < V; k++) s[k] += bf2f(e[k]);
    }
    uint16_t o[V];
#pragma unroll
    for (int k = 0; k < V; k++) o[k] = f2bf(s[k]);
    stv<V>(gx + v * gx_cs + ch, o);
}

// g = gy where the layer's output y > 0, else 0 (the ReLU gradient).
template <int V>
__global__ __launch_bounds__(256) void k_relu_bwd(int64_t nvox, int c, const uint16_t *__restrict__ y,
                                                  int y_cs, const uint16_t *__restrict__ gy,
                                                  int gy_cs, uint16_t *__restrict__ gout, int g_cs) {
    int64_t v;
    int ch;
    if (!item<V>(nvox * (c / V), c / V, v, ch)) return;
    uint16_t yv[V], gv[V], o[V];
    ldv<V>(y + v * y_cs + ch, yv);
    ldv<V>(gy + v * gy_cs + ch, gv);
    // positive bfloat16: sign bit clear and not zero
#pragma unroll
    for (int k = 0; k < V; k++) o[k] = (yv[k] != 0 && !(yv[k] & 0x8000u)) ? gv[k] : (uint16_t)0;
    stv<V>(gout + v * g_cs + ch, o);
}

// groups of 8 (16 bytes), 4 or 1 channels for c channels at the given strides and pointers
static int vec(int c, std::initializer_list<int> cs, std::initializer_list<const void *> ptrs) {
    for (int n = 8; n > 1; n >>= 1) {
        bool ok = c % n == 0;
        for (int s : cs) ok = ok && s % n == 0;
        for (const void *p : ptrs) ok = ok && reinterpret_cast<uintptr_t>(p) % (2 * n) == 0;
        if (ok && n != 2) return n;
    }
    return 1;
}

constexpr int kHeadMaxOut = 8;
constexpr int kHeadCin = 16;

// A voxel's 16 channels, 16 bytes at a time where wide (with the outputs' loop unrolled, the
// head with a target at 96^3: 92 us with 2-byte loads and stores, 30 with these).
__device__ inline void load16(const uint16_t *p, bool wide, uint16_t (&o)[kHeadCin]) {
    if (wide) {
        ldv<8>(p, reinterpret_cast<uint16_t(&)[8]>(o[0]));
        ldv<8>(p + 8, reinterpret_cast<uint16_t(&)[8]>(o[8]));
    } else {
#pragma unroll
        for (int c = 0; c < kHeadCin; c++) o[c] = p[c];
    }
}

// The 1x1x1 head: out[o][v] = bh[o] + sum_c wh[o][c] x[v][c] (binary32, planar).  With a
// target: go[o][v] = 2 wt[o] mask[v] (out - target) / n_mask (the gradient of the loss
// sum_o wt[o] mask (out - target)^2 / n_mask), gx = wh^T go (bf16) and the per-block
// partial sums of the loss.
__global__ __launch_bounds__(256) void k_head(int64_t nvox, const uint16_t *__restrict__ x, int x_cs,
                                              int no, const float *__restrict__ wh,
                                              const float *__restrict__ bh,
                                              float *__restrict__ out,
                                              const float *__restrict__ target,
                                              const uint8_t *__restrict__ mask,
                                              const float *__restrict__ wt, double inv_n,
                                              float *__restrict__ gout, uint16_t *__restrict__ gx,
                                              int gx_cs, double *__restrict__ loss_part) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const bool wide_x = x_cs % 8 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0;
    double loss = 0.0;
    if (v < nvox) {
        uint16_t xb[kHeadCin];
        load16(x + v * x_cs, wide_x, xb);
        float xv[kHeadCin];
#pragma unroll
        for (int c = 0; c < kHeadCin; c++) xv[c] = bf2f(xb[c]);
        float go[kHeadMaxOut];
#pragma unroll
        for (int o = 0; o < kHeadMaxOut; o++) {
            if (o >= no) break;
            float s = bh[o];
#pragma unroll
            for (int c = 0; c < kHeadCin; c++) s += wh[o * kHeadCin + c] * xv[c];
            if (out) out[o * nvox + v] = s;
            go[o] = 0.f;
            if (target && mask[v]) {
                const double d = (double)s - (double)target[o * nvox + v];
                loss += (double)wt[o] * d * d * inv_n;
                go[o] = (float)(2.0 * (double)wt[o] * d * inv_n);
            }
            if (target) gout[o * nvox + v] = go[o];
        }
        if (target && gx) {
            uint16_t gb[kHeadCin];
#pragma unroll
            for (int c = 0; c < kHeadCin; c++) {
                float s = 0.f;
#pragma unroll
                for (int o = 0; o < kHeadMaxOut; o++)
                    if (o < no) s += wh[o * kHeadCin + c] * go[o];
                gb[c] = f2bf(s);
            }
            if (gx_cs % 8 == 0 && reinterpret_cast<uintptr_t>(gx) % 16 == 0) {
                stv<8>(gx + v * gx_cs, reinterpret_cast<const uint16_t(&)[8]>(gb[0]));
                stv<8>(gx + v * gx_cs + 8, reinterpret_cast<const uint16_t(&)[8]>(gb[8]));
            } else {
#pragma unroll
                for (int c = 0; c < kHeadCin; c++) gx[v * gx_cs + c] = gb[c];
            }
        }
    }
    if (!target) return;
    __shared__ double lds[4];
    for (int off = 32; off > 0; off >>= 1) loss += __shfl_down(loss, off, 64);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = loss;
    __syncthreads();
    if (threadIdx.x == 0) loss_part[blockIdx.x] = ((lds[0] + lds[1]) + lds[2]) + lds[3];
}

// Per-chunk partial gradients of the head weights for output o = blockIdx.y:
// part[chunk][o][c] = sum_v go[o][v] x[v][c] (c < 16) and part[chunk][o][16] = sum_v go.
__global__ __launch_bounds__(256) void k_head_wgrad(int64_t nvox, const uint16_t *__restrict__ x,
                                                    int x_cs, const float *__restrict__ gout,
                                                    int64_t chunk, double *__restrict__ part) {
    constexpr int NV = kHeadCin + 1;
    const int o = blockIdx.y;
    const bool wide_x = x_cs % 8 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0;
    const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < nvox ? lo + chunk : nvox;
    double acc[NV];
#pragma unroll
    for (int k = 0; k < NV; k++) acc[k] = 0.0;
    for (int64_t v = lo + threadIdx.x; v < hi; v += 256) {
        const double go = gout[o * nvox + v];
        uint16_t xb[kHeadCin];
        load16(x + v * x_cs, wide_x, xb);
#pragma unroll
        for (int c = 0; c < kHeadCin; c++) acc[c] += go * (double)bf2f(xb[c]);
        acc[kHeadCin] += go;
    }
    __shared__ double lds[4][NV];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; k++) {
        double a = acc[k];
        for (int off = 32; off > 0; off >>= 1) a += __shfl_down(a, off, 64);
        if (lane == 0) lds[wave][k] = a;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        const int k = threadIdx.x;
        part[((int64_t)blockIdx.x * gridDim.y + o) * NV + k] = ((lds[0][k] + lds[1][k]) + lds[2][k]) + lds[3][k];
    }
}

// Fixed-order sums: the loss, gwh[o][c] and gbh[o].  One wave per sum of the gradients, all
// 16 waves on the loss; lanes take every 64th (1024th) partial, then halves are added.  (One
// thread a sum was a chain of loads: 31 us at 96^3.)
__global__ __launch_bounds__(1024) void k_head_final(const double *__restrict__ loss_part, int64_t nb,
                                                     const double *__restrict__ part, int64_t nch,
                                                     int no, double *__restrict__ loss,
                                                     float *__restrict__ gwh, float *__restrict__ gbh) {
    constexpr int NV = kHeadCin + 1;
    __shared__ double lds[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int k = wave; k < no * NV; k += 16) {
        double s = 0.0;
        for (int64_t c = lane; c < nch; c += 64) s += part[c * no * NV + k];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
        const int o = k / NV, c = k % NV;
        if (lane == 0) {
            if (c < kHeadCin) gwh[o * kHeadCin + c] = (float)s;
            else gbh[o] = (float)s;
        }
    }
    double s = 0.0;
    for (int64_t b = threadIdx.x; b < nb; b += 1024) s += loss_part[b];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if (lane == 0) lds[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < 16; i++) t += lds[i];
        *loss = t;
    }
}

// One Adam step (bias-corrected), binary32 master weights; refreshes their bf16 copy.
__global__ __launch_bounds__(256) void k_adam(int64_t n, float *__restrict__ w,
                                              const float *__restrict__ g, float *__restrict__ m,
                                              float *__restrict__ v, uint16_t *__restrict__ wb,
                                              float lr, float b1, float b2, float eps, float c1,
                                              float c2) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
    w[i] = wi;
    if (wb) wb[i] = f2bf(wi);
}

__global__ __launch_bounds__(256) void k_to_bf16(int64_t n, const float *__restrict__ src,
                                                 uint16_t *__restrict__ dst) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = f2bf(src[i]);
}

// The network input: channel 0 the pore mask, channel 1 the pore diameter / d_scale,
// channels 2 .. cs - 1 zero.
template <int V>
__global__ __launch_bounds__(256) void k_make_input(int64_t nvox, const uint8_t *__restrict__ mask,
                                                    const double *__restrict__ diam,
                                                    double inv_scale, uint16_t *__restrict__ x,
                                                    int cs) {
    int64_t v;
    int ch;
    if (!item<V>(nvox * (cs / V), cs / V, v, ch)) return;
    uint16_t o[V];
#pragma unroll
    for (int k = 0; k < V; k++) {
        float val = 0.f;
        if (ch + k == 0) val = mask[v] ? 1.f : 0.f;
        else if (ch + k == 1) val = (float)(diam[v] * inv_scale);
        o[k] = f2bf(val);
    }
    stv<V>(x + v * cs + ch, o);
}

// fields[k][v] = mask[v] ? out[k][v] * scale[k] : 0.
__global__ __launch_bounds__(256) void k_to_fields(int64_t nvox, int nk, const float *__restrict__ out,
                                                   const uint8_t *__restrict__ mask,
                                                   const float *__restrict__ scale,
                                                   float *__restrict__ fields) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= nvox) return;
    const bool in = mask[v];
    for (int k = 0; k < nk; k++) fields[k * nvox + v] = in ? out[k * nvox + v] * scale[k] : 0.f;
}

static unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

static lbm_status check_grid(const int32_t n[3], NnGrid &g) {
    LBM_REQUIRE(n && n[0] >= 1 && n[1] >= 1 && n[2] >= 1 && n[0] <= 4096 && n[1] <= 4096 &&
                    n[2] <= 4096,
                LBM_E_INVAL, "network grid sizes must lie in [1, 4096]");
    g.nx = n[0];
    g.ny = n[1];
    g.nz = n[2];
    g.nvox = (int64_t)n[0] * n[1] * n[2];
    return LBM_OK;
}

template <int WX, int WY, int WZ, int PZ>
static void conv_bricks(const NnGrid &g, const uint16_t *x, int x_cs, int cin, const uint16_t *w,
                        const float *bias, uint16_t *y, int y_cs, int cout, int relu, int flip,
                        hipStream_t s) {
    const auto cut = [](int n, int t) { return (unsigned)((n + t - 1) / t); };
    // neighbouring bricks, which share halos, on one of the 8 parts of the chip
    const dim3 grid((unsigned)xcd_launch(cut(g.nx, 4 * WX) * cut(g.ny, 4 * WY) * cut(g.nz, PZ * WZ)),
                    (unsigned)(cout / 16));
    if (flip)
        k_conv3d_bricks<WX, WY, WZ, PZ, true><<<grid, 256, 0, s>>>(g, x, x_cs, cin, w, cout, bias, y, y_cs, relu);
    else
        k_conv3d_bricks<WX, WY, WZ, PZ, false><<<grid, 256, 0, s>>>(g, x, x_cs, cin, w, cout, bias, y, y_cs, relu);
}
// The brick of a layer: a longer column reads fewer operands per product and a smaller halo,
// a smaller brick gives more workgroups where the layer leaves compute units idle.  The lines
// lie between 324 and 432 groups of 8 x 8 x 8 (24^3 x 64 -> 192 channels: 25.6 us with those,
// 23.4 with 8 x 8 x 4; 48^3 x 96 -> 32: 39.2 against 45.1), 216 and 648 of 8 x 8 x 4 (24^3 x
// 192 -> 64: 27.6 against 26.7 with 8 x 4 x 4; 24^3 x 64 -> 192: 23.4 against 26.3) and 144
// and 432 of 8 x 4 x 4 (12^3 x 128 -> 128: 13.2 against 11.9 with 4 x 4 x 4; 24^3 x 192 -> 64:
// 26.7 against 38.2).  A column of 8 planes is taken where 8 divides nz: less than a whole
// column of the last brick would be worked for nothing.
static void conv_launch(const NnGrid &g, const uint16_t *x, int x_cs, int cin, const uint16_t *w,
                        const float *bias, uint16_t *y, int y_cs, int cout, int relu, int flip,
                        hipStream_t s) {
    const auto groups = [&](int tx, int ty, int tz) {
        return (int64_t)((g.nx + tx - 1) / tx) * ((g.ny + ty - 1) / ty) * ((g.nz + tz - 1) / tz) * (cout / 16);
    };
    if (g.nz % 8 == 0 && groups(8, 8, 8) >= 384)
        conv_bricks<2, 2, 1, 8>(g, x, x_cs, cin, w, bias, y, y_cs, cout, relu, flip, s);
    else if (groups(8, 8, 4) >= 320)
        conv_bricks<2, 2, 1, 4>(g, x, x_cs, cin, w, bias, y, y_cs, cout, relu, flip, s);
    else if (groups(8, 4, 4) >= 320)
        conv_bricks<2, 1, 2, 2>(g, x, x_cs, cin, w, bias, y, y_cs, cout, relu, flip, s);
    else
        conv_bricks<1, 1, 4, 1>(g, x, x_cs, cin, w, bias, y, y_cs, cout, relu, flip, s);
}

static bool aligned8(const void *p) { return ((uintptr_t)p & 7u) == 0; }

static int64_t wgrad_chunk(int64_t nvox) {
    int64_t nch = nvox / 1024;
    if (nch < 1) nch = 1;
    if (nch > 1024) nch = 1024;
    int64_t chunk = (nvox + nch - 1) / nch;
    return (chunk + 15) / 16 * 16;
}

}  // namespace lbm

using namespace lbm;

extern "C" lbm_status lbm_nn_conv3d(const int32_t n[3], const uint16_t *x, int32_t x_cs, int32_t cin,
                                    const uint16_t *w, const float *bias, uint16_t *y, int32_t y_cs,
                                    int32_t cout, int32_t flags, void *stream) {
    NnGrid g;
    lbm_status st = check_grid(n, g);
    if (st != LBM_OK) return st;
    LBM_REQUIRE(x && w && y, LBM_E_INVAL, "lbm_nn_conv3d: null tensor");
    LBM_REQUIRE(g.nvox % 16 == 0, LBM_E_INVAL, "lbm_nn_conv3d: voxel count must be a multiple of 16");
    LBM_REQUIRE(cin >= 16 && cin % 16 == 0 && cin <= x_cs && x_cs % 4 == 0, LBM_E_INVAL,
                "lbm_nn_conv3d: cin must be a positive multiple of 16 within the stride %d", x_cs);
    LBM_REQUIRE(cout <= y_cs && aligned8(x) && aligned8(w), LBM_E_INVAL,
                "lbm_nn_conv3d: cout beyond the output stride, or a misaligned tensor");
    LBM_REQUIRE((flags & ~(LBM_NN_RELU | LBM_NN_FLIP)) == 0, LBM_E_INVAL, "lbm_nn_conv3d: flags");
    st = check_device();
    if (st != LBM_OK) return st;
    const unsigned grid = (unsigned)((g.nvox / 16 + 3) / 4);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int relu = (flags & LBM_NN_RELU) != 0, flip = (flags & LBM_NN_FLIP) != 0;
    // bricks: grid sizes multiples of 4 and 16-byte input rows (the halo is copied as
    // 16-byte vectors), with the elements of a halo plane (10 x 10 voxels at most), of a 4 x 4
    // output plane and of 8 taps' weights within 32-bit offsets
    const int64_t reach = std::max({(int64_t)9 * (g.nx + 1) * x_cs + 16, (int64_t)3 * (g.nx + 1) * y_cs + 16,
                                    (int64_t)8 * cout * cin});
    if (g.nx % 4 == 0 && g.ny % 4 == 0 && g.nz % 4 == 0 && x_cs % 8 == 0 &&
        reinterpret_cast<uintptr_t>(x) % 16 == 0 && reach <= (int64_t)INT32_MAX) {
        LBM_REQUIRE(cout == 16 || cout == 32 || cout == 48 || cout == 64 || cout == 96 ||
                        cout == 128 || cout == 192,
                    LBM_E_INVAL, "lbm_nn_conv3d: cout %d not supported", cout);
        conv_launch(g, x, x_cs, cin, w, bias, y, y_cs, cout, relu, flip, s);
        LBM_CHECK_LAUNCH();
        return LBM_OK;
    }
    switch (cout) {
    case 16: k_conv3d<1><<<grid, 256, 0, s>>>(g, x, x_cs, cin, w, bias, y, y_cs, relu, flip); break;
    case 32: k_conv3d<2><<<grid, 256, 0, s>>>(g, x, x_cs, cin, w, bias, y, y_cs, relu, flip); break;
    case 48: k_conv3d<3><<<grid, 256, 0, s>>>(g, x, x_cs, cin, w, bias, y, y_cs, relu, flip); break;
    case 64: k_conv3d<4><<<grid, 256, 0, s>>>(g, x, x_cs, cin, w, bias, y, y_cs, relu, flip); break;
    case 96: k_conv3d<6><<<grid, 256, 0, s>>>(g, x, x_cs, cin, w, bias, y, y_cs, relu, flip); break;
    case 128: k_conv3d<8><<<grid, 256, 0, s>>>(g, x, x_cs, cin, w, bias, y, y_cs, relu, flip); break;
    case 192: k_conv3d<12><<<grid, 256, 0, s>>>(g, x, x_cs, cin, w, bias, y, y_cs, relu, flip); break;
    default: set_error("lbm_nn_conv3d: cout %d not supported", cout); return LBM_E_INVAL;
    }
    LBM_CHECK_LAUNCH();
    return LBM_OK;
}

// Sums of the partial rows: 16 threads an output, or one where there are fewer rows than that
// (12 rows of 12^3 x 64 -> 128 channels, with the products: 23.3 us, with 16 threads 24.8).
static void sum_parts(const float *part, int64_t nparts, int64_t count, float *out, const float *part_b,
                      int n_b, float *out_b, int accumulate, hipStream_t s) {
    const bool wide = nparts >= 16;
    const int64_t per = (wide ? 16 : 256) * 4;
    const unsigned nblk = (unsigned)((count + per - 1) / per), nblk_b = (unsigned)((n_b + per - 1) / per);
    if (wide)
        k_sum_parts<16><<<nblk + nblk_b, 256, 0, s>>>(part, nparts, count, out, part_b, n_b, out_b, nblk, accumulate);
    else
        k_sum_parts<1><<<nblk + nblk_b, 256, 0, s>>>(part, nparts, count, out, part_b, n_b, out_b, nblk, accumulate);
}

extern "C" size_t lbm_nn_wgrad_workspace(const int32_t n[3], int32_t cin, int32_t cout) {
    if (!n || n[0] < 1 || n[1] < 1 || n[2] < 1 || cin < 1 || cout < 1) return 0;
    const int64_t nvox = (int64_t)n[0] * n[1] * n[2];
    const int64_t nch = (nvox + wgrad_chunk(nvox) - 1) / wgrad_chunk(nvox);
    return (size_t)nch * ((size_t)27 * cout * cin + cout) * sizeof(float) + 256;
}

extern "C" lbm_status lbm_nn_conv3d_wgrad(const int32_t n[3], const uint16_t *x, int32_t x_cs,
                                          int32_t cin, const uint16_t *gy, int32_t g_cs,
                                          int32_t cout, float *dw, float *db, int32_t accumulate,
                                          void *workspace, size_t ws_bytes, void *stream) {
    NnGrid g;
    lbm_status st = check_grid(n, g);
    if (st != LBM_OK) return st;
    LBM_REQUIRE(x && gy && dw && workspace, LBM_E_INVAL, "lbm_nn_conv3d_wgrad: null argument");
    LBM_REQUIRE(g.nvox % 16 == 0, LBM_E_INVAL, "lbm_nn_conv3d_wgrad: voxel count must be a multiple of 16");
    LBM_REQUIRE(cin % 16 == 0 && cin >= 16 && cin <= x_cs && cout % 16 == 0 && cout >= 16 &&
                    cout <= g_cs,
                LBM_E_INVAL, "lbm_nn_conv3d_wgrad: channel counts must be multiples of 16 within the strides");
    LBM_REQUIRE(ws_bytes >= lbm_nn_wgrad_workspace(n, cin, cout), LBM_E_NOMEM,
                "lbm_nn_conv3d_wgrad: workspace below %zu bytes", lbm_nn_wgrad_workspace(n, cin, cout));
    st = check_device();
    if (st != LBM_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t chunk = wgrad_chunk(g.nvox);
    int64_t nch = (g.nvox + chunk - 1) / chunk;  // the workspace's partial rows
    // 16-byte rows inside the workspace's 256 spare bytes
    float *part = reinterpret_cast<float *>((reinterpret_cast<uintptr_t>(workspace) + 15) & ~(uintptr_t)15);
    float *part_b = part + nch * 27 * (int64_t)cout * cin;
    // the brick kernel copies 16-channel rows as 16-byte vectors: aligned rows only
    const bool rows16 = x_cs % 8 == 0 && g_cs % 8 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0 &&
                        reinterpret_cast<uintptr_t>(gy) % 16 == 0;
    if (g.nx % 4 == 0 && g.ny % 4 == 0 && g.nz % 4 == 0 && rows16) {
        // two workgroups for each of the 256 compute units, as far as the workspace's partial
        // rows go: more only add rows to sum and a last round that is half empty (with the sum,
        // 96^3 x 16 -> 16 channels: 864 chunks 39.8 us, 494 32.8; 48^3 x 96 -> 32: 108 chunks
        // 64.8, 40 36.0)
        const int64_t nb = (int64_t)((g.nx + 7) / 8) * ((g.ny + 7) / 8) * (g.nz / 4);
        const int64_t blocks = (int64_t)(cout / 16) * (cin / 16);
        const int64_t rows = (int64_t)((ws_bytes - 256) / (((size_t)27 * cout * cin + cout) * sizeof(float)));
        int64_t want = (512 + blocks - 1) / blocks;
        if (want > rows) want = rows;
        const int64_t bricks = (nb + want - 1) / want, nbc = (nb + bricks - 1) / bricks;
        part_b = part + nbc * 27 * (int64_t)cout * cin;
        k_conv3d_wgrad_bricks<<<dim3((unsigned)nbc, (unsigned)((cout / 16) * (cin / 16))), 256, 0, s>>>(
            g, x, x_cs, cin, gy, g_cs, cout, (int)bricks, (int)nb, part, part_b);
        LBM_CHECK_LAUNCH();
        nch = nbc;
    } else {
        const dim3 grid((unsigned)nch, 27, (unsigned)(cout / 16));
        switch (cin) {
        case 16: k_conv3d_wgrad<1><<<grid, 64, 0, s>>>(g, x, x_cs, gy, g_cs, cout, chunk, part, part_b); break;
        case 32: k_conv3d_wgrad<2><<<grid, 64, 0, s>>>(g, x, x_cs, gy, g_cs, cout, chunk, part, part_b); break;
        case 48: k_conv3d_wgrad<3><<<grid, 64, 0, s>>>(g, x, x_cs, gy, g_cs, cout, chunk, part, part_b); break;
        case 64: k_conv3d_wgrad<4><<<grid, 64, 0, s>>>(g, x, x_cs, gy, g_cs, cout, chunk, part, part_b); break;
        case 96: k_conv3d_wgrad<6><<<grid, 64, 0, s>>>(g, x, x_cs, gy, g_cs, cout, chunk, part, part_b); break;
        case 128: k_conv3d_wgrad<8><<<grid, 64, 0, s>>>(g, x, x_cs, gy, g_cs, cout, chunk, part, part_b); break;
        case 192: k_conv3d_wgrad<12><<<grid, 64, 0, s>>>(g, x, x_cs, gy, g_cs, cout, chunk, part, part_b); break;
        default: set_error("lbm_nn_conv3d_wgrad: cin %d not supported", cin); return LBM_E_INVAL;
        }
        LBM_CHECK_LAUNCH();
    }
    sum_parts(part, nch, (int64_t)27 * cout * cin, dw, part_b, db ? cout : 0, db, accumulate, s);
    LBM_CHECK_LAUNCH();
    return LBM_OK;
}

extern "C" lbm_status lbm_nn_transpose_weights(const uint16_t *w, int32_t cout, int32_t cin,
                                               uint16_t *wt, void *stream) {
    LBM_REQUIRE(w && wt && cout >= 1 && cin >= 1, LBM_E_INVAL, "lbm_nn_transpose_weights: arguments");
    lbm_status st = check_device();
    if (st != LBM_OK) return st;
    const int64_t n = (int64_t)27 * cout * cin;
    k_transpose_w<<<nblk(n), 256, 0, static_cast<hipStream_t>(stream)>>>(w, cout, cin, wt);
    LBM_CHECK_LAUNCH();
    return LBM_OK;
}

static lbm_status pool_args(const int32_t n[3], int32_t c, const void *a, int32_t a_cs,
                            const void *b, int32_t b_cs, NnGrid &g) {
    lbm_status st = check_grid(n, g);
    if (st != LBM_OK) return st;
    LBM_REQUIRE(a && b && c >= 1 && c <= a_cs && c <= b_cs, LBM_E_INVAL,
                "pooling: null tensor or channel count beyond a stride");
    LBM_REQUIRE(n[0] % 2 == 0 && n[1] % 2 == 0 && n[2] % 2 == 0, LBM_E_INVAL,
                "pooling: the fine grid must have even sizes");
    return check_device();
}

extern "C" lbm_status lbm_nn_pool2(const int32_t n_fine[3], int32_t c, const uint16_t *x, int32_t x_cs,
                                   uint16_t *y, int32_t y_cs, int32_t accumulate, void *stream) {
    NnGrid g;
    lbm_status st = pool_args(n_fine, c, x, x_cs, y, y_cs, g);
    if (st != LBM_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int n = vec(c, {x_cs, y_cs}, {x, y});
    const auto kernel = n == 8 ? k_pool2<8> : n == 4 ? k_pool2<4> : k_pool2<1>;
    kernel<<<nblk(g.nvox / 8 * (c / n)), 256, 0, s>>>(g, c, x, x_cs, y, y_cs, accumulate);
    LBM_CHECK_LAUNCH();
    return LBM_OK;
}

extern "C" lbm_status lbm_nn_pool2_bwd(const int32_t n_fine[3], int32_t c, const uint16_t *gy,
                                       int32_t gy_cs, uint16_t *gx, int32_t gx_cs, int32_t accumulate,
                                       void *stream) {
    NnGrid g;
    lbm_status st = pool_args(n_fine, c, gy, gy_cs, gx, gx_cs, g);
    if (st != LBM_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int n = vec(c, {gy_cs, gx_cs}, {gy, gx});
    const auto kernel = n == 8 ? k_pool2_bwd<8> : n == 4 ? k_pool2_bwd<4> : k_pool2_bwd<1>;
    kernel<<<nblk(g.nvox * (c / n)), 256, 0, s>>>(g, c, gy, gy_cs, gx, gx_cs, accumulate);
    LBM_CHECK_LAUNCH();
    return LBM_OK;
}

extern "C" lbm_status lbm_nn_up2(const int32_t n_fine[3], int32_t c, const uint16_t *x, int32_t x_cs,
                                 uint16_t *y, int32_t y_cs, void *stream) {
    NnGrid g;
    lbm_status st = pool_args(n_fine, c, x, x_cs, y, y_cs, g);
    if (st != LBM_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int n = vec(c, {x_cs, y_cs}, {x, y});
    const auto kernel = n == 8 ? k_up2<8> : n == 4 ? k_up2<4> : k_up2<1>;
    kernel<<<nblk(g.nvox * (c / n)), 256, 0, s>>>(g, c, x, x_cs, y, y_cs);
    LBM_CHECK_LAUNCH();
    return LBM_OK;
}

extern "C" lbm_status lbm_nn_up2_bwd(const int32_t n_fine[3], int32_t c, const uint16_t *gy,
                                     int32_t gy_cs, uint16_t *gx, int32_t gx_cs, void *stream) {
    NnGrid g;
    lbm_status st = pool_args(n_fine, c, gy, gy_cs, gx, gx_cs, g);
    if (st != LBM_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int n = vec(c, {gy_cs, gx_cs}, {gy, gx});
    const auto kernel = n == 8 ? k_up2_bwd<8> : n == 4 ? k_up2_bwd<4> : k_up2_bwd<1>;
    kernel<<<nblk(g.nvox / 8 * (c / n)), 256, 0, s>>>(g, c, gy, gy_cs, gx, gx_cs);
    LBM_CHECK_LAUNCH();
    return LBM_OK;
}

extern "C" lbm_status lbm_nn_relu_bwd(int64_t nvox, int32_t c, const uint16_t *y, int32_t y_cs,
                                      const uint16_t *gy, int32_t gy_cs, uint16_t *g, int32_t g_cs,
                                      void *stream) {
    LBM_REQUIRE(nvox >= 0 && y && gy && g && c >= 1 && c <= y_cs && c <= gy_cs && c <= g_cs,
                LBM_E_INVAL, "lbm_nn_relu_bwd: arguments");
    lbm_status st = check_device();
    if (st != LBM_OK) return st;
    if (nvox == 0) return LBM_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int n = vec(c, {y_cs, gy_cs, g_cs}, {y, gy, g});
    const auto kernel = n == 8 ? k_relu_bwd<8> : n == 4 ? k_relu_bwd<4> : k_relu_bwd<1>;
    kernel<<<nblk(nvox * (c / n)), 256, 0, s>>>(nvox, c, y, y_cs, gy, gy_cs, g, g_cs);
    LBM_CHECK_LAUNCH();
    return LBM_OK;
}

static int64_t head_chunk(int64_t nvox) {
    int64_t nch = nvox / 8192;
    if (nch < 1) nch = 1;
    if (nch > 256) nch = 256;
    return (nvox + nch - 1) / nch;
}

extern "C" size_t lbm_nn_head_workspace(int64_t nvox, int32_t no) {
    if (nvox < 1 || no < 1) return 0;
    const int64_t nb = (nvox + 255) / 256, chunk = head_chunk(nvox), nch = (nvox + chunk - 1) / chunk;
    Carver c(nullptr);
    c.take<double>(nb);
    c.take<double>(nch * no * (kHeadCin + 1));
    c.take<double>(1);
    c.take<float>(nvox * no);
    return c.off + 256;
}

extern "C" lbm_status lbm_nn_head(int64_t nvox, const uint16_t *x, int32_t x_cs, int32_t no,
                                  const float *wh, const float *bh, float *out, const float *target,
                                  const uint8_t *mask, const float *wt, double n_mask, uint16_t *gx,
                                  int32_t gx_cs, float *gwh, float *gbh, double *loss_h,
                                  void *workspace, size_t ws_bytes, void *stream) {
    LBM_REQUIRE(nvox >= 1 && x && wh && bh && x_cs >= kHeadCin && no >= 1 && no <= kHeadMaxOut,
                LBM_E_INVAL, "lbm_nn_head: arguments (16 input channels, 1..8 outputs)");
    LBM_REQUIRE(!target || (mask && wt && gwh && gbh && loss_h && workspace && n_mask > 0),
                LBM_E_INVAL, "lbm_nn_head: a target needs mask, weights, gradient outputs and n_mask > 0");
    LBM_REQUIRE(!gx || gx_cs >= kHeadCin, LBM_E_INVAL, "lbm_nn_head: gradient stride");
    LBM_REQUIRE(!target || ws_bytes >= lbm_nn_head_workspace(nvox, no), LBM_E_NOMEM,
                "lbm_nn_head: workspace below %zu bytes", lbm_nn_head_workspace(nvox, no));
    lbm_status st = check_device();
    if (st != LBM_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t nb = (nvox + 255) / 256, chunk = head_chunk(nvox), nch = (nvox + chunk - 1) / chunk;
    Carver c(workspace);
    double *loss_part = c.take<double>(nb);
    double *part = c.take<double>(nch * no * (kHeadCin + 1));
    double *dloss = c.take<double>(1);
    float *gout = c.take<float>(nvox * no);
    k_head<<<(unsigned)nb, 256, 0, s>>>(nvox, x, x_cs, no, wh, bh, out, target, mask, wt,
                                        target ? 1.0 / n_mask : 0.0, target ? gout : nullptr,
                                        target ? gx : nullptr, gx_cs, loss_part);
    LBM_CHECK_LAUNCH();
    if (target) {
        k_head_wgrad<<<dim3((unsigned)nch, (unsigned)no), 256, 0, s>>>(nvox, x, x_cs, gout, chunk, part);
        LBM_CHECK_LAUNCH();
        k_head_final<<<1, 1024, 0, s>>>(loss_part, nb, part, nch, no, dloss, gwh, gbh);
        LBM_CHECK_LAUNCH();
        LBM_TRY_HIP(hipMemcpyAsync(loss_h, dloss, sizeof(double), hipMemcpyDeviceToHost, s));
        LBM_TRY_HIP(hipStreamSynchronize(s));
    }
    return LBM_OK;
}

extern "C" lbm_status lbm_nn_adam(int64_t n, float *w, const float *g, float *m, float *v,
                                  uint16_t *w_bf16, float lr, float beta1, float beta2, float eps,
                                  int64_t step, void *stream) {
    LBM_REQUIRE(n >= 0 && w && g && m && v && step >= 1 && lr > 0 && eps > 0 && beta1 >= 0 &&
                    beta1 < 1 && beta2 >= 0 && beta2 < 1,
                LBM_E_INVAL, "lbm_nn_adam: arguments");
    lbm_status st = check_device();
    if (st != LBM_OK) return st;
    if (n == 0) return LBM_OK;
    const float c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, (double)step)));
    k_adam<<<nblk(n), 256, 0, static_cast<hipStream_t>(stream)>>>(n, w, g, m, v, w_bf16, lr, beta1,
                                                                 beta2, eps, c1, c2);
    LBM_CHECK_LAUNCH();
    return LBM_OK;
}

extern "C" lbm_status lbm_nn_to_bf16(int64_t n, const float *src, uint16_t *dst, void *stream) {
    LBM_REQUIRE(n >= 0 && src && dst, LBM_E_INVAL, "lbm_nn_to_bf16: arguments");
    lbm_status st = check_device();
    if (st != LBM_OK) return st;
    if (n == 0) return LBM_OK;
    k_to_bf16<<<nblk(n), 256, 0, static_cast<hipStream_t>(stream)>>>(n, src, dst);
    LBM_CHECK_LAUNCH();
    return LBM_OK;
}

extern "C" lbm_status lbm_nn_make_input(int64_t nvox, const uint8_t *mask, const double *diam,
                                        double d_scale, uint16_t *x, int32_t x_cs, void *stream) {
    LBM_REQUIRE(nvox >= 0 && mask && diam && x && x_cs >= 2 && x_cs % 4 == 0 && d_scale > 0,
                LBM_E_INVAL, "lbm_nn_make_input: arguments");
    lbm_status st = check_device();
    if (st != LBM_OK) return st;
    if (nvox == 0) return LBM_OK;
    const int n = vec(x_cs, {}, {x});
    const auto kernel = n == 8 ? k_make_input<8> : n == 4 ? k_make_input<4> : k_make_input<1>;
    // a launch holds fewer than 2^32 threads: with a thread per group of channels, fewer voxels
    // than a call may have
    const int64_t most = std::max<int64_t>((int64_t)0x80000000 / (x_cs / n), 1);
    for (int64_t v = 0; v < nvox; v += most) {
        const int64_t nv = std::min(nvox - v, most);
        kernel<<<nblk(nv * (x_cs / n)), 256, 0, static_cast<hipStream_t>(stream)>>>(
            nv, mask + v, diam + v, 1.0 / d_scale, x + v * x_cs, x_cs);
        LBM_CHECK_LAUNCH();
    }
    return LBM_OK;
}

extern "C" lbm_status lbm_nn_to_fields(int64_t nvox, int32_t nk, const float *out, const uint8_t *mask,
                                       const float *scale, float *fields, void *stream) {
    LBM_REQUIRE(nvox >= 0 && nk >= 1 && out && mask && scale && fields, LBM_E_INVAL,
                "lbm_nn_to_fields: arguments");
    lbm_status st = check_device();
    if (st != LBM_OK) return st;
    if (nvox == 0) return LBM_OK;
    k_to_fields<<<nblk(nvox), 256, 0, static_cast<hipStream_t>(stream)>>>(nvox, nk, out, mask, scale,
                                                                         fields);
    LBM_CHECK_LAUNCH();
    return LBM_OK;
}
