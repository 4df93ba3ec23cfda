// Structure characterisation on the GPU (Section 4.1): 18-neighbour connected-component
// labelling with transport flags, the 13-direction chord pore size, and the exact
// squared Euclidean distance map with its maximum-inscribed-sphere pore width.
// Everything is integer except the final FP64 formulas, which are evaluated in the
// stated order (this file is compiled with -ffp-contract=off).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "lbm_internal.h"

namespace lbm {

constexpr int32_t kInf = 0x3fffffff;

// Every kernel here takes its voxels by (x, y, z) from a 3-D grid, one wave per 64-voxel
// segment of a row (lane = x), four rows per workgroup: no 64-bit divisions, coalesced
// rows, and a wave's ballot is the segment's occupancy.
static dim3 row_grid(const Grid &g) {
    return dim3((unsigned)g.nseg, (unsigned)((g.ny + 3) / 4), (unsigned)g.nz);
}
constexpr int kRows = 4;

// The distance passes give a wave several rows of a box of up to 32 voxels in x: rows of 2^lane_log
// lanes each (nx = 1, ny = nz = 1000: 386 us for the three passes with a wave a row, now 20).
// The number is the template argument LL, 6 for a row a wave, or -1 where it comes as `ll`.
static int lane_log(const Grid &g) {
    int s = 0;
    while ((1 << s) < g.nx && s < 6) s++;
    return s;
}

// ================================================================ labelling
// Union-find over the pore voxels.  What bounds it is the chains of dependent loads a
// find walks, so the trees are kept flat and the unions few:
//  1. k_ccl_tile joins the voxels of a 64 x 8 x 8 tile in LDS and leaves in every voxel the
//     global index of its tile component's first voxel;
//  2. k_ccl_border and k_ccl_cross join tile components across the tile faces;
//  3. k_ccl_faces / k_ccl_finish: transport flags by root, final labels and counts.
// A run of consecutive pore voxels in a segment is one node of the graph (its first voxel
// stands for it), and two touching runs are joined once, at their first contact, found
// from the bits of the two rows.  One union per voxel and neighbour, straight in global
// memory, took 2.9 ms at 128^3 (porosity 0.40) and 46 ms at 512^3 (with one atomic per
// wave on each of three counters in the last pass, 33 ms of it); now 0.13 and 2.5 ms.
constexpr int kTy = 8, kTz = 8;  // rows of a labelling tile

// First lane of the run of set bits that holds `lane` (bit `lane` of w is set).
__device__ inline int run_start(uint64_t w, int lane) {
    const uint64_t zeros = ~w & ((1ull << lane) - 1);
    return zeros ? 64 - __builtin_clzll(zeros) : 0;
}

// The contacts of the run at bit x of row A with row B: bits `o` (same x), `p` (x + 1), `m`
// (x - 1) of this lane that carry a union.  am/bm, ap/bp: the rows' bits at x - 1, x + 1.
struct Contact {
    bool o, p, m;
};
__device__ inline Contact contact(bool a, bool am, bool ap, bool b, bool bm, bool bp, bool diag) {
    Contact c;
    c.o = a && b && !(am && bm);  // the same pair of runs already met at x - 1
    c.p = diag && a && !b && bp && !ap;
    c.m = diag && a && !b && bm && !am;
    return c;
}

template <int SCOPE>
__device__ inline int32_t ccl_root(int32_t *L, int32_t v) {
    int32_t p = __hip_atomic_load(&L[v], __ATOMIC_RELAXED, SCOPE);
    if (p == v) return v;
    int32_t r = p;
    for (;;) {
        const int32_t q = __hip_atomic_load(&L[r], __ATOMIC_RELAXED, SCOPE);
        if (q == r) break;
        r = q;
    }
    // v is no root, so its parent may be any of its ancestors
    if (r != p) __hip_atomic_store(&L[v], r, __ATOMIC_RELAXED, SCOPE);
    return r;
}

// Union of the trees of a and b: the larger root is pointed at the smaller one, so the
// final root of every component is its smallest index.  When the atomic finds that b
// was no longer a root, the merge continues with b's new parent.
template <int SCOPE>
__device__ inline void ccl_unite(int32_t *L, int32_t a, int32_t b) {
    for (;;) {
        a = ccl_root<SCOPE>(L, a);
        b = ccl_root<SCOPE>(L, b);
        if (a == b) return;
        if (a > b) { int32_t t = a; a = b; b = t; }
        const int32_t old = __hip_atomic_fetch_min(&L[b], a, __ATOMIC_RELAXED, SCOPE);
        if (old == b) return;
        b = old;
    }
}

// Components of one tile (no links across its faces).  Local indices are 64 (8 z + y) + x,
// in the order of the global ones, so a local root is the component's smallest voxel.
// Each component's first voxel also clears its face flags (a final root is one of them),
// and the first workgroup the counters.
constexpr int kTileWaves = 16;  // four rows per wave: short chains of dependent LDS accesses
__global__ __launch_bounds__(kTileWaves * 64) void k_ccl_tile(Grid g, const uint8_t *__restrict__ pore,
                                                  int32_t *__restrict__ L,
                                                  uint8_t *__restrict__ fin,
                                                  uint8_t *__restrict__ fout,
                                                  unsigned long long *__restrict__ counts) {
    __shared__ uint64_t bits[kTz][kTy];
    __shared__ int32_t lab[kTz * kTy * 64];
    constexpr int S = __HIP_MEMORY_SCOPE_WORKGROUP;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int x = (int)blockIdx.x * 64 + lane, y0 = (int)blockIdx.y * kTy, z0 = (int)blockIdx.z * kTz;
    if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x < 4)
        counts[threadIdx.x] = 0;
    bool pr[kTz * kTy / kTileWaves];
#pragma unroll
    for (int i = 0; i < kTz * kTy / kTileWaves; i++) {  // the wave's rows, all loads in flight
        const int r = wave + kTileWaves * i, y = y0 + r % kTy, z = z0 + r / kTy;
        pr[i] = x < g.nx && y < g.ny && z < g.nz && pore[g.lin(x, y, z)] != 0;
    }
#pragma unroll
    for (int i = 0; i < kTz * kTy / kTileWaves; i++) {
        const int r = wave + kTileWaves * i;
        const uint64_t w = __ballot(pr[i]);
        if (lane == 0) bits[r / kTy][r % kTy] = w;
        lab[r * 64 + lane] = pr[i] ? r * 64 + run_start(w, lane) : -1;
    }
    __syncthreads();
    for (int r = wave; r < kTz * kTy; r += kTileWaves) {
        const int ty = r % kTy, tz = r / kTy;
        const uint64_t A = bits[tz][ty];
        const bool a = (A >> lane) & 1, am = lane > 0 && ((A >> (lane - 1)) & 1),
                   ap = lane < 63 && ((A >> (lane + 1)) & 1);
        for (int k = 0; k < 4; k++) {
            const int dy = k == 0 ? 1 : (k == 1 ? 0 : (k == 2 ? 1 : -1)), dz = k == 0 ? 0 : 1;
            if (ty + dy < 0 || ty + dy >= kTy || tz + dz >= kTz) continue;
            const uint64_t B = bits[tz + dz][ty + dy];
            const bool b = (B >> lane) & 1, bm = lane > 0 && ((B >> (lane - 1)) & 1),
                       bp = lane < 63 && ((B >> (lane + 1)) & 1);
            const Contact c = contact(a, am, ap, b, bm, bp, k < 2);
            const int32_t v = r * 64 + lane, u = v + 64 * (dy + kTy * dz);
            if (c.o) ccl_unite<S>(lab, v, u);
            if (c.p) ccl_unite<S>(lab, v, u + 1);
            if (c.m) ccl_unite<S>(lab, v, u - 1);
        }
    }
    __syncthreads();
    for (int r = wave; r < kTz * kTy; r += kTileWaves) {
        const int y = y0 + r % kTy, z = z0 + r / kTy;
        if (x >= g.nx || y >= g.ny || z >= g.nz) continue;
        const int32_t v = r * 64 + lane;
        int32_t l = lab[v];
        if (l >= 0) l = ccl_root<S>(lab, v);
        const int64_t gv = g.lin(x, y, z);
        const int rr = l >> 6;
        L[gv] = l < 0 ? -1
                      : (int32_t)g.lin((int)blockIdx.x * 64 + (l & 63), y0 + rr % kTy, z0 + rr / kTy);
        if (l == v) {
            fin[gv] = 0;
            fout[gv] = 0;
        }
    }
}

// Unions of v and u in the lanes where c holds (the whole wave calls).  Along a row most
// contacts join the same two components of the tiles, so a lane leaves its union to the last
// lane before it that joins the same two parents: the finds all end at the few roots of the
// large components, whose words serve one access at a time.  (A union per contact: k_ccl_border
// 110 us at 128^3, porosity 0.40, and 865 us at 512^3, 0.25; now 70 and 755.)
template <int SCOPE>
__device__ inline void ccl_unite_wave(int32_t *L, bool c, int32_t v, int32_t u) {
    const uint64_t m = __ballot(c);
    if (!m) return;
    const int lane = threadIdx.x & 63;
    int32_t pv = -1, pu = -1;
    if (c) {
        pv = __hip_atomic_load(&L[v], __ATOMIC_RELAXED, SCOPE);
        pu = __hip_atomic_load(&L[u], __ATOMIC_RELAXED, SCOPE);
    }
    const uint64_t before = m & ((1ull << lane) - 1);
    const int last = before ? 63 - __clzll((long long)before) : lane;
    const int32_t qv = __shfl(pv, last, 64), qu = __shfl(pu, last, 64);
    if (c && !(before && qv == pv && qu == pu)) ccl_unite<SCOPE>(L, pv, pu);
}

// The links of a row with its neighbour rows across a tile face in y or z (periodic).
// All rows' bytes are loaded before the first union, whose atomics nothing moves across.
__global__ __launch_bounds__(256) void k_ccl_border(Grid g, const uint8_t *__restrict__ pore,
                                                    int32_t *L) {
    constexpr int S = __HIP_MEMORY_SCOPE_AGENT;
    const int lane = threadIdx.x & 63;
    const int x = (int)blockIdx.x * 64 + lane, y = (int)blockIdx.y * kRows + (threadIdx.x >> 6),
              z = (int)blockIdx.z;
    if (y >= g.ny) return;  // uniform per wave
    const bool yl = y % kTy == 0, yh = y % kTy == kTy - 1 || y == g.ny - 1,
               zh = z % kTz == kTz - 1 || z == g.nz - 1;
    if (!yl && !yh && !zh) return;  // no neighbour row in another tile
    const bool inx = x < g.nx;
    const int64_t row = g.lin(0, y, z);
    // bits of this lane and, for the outer lanes, of the voxel beyond the segment
    const int xe = lane == 0 ? x - 1 : x + 1;
    const bool outer = (lane == 0 || lane == 63) && xe >= 0 && xe < g.nx;
    int64_t brow[4];
    bool out[4], b[4], be[4];
    const bool a = inx && pore[row + x] != 0, ae = outer && pore[row + xe] != 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int dy = k == 0 ? 1 : (k == 1 ? 0 : (k == 2 ? 1 : -1)), dz = k == 0 ? 0 : 1;
        out[k] = (dz == 1 && zh) || (dy == 1 && yh) || (dy == -1 && yl);
        int yy = y + dy, zz = z + dz;
        yy = yy < 0 ? yy + g.ny : (yy >= g.ny ? yy - g.ny : yy);
        zz = zz >= g.nz ? zz - g.nz : zz;
        brow[k] = g.lin(0, yy, zz);
        b[k] = inx && out[k] && pore[brow[k] + x] != 0;
        be[k] = outer && out[k] && k < 2 && pore[brow[k] + xe] != 0;
    }
    const uint64_t A = __ballot(a);
    const bool am = lane > 0 ? (A >> (lane - 1)) & 1 : ae, ap = lane < 63 ? (A >> (lane + 1)) & 1 : ae;
    const int32_t v = (int32_t)(row + x);
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const uint64_t B = __ballot(b[k]);
        const bool bm = lane > 0 ? (B >> (lane - 1)) & 1 : be[k],
                   bp = lane < 63 ? (B >> (lane + 1)) & 1 : be[k];
        // diagonal rows have no outer bytes: a contact already made at x - 1 in the
        // segment before is then made once more
        const Contact c = contact(a, am, ap, b[k], bm, bp, k < 2);
        const int32_t u = (int32_t)(brow[k] + x);
        ccl_unite_wave<S>(L, c.o, v, u);
        ccl_unite_wave<S>(L, c.p, v, u + 1);
        ccl_unite_wave<S>(L, c.m, v, u - 1);
    }
}

// The links across the segment boundaries of a row, one thread per boundary: along the row
// itself, and diagonally to the two neighbour rows that k_ccl_border leaves out when they
// lie in the same tile.
__global__ __launch_bounds__(256) void k_ccl_cross(Grid g, const uint8_t *__restrict__ pore,
                                                   int32_t *L) {
    constexpr int S = __HIP_MEMORY_SCOPE_AGENT;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int nb = g.nseg - 1;
    if (t >= (int64_t)nb * g.ny * g.nz) return;
    const int64_t r = t / nb;
    const int y = (int)(r % g.ny), z = (int)(r / g.ny);
    const int32_t xr = (int32_t)(r * g.nx) + ((int)(t % nb) + 1) * 64, xl = xr - 1;
    const bool al = pore[xl] != 0, ar = pore[xr] != 0;
    if (!al && !ar) return;
    if (al && ar) ccl_unite<S>(L, xl, xr);
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const bool inside = k == 0 ? y % kTy != kTy - 1 && y != g.ny - 1
                                   : z % kTz != kTz - 1 && z != g.nz - 1;
        if (!inside) continue;
        const int32_t d = k == 0 ? g.nx : g.nx * g.ny;
        const bool bl = pore[xl + d] != 0, br = pore[xr + d] != 0;
        if (al && !ar && !bl && br) ccl_unite<S>(L, xl, xr + d);
        if (ar && !al && !br && bl) ccl_unite<S>(L, xr, xl + d);
    }
}

__global__ __launch_bounds__(256) void k_ccl_faces(Grid g, int32_t *__restrict__ L,
                                                   uint8_t *__restrict__ fin,
                                                   uint8_t *__restrict__ fout) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= (int64_t)g.ny * g.nz) return;
    const int64_t va = k * g.nx, vb = va + g.nx - 1;
    constexpr int S = __HIP_MEMORY_SCOPE_AGENT;
    if (L[va] >= 0) fin[ccl_root<S>(L, (int32_t)va)] = 1;
    if (L[vb] >= 0) fout[ccl_root<S>(L, (int32_t)vb)] = 1;
}

// Final labels (the roots), transport flags and the three counts.  A bounded number of
// workgroups loops over the volume, so that few atomics reach the counters (one per wave
// and counter over the whole volume took 33 ms at 512^3).
constexpr unsigned kFinishBlocks = 2048;
constexpr int kFinishVox = 4;  // voxels a thread follows at a time
__global__ __launch_bounds__(256) void k_ccl_finish(int64_t nv, int32_t *__restrict__ L,
                                                    const uint8_t *__restrict__ fin,
                                                    const uint8_t *__restrict__ fout,
                                                    uint8_t *__restrict__ transport,
                                                    unsigned long long *counts) {
    unsigned c[3] = {0, 0, 0};
    for (int64_t b = blockIdx.x; b * (256 * kFinishVox) < nv; b += gridDim.x) {
        const int64_t v0 = b * (256 * kFinishVox) + threadIdx.x;
        int32_t l[kFinishVox], r[kFinishVox];
#pragma unroll
        for (int k = 0; k < kFinishVox; k++)
            r[k] = l[k] = v0 + 256 * k < nv ? L[v0 + 256 * k] : -1;
        for (bool more = true; more;) {  // parents change to their roots only
            int32_t q[kFinishVox];
#pragma unroll
            for (int k = 0; k < kFinishVox; k++)
                q[k] = r[k] < 0 ? r[k]
                                : __hip_atomic_load(&L[r[k]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            more = false;
#pragma unroll
            for (int k = 0; k < kFinishVox; k++) {
                more |= q[k] != r[k];
                r[k] = q[k];
            }
        }
#pragma unroll
        for (int k = 0; k < kFinishVox; k++) {
            const int64_t v = v0 + 256 * k;
            if (v >= nv) continue;
            bool t = false;
            if (r[k] >= 0) {
                if (r[k] != l[k])
                    __hip_atomic_store(&L[v], r[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                t = fin[r[k]] && fout[r[k]];
                c[0]++;
                c[1] += t;
                c[2] += r[k] == (int32_t)v;
            }
            if (transport) transport[v] = (uint8_t)t;
        }
    }
    __shared__ unsigned lds[kRows][3];
#pragma unroll
    for (int k = 0; k < 3; k++) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) c[k] += __shfl_down(c[k], off, 64);
        if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6][k] = c[k];
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        unsigned long long t = 0;
        for (int w = 0; w < kRows; w++) t += lds[w][threadIdx.x];
        if (t) atomicAdd(&counts[threadIdx.x], t);
    }
}

// ================================================================ 13-direction chords
// Per direction, the pore bits along its lines: 32 consecutive voxels of a line in one
// word.  A direction's primary axis is z if it has a z component, else y, else x (its
// components along the primary axis are taken as +1: a line has no sense); the position
// along the line is the primary coordinate t, and the line's other coordinates are those
// it has at t = 0, taken cyclically (x = (X + sx t) mod nx), so that every direction's
// bits are one rearrangement of the volume.  Where a line leaves the box and enters again
// on the other side a chord ends: k_chords caps every count by the steps to the faces.
//
// One pass forms the words of all directions, one the chords of every voxel: 13 words
// and a count of their ones around the voxel, where walking every line voxel by voxel
// with a read and write of the counts took 13 passes of dependent loads: 13 x 56 us at
// 45 x 37 x 32, now 8.5 + 6.9 us.
struct ChordDir {
    int axis, sx, sy;  // primary axis (0 x, 1 y, 2 z); steps in x and y per step of t
    int cls;           // components: 0 axis, 1 face diagonal, 2 body diagonal
};
#define LBM_DIR13                                                                              \
    constexpr ChordDir kDir13[13] = {{0, 0, 0, 0},  {1, 0, 0, 0},   {2, 0, 0, 0},              \
                                     {1, 1, 0, 1},  {1, -1, 0, 1},  {2, 1, 0, 1},              \
                                     {2, -1, 0, 1}, {2, 0, 1, 1},   {2, 0, -1, 1},             \
                                     {2, 1, 1, 2},  {2, -1, -1, 2}, {2, 1, -1, 2}, {2, -1, 1, 2}};

// Words of the lines of the three primary axes, and the offset of direction d's words.
// Lines of primary axis z in a box one voxel deep hold one voxel each and need no words.
struct ChordWords {
    int nwx, nwy, nwz;     // words along a line
    int64_t cx, cy, cz;    // words of a direction
    __host__ __device__ explicit ChordWords(const Grid &g) {
        nwx = (g.nx + 31) / 32;
        nwy = (g.ny + 31) / 32;
        nwz = (g.nz + 31) / 32;
        cx = (int64_t)nwx * g.ny * g.nz;
        cy = (int64_t)nwy * g.nx * g.nz;
        cz = g.nz > 1 ? (int64_t)nwz * g.nx * g.ny : 0;
    }
    // directions 0 | 1, 3, 4 | 2, 5 .. 12
    __host__ __device__ int64_t base(int d) const {
        return d == 0   ? 0
               : d == 1 ? cx
               : d == 3 ? cx + cy
               : d == 4 ? cx + 2 * cy
                        : cx + 3 * cy + (d == 2 ? 0 : d - 4) * cz;
    }
    __host__ __device__ int64_t total() const { return cx + 3 * cy + 9 * cz; }
};

// blockIdx.y = direction; one thread per word (primary axis y, z: lanes along X, so the
// 32 bytes a thread collects are coalesced over the wave at every t), one wave per 64
// voxels of a row for the x direction (its ballot is two words).
__global__ __launch_bounds__(256) void k_chord_bits(Grid g, const uint8_t *__restrict__ pore,
                                                    uint32_t *__restrict__ words) {
    LBM_DIR13
    const int d = blockIdx.y;
    ChordDir D{0, 0, 0, 0};
#pragma unroll
    for (int k = 1; k < 13; k++)
        if (d == k) D = kDir13[k];
    const ChordWords W(g);
    uint32_t *__restrict__ out = words + W.base(d);
    if (D.axis == 0) {
        const int64_t rows = (int64_t)g.ny * g.nz;
        const int lane = threadIdx.x & 63;
        for (int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < rows; r += (int64_t)gridDim.x * 4)
            for (int x0 = 0; x0 < g.nx; x0 += 64) {
                const int x = x0 + lane;
                const uint64_t w = __ballot(x < g.nx && pore[r * g.nx + x] != 0);
                const int k = x0 / 32 + lane;
                if (lane < 2 && k < W.nwx) out[r * W.nwx + k] = (uint32_t)(w >> (32 * lane));
            }
        return;
    }
    const int n = D.axis == 1 ? g.ny : g.nz;     // along t
    const int m = D.axis == 1 ? g.nz : g.ny;     // the line's second coordinate (z or Y)
    const int nm = (D.axis == 1 ? W.nwy : W.nwz) * m;
    const int lanes = (g.nx + 63) / 64;
    const int lane = threadIdx.x & 63;
    if (D.axis == 2 && W.cz == 0) return;
    // one wave per 64 lines (X) of one (word, second coordinate)
    for (int64_t u = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); u < (int64_t)nm * lanes;
         u += (int64_t)gridDim.x * 4) {
        const int q = (int)(u / lanes), X = (int)(u % lanes) * 64 + lane;
        const int w = q / m, s = q % m, t0 = 32 * w;
        if (X >= g.nx) continue;
        int x = (X + D.sx * (t0 % g.nx) + g.nx) % g.nx;
        int y = D.axis == 1 ? t0 : (s + D.sy * (t0 % g.ny) + g.ny) % g.ny;
        uint32_t b = 0;
        const int tn = n - t0 < 32 ? n - t0 : 32;
#pragma unroll 8
        for (int t = 0; t < tn; t++) {
            const int64_t v = D.axis == 1 ? g.lin(x, y, s) : g.lin(x, y, t0 + t);
            b |= (uint32_t)(pore[v] != 0) << t;
            x += D.sx;
            x = x < 0 ? x + g.nx : (x >= g.nx ? x - g.nx : x);
            if (D.axis == 1) {
                y++;
            } else {
                y += D.sy;
                y = y < 0 ? y + g.ny : (y >= g.ny ? y - g.ny : y);
            }
        }
        out[(int64_t)q * g.nx + X] = b;
    }
}

// Ones in a row from bit t upwards (downwards) of the line whose words lie `stride`
// apart from p, where the word of t, w, is set at t.
__device__ inline int ones_up(const uint32_t *p, int64_t stride, int t, int nw, uint32_t w) {
    const int b = t & 31;
    const uint32_t s = ~(w >> b);  // the b bits shifted in count as the end of the word
    int k = s ? __builtin_ctz(s) : 32;
    if (k < 32 - b) return k;
    for (int j = (t >> 5) + 1; j < nw; j++) {
        const uint32_t v = ~p[j * stride];
        if (v) return k + __builtin_ctz(v);
        k += 32;
    }
    return k;
}
__device__ inline int ones_down(const uint32_t *p, int64_t stride, int t, uint32_t w) {
    const int b = t & 31;
    const uint32_t s = ~(w << (31 - b));
    int k = s ? __builtin_clz(s) : 32;
    if (k < b + 1) return k;
    k = b + 1;
    for (int j = (t >> 5) - 1; j >= 0; j--) {
        const uint32_t v = ~p[j * stride];
        if (v) return k + __builtin_clz(v);
        k += 32;
    }
    return k;
}

__global__ __launch_bounds__(256) void k_chords(Grid g, const uint8_t *__restrict__ pore,
                                                const uint32_t *__restrict__ words, double s2,
                                                double s3, double *__restrict__ diam) {
    const int x = (int)blockIdx.x * 64 + (threadIdx.x & 63),
              y = (int)blockIdx.y * kRows + (threadIdx.x >> 6), z = (int)blockIdx.z;
    if (x >= g.nx || y >= g.ny) return;
    const int64_t v = g.lin(x, y, z);
    if (pore[v] == 0) {
        diam[v] = 0.0;
        return;
    }
    LBM_DIR13
    const ChordWords W(g);
    const int ym = y % g.nx, zmx = z % g.nx, zmy = z % g.ny;
    uint32_t w[13];
    const uint32_t *p[13];
#pragma unroll
    for (int d = 0; d < 13; d++) {
        const ChordDir D = kDir13[d];
        w[d] = 1u;  // a line of one voxel (primary axis z, nz = 1)
        p[d] = words + W.base(d);
        if (D.axis == 0) {
            p[d] += ((int64_t)z * g.ny + y) * W.nwx;
            w[d] = p[d][x >> 5];
        } else if (D.axis == 1 || W.cz != 0) {
            int X = x - D.sx * (D.axis == 1 ? ym : zmx);  // at t = 0, cyclically
            X = X < 0 ? X + g.nx : (X >= g.nx ? X - g.nx : X);
            int s = D.axis == 1 ? z : y - D.sy * zmy;
            if (D.axis == 2) s = s < 0 ? s + g.ny : (s >= g.ny ? s - g.ny : s);
            const int t = D.axis == 1 ? y : z, m = D.axis == 1 ? g.nz : g.ny;
            p[d] += (int64_t)s * g.nx + X;
            w[d] = p[d][(int64_t)(t >> 5) * m * g.nx];
        }
    }
    int sum[3] = {0, 0, 0};
#pragma unroll
    for (int d = 0; d < 13; d++) {
        const ChordDir D = kDir13[d];
        const int t = D.axis == 0 ? x : (D.axis == 1 ? y : z);
        const int n = D.axis == 0 ? g.nx : (D.axis == 1 ? g.ny : g.nz);
        const int64_t stride = D.axis == 0 ? 1 : (int64_t)(D.axis == 1 ? g.nz : g.ny) * g.nx;
        // voxels up to the faces, the voxel itself included
        int cu = n - t, cd = t + 1;
        if (D.sx) {
            const int r = g.nx - x, l = x + 1;
            cu = min(cu, D.sx > 0 ? r : l);
            cd = min(cd, D.sx > 0 ? l : r);
        }
        if (D.sy) {
            const int r = g.ny - y, l = y + 1;
            cu = min(cu, D.sy > 0 ? r : l);
            cd = min(cd, D.sy > 0 ? l : r);
        }
        if (D.axis == 2 && W.cz == 0) {
            sum[D.cls] += 1;
            continue;
        }
        const int nw = D.axis == 0 ? W.nwx : (D.axis == 1 ? W.nwy : W.nwz);
        const int up = min(ones_up(p[d], stride, t, nw, w[d]), cu);
        const int dn = min(ones_down(p[d], stride, t, w[d]), cd);
        sum[D.cls] += up + dn - 1;
    }
    const double a = (double)sum[0], b = (double)sum[1], c = (double)sum[2];
    const double t1 = s2 * b;
    const double t2 = a + t1;
    const double t3 = s3 * c;
    const double t4 = t2 + t3;
    diam[v] = t4 / 13.0;
}

// ================================================================ distance map
// Squared distance to the nearest solid voxel along x: one wave per row, or several short
// rows, from the bits of its segments.  (One thread per row, two scans of it, ran 7.7 ms at 512^3 on
// uncoalesced rows; now 0.28 ms.)
template <int LL>
__global__ __launch_bounds__(256) void k_edt_x(Grid g, int ll, const uint8_t *__restrict__ pore,
                                               int32_t *__restrict__ out, int *__restrict__ emax) {
    __shared__ uint64_t solid[kRows][kMaxEdge / 64];
    const int wave = threadIdx.x >> 6, sh = LL < 0 ? ll : LL;
    const int lane = threadIdx.x & ((1 << sh) - 1), first = (threadIdx.x & 63) - lane;  // of the row
    const int64_t row = ((int64_t)blockIdx.x * kRows + wave) * (64 >> sh) + (first >> sh);
    if (blockIdx.x == 0 && threadIdx.x == 0) *emax = 0;
    const bool live = row < (int64_t)g.ny * g.nz;
    const int64_t base = row * g.nx;
    uint64_t own = 0;  // the solid bits of a row of one segment
    for (int k = 0; k < g.nseg; k++) {
        const int x = k * 64 + lane;
        own = __ballot(live && x < g.nx && pore[base + x] == 0);
        if ((threadIdx.x & 63) == 0) solid[wave][k] = own;
    }
    if (LL < 0) own = own >> first & (~0ull >> (64 - (1 << sh)));
    __syncthreads();
    if (!live) return;
    int left = -kInf;  // last solid before this segment
    for (int k = 0; k < g.nseg; k++) {
        const uint64_t w = LL < 0 ? own : solid[wave][k];  // short rows: of one segment
        int right = kInf;  // first solid after this segment
        for (int j = k + 1; j < g.nseg; j++) {
            const uint64_t n = solid[wave][j];
            if (n) {
                right = j * 64 + __builtin_ctzll(n);
                break;
            }
        }
        const int x = k * 64 + lane;
        const uint64_t below = w & (~0ull >> (63 - lane)), above = w >> lane;
        const int l = below ? k * 64 + 63 - __builtin_clzll(below) : left;
        const int r = above ? x + __builtin_ctzll(above) : right;
        if (x < g.nx) {
            int d = kInf;
            if (l >= 0) d = x - l;
            if (r < kInf && r - x < d) d = r - x;
            out[base + x] = d >= kInf ? kInf : d * d;
        }
        if (w) left = k * 64 + 63 - __builtin_clzll(w);
    }
}

// One more axis of the separable minimum: out(p) = min_t in(p with axis = t) + (p_a - t)^2,
// searched outwards from p until the distance term alone reaches the best value.  Bound by
// the chain of those searches: 0.61-0.67 ms an axis at 512^3 (1.26 ms with one distance at
// a time and the voxel's coordinates from 64-bit divisions).
template <int AXIS, int LL>
__global__ __launch_bounds__(256) void k_edt_axis(Grid g, int ll, const int32_t *__restrict__ in,
                                                  int32_t *__restrict__ out) {
    const int sh = LL < 0 ? ll : LL, rows = 64 >> sh, lane = threadIdx.x & 63;
    const int x = (int)blockIdx.x * 64 + (lane & ((1 << sh) - 1)),
              y = ((int)blockIdx.y * kRows + (threadIdx.x >> 6)) * rows + (lane >> sh), z = (int)blockIdx.z;
    if (x >= g.nx || y >= g.ny) return;
    const int64_t v = g.lin(x, y, z);
    const int64_t stride = AXIS == 1 ? (int64_t)g.nx : (int64_t)g.nx * g.ny;
    const int len = AXIS == 1 ? g.ny : g.nz, p = AXIS == 1 ? y : z;
    int best = in[v];
    // four distances at a time, their loads in flight together (a term beyond the
    // stopping distance is a valid one that cannot win)
    for (int r0 = 1; r0 < len && r0 * r0 < best; r0 += 4) {
        int a[4], b[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int r = r0 + k;
            a[k] = p - r >= 0 ? in[v - r * stride] : kInf;
            b[k] = p + r < len ? in[v + r * stride] : kInf;
        }
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int m = min(a[k], b[k]), r = r0 + k;
            if (m < kInf) best = min(best, m + r * r);
        }
    }
    out[v] = best;
}

// ================================================================ inscribed spheres
// Widest inscribed ball covering each pore voxel: max E(c) over centres c with
// |p - c|^2 < E(c).
//  1. k_mis_centres keeps the centres whose ball no ball of one of the 26 neighbours
//     holds: with v the step to the neighbour and k = |v|^2, every |p|^2 <= E - 1 has
//     |p - v|^2 <= E - 1 + 2 p.v + k <= E - 1 + 2 isqrt(k (E - 1)) + k, so a neighbour
//     with E' >= E + 2 isqrt(k (E - 1)) + k covers all of it.  E' > E, so the balls that
//     are dropped are held by one that is kept.  12 % of the pore voxels of the 128^3
//     workload are kept.  They go to a list per cell of 8^3 voxels.
//  2. k_mis_cover: one workgroup per tile of 32 x 8 x 8 voxels; lane = row of the tile;
//     each wave takes cells in reach of the tile, drops the centres that do not reach it
//     64 at a time, and raises the span of each row inside the ball.  A span of 2^k to
//     2^(k+1) - 1 voxels is two (overlapping) spans of 2^k: table k holds, per start, the
//     largest E of such a span, and the tables are folded downwards at the end.  That is
//     two LDS maxima per row and ball; one per covered voxel took 378 us at 128^3.
// Testing every centre of the cube of half-width sqrt(max E) around each voxel (21^3 at
// 128^3, 43^3 at 512^3) took 4.0 ms and 1034 ms; these two take 0.15 and 5.0 ms.
constexpr int kCell = 8;
constexpr int kMx = 32, kMy = 8, kMz = 8;  // tile of k_mis_cover: 64 rows, one per lane
static_assert(kMy * kMz == 64 && kMx % kCell == 0 && kMy % kCell == 0 && kMz % kCell == 0,
              "one row of the tile per lane, whole cells");

struct CellInfo {
    int32_t count, emax;  // centres of the cell and their largest E
};

// First list entry of cell (cx, cy, cz): the voxels of the cells before it.
__device__ inline int64_t cell_base(const Grid &g, int cx, int cy, int cz) {
    const int hz = min(kCell, g.nz - cz * kCell), hy = min(kCell, g.ny - cy * kCell);
    return (int64_t)g.nx * g.ny * (cz * kCell) + (int64_t)g.nx * (cy * kCell) * hz +
           (int64_t)(cx * kCell) * hy * hz;
}

// floor(sqrt(n)), 0 <= n < 2^24: the binary32 root (v_sqrt_f32, 1 ulp) is within one of it
__device__ inline int isqrt24(int n) {
    int r = (int)__builtin_amdgcn_sqrtf((float)n);
    if (r * r > n) r--;
    if ((r + 1) * (r + 1) <= n) r++;
    return r;
}

// One workgroup (512 threads) per cell.  An entry is E << 9 | local voxel (E < 2^22).
// The largest E of all goes to *emax, one atomic per cell at most (one per wave of the
// last distance pass queued 40 us on the counter at 128^3).  Without a solid voxel every E
// is infinite: then only that is recorded, and the call fails.
__global__ __launch_bounds__(512) void k_mis_centres(Grid g, const int32_t *__restrict__ E,
                                                     int *__restrict__ emax,
                                                     uint32_t *__restrict__ list,
                                                     CellInfo *__restrict__ info) {
    __shared__ int n, m;
    const int cx = blockIdx.x, cy = blockIdx.y, cz = blockIdx.z, t = threadIdx.x;
    const int x = cx * kCell + (t & 7), y = cy * kCell + ((t >> 3) & 7), z = cz * kCell + (t >> 6);
    if (t == 0) n = m = 0;
    __syncthreads();
    bool keep = false;
    int e = 0;
    if (x < g.nx && y < g.ny && z < g.nz) {
        const int64_t v = g.lin(x, y, z);
        e = E[v];
        if (e >= kInf) atomicMax(&m, e);
        if (e > 0 && e < kInf) {
            const int lim[4] = {0, e + 2 * isqrt24(e - 1) + 1, e + 2 * isqrt24(2 * (e - 1)) + 2,
                                e + 2 * isqrt24(3 * (e - 1)) + 3};
            keep = true;
#pragma unroll
            for (int dz = -1; dz <= 1; dz++)
#pragma unroll
                for (int dy = -1; dy <= 1; dy++)
#pragma unroll
                    for (int dx = -1; dx <= 1; dx++) {
                        const int k = dx * dx + dy * dy + dz * dz;
                        if (k == 0) continue;
                        const bool in = x + dx >= 0 && x + dx < g.nx && y + dy >= 0 &&
                                        y + dy < g.ny && z + dz >= 0 && z + dz < g.nz;
                        const int o = in ? E[v + dx + (int64_t)g.nx * (dy + (int64_t)g.ny * dz)] : 0;
                        if (o >= lim[k]) keep = false;
                    }
        }
    }
    if (keep) {
        const int k = atomicAdd(&n, 1);
        atomicMax(&m, e);
        list[cell_base(g, cx, cy, cz) + k] = (uint32_t)e << 9 | (uint32_t)t;
    }
    __syncthreads();
    if (t == 0) {
        info[((int64_t)cz * gridDim.y + cy) * gridDim.x + cx] = CellInfo{n, m};
        if (m > __hip_atomic_load(emax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(emax, m);
    }
}

// Distance from the interval [lo, hi] of integers to a (0 inside).
__device__ inline int gap(int a, int lo, int hi) { return a < lo ? lo - a : (a > hi ? a - hi : 0); }

__global__ __launch_bounds__(512) void k_mis_cover(Grid g, int ncx, int ncy, int ncz,
                                                   const int *__restrict__ emax_d,
                                                   const uint32_t *__restrict__ list,
                                                   const CellInfo *__restrict__ info,
                                                   double *__restrict__ diam) {
    // [level][row][start]; rows padded: the lanes of a wave in different banks
    constexpr int kLev = 6, kRow = kMx + 1, kTab = 64 * kRow;
    static_assert(kMx == 1 << (kLev - 1), "spans of up to a whole row");
    __shared__ int best[kLev * kTab];
    const int emax = *emax_d;
    if (emax >= kInf) return;
    const int lane = threadIdx.x & 63, nwave = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int x0 = (int)blockIdx.x * kMx, y0 = (int)blockIdx.y * kMy, z0 = (int)blockIdx.z * kMz;
    const int x1 = min(x0 + kMx, g.nx) - 1, y1 = min(y0 + kMy, g.ny) - 1, z1 = min(z0 + kMz, g.nz) - 1;
    for (int k = threadIdx.x; k < kLev * kTab; k += blockDim.x) best[k] = 0;
    __syncthreads();
    const int R = emax > 0 ? isqrt24(emax - 1) : 0;  // no ball reaches further
    const int cx0 = max(x0 - R, 0) / kCell, cx1 = min(x1 + R, g.nx - 1) / kCell;
    const int cy0 = max(y0 - R, 0) / kCell, cy1 = min(y1 + R, g.ny - 1) / kCell;
    const int cz0 = max(z0 - R, 0) / kCell, cz1 = min(z1 + R, g.nz - 1) / kCell;
    const int wx = cx1 - cx0 + 1, wy = cy1 - cy0 + 1, cells = wx * wy * (cz1 - cz0 + 1);
    const int ry = y0 + (lane & 7), rz = z0 + (lane >> 3);
    int *row = best + lane * kRow - x0;
    const bool inrow = ry <= y1 && rz <= z1;
    for (int c0 = 0; c0 < cells; c0 += nwave * 64) {
        // 64 cells at a time, dealt to the waves in turn: those whose centres can reach
        // the tile
        const int c = c0 + lane * nwave + wave;
        int cx = 0, cy = 0, cz = 0;
        CellInfo ci{0, 0};
        if (c < cells) {
            cx = cx0 + c % wx;
            cy = cy0 + (c / wx) % wy;
            cz = cz0 + c / (wx * wy);
            ci = info[((int64_t)cz * ncy + cy) * ncx + cx];
            const int gx = max(max(x0 - (cx * kCell + kCell - 1), cx * kCell - x1), 0);
            const int gy = max(max(y0 - (cy * kCell + kCell - 1), cy * kCell - y1), 0);
            const int gz = max(max(z0 - (cz * kCell + kCell - 1), cz * kCell - z1), 0);
            if (gx * gx + gy * gy + gz * gz >= ci.emax) ci.count = 0;
        }
        uint64_t live = __ballot(ci.count > 0);
        while (live) {
            const int s = __builtin_ctzll(live);
            live &= live - 1;
            const int sx = __builtin_amdgcn_readlane(cx, s) * kCell,
                      sy = __builtin_amdgcn_readlane(cy, s) * kCell,
                      sz = __builtin_amdgcn_readlane(cz, s) * kCell;
            const int cnt = __builtin_amdgcn_readlane(ci.count, s);
            const uint32_t *src = list + cell_base(g, sx / kCell, sy / kCell, sz / kCell);
            for (int k0 = 0; k0 < cnt; k0 += 64) {
                const uint32_t e = k0 + lane < cnt ? src[k0 + lane] : 0u;
                const int ex = sx + (int)(e & 7), ey = sy + (int)((e >> 3) & 7),
                          ez = sz + (int)((e >> 6) & 7), E = (int)(e >> 9);
                const int gx = gap(ex, x0, x1), gy = gap(ey, y0, y1), gz = gap(ez, z0, z1);
                uint64_t hit = __ballot(gx * gx + gy * gy + gz * gz < E);
                while (hit) {
                    const int h = __builtin_ctzll(hit);
                    hit &= hit - 1;
                    const uint32_t f = (uint32_t)__builtin_amdgcn_readlane((int)e, h);
                    const int fx = sx + (int)(f & 7), fy = sy + (int)((f >> 3) & 7),
                              fz = sz + (int)((f >> 6) & 7), F = (int)(f >> 9);
                    const int dy = ry - fy, dz = rz - fz, rem = F - 1 - dy * dy - dz * dz;
                    if (rem >= 0 && inrow) {
                        const int w = isqrt24(rem);
                        const int lo = max(fx - w, x0), hi = min(fx + w, x1);
                        if (lo <= hi) {
                            const int lev = 31 - __builtin_clz(hi - lo + 1);
                            int *tab = row + lev * kTab;
                            atomicMax(&tab[lo], F);
                            atomicMax(&tab[hi + 1 - (1 << lev)], F);
                        }
                    }
                }
            }
        }
    }
    __syncthreads();
    for (int lev = kLev - 1; lev > 0; lev--) {  // a span of 2^lev is two of 2^(lev - 1)
        const int h = 1 << (lev - 1);
        const int *up = best + lev * kTab;
        int *lo = best + (lev - 1) * kTab;
        for (int k = threadIdx.x; k < 64 * kMx; k += blockDim.x) {
            const int r = k / kMx, x = k % kMx, i = r * kRow + x;
            lo[i] = max(lo[i], max(up[i], x >= h ? up[i - h] : 0));
        }
        __syncthreads();
    }
    // 2 sqrt(E) - 1 (the correctly rounded root); no ball covers a solid voxel
    for (int k = threadIdx.x; k < 64 * kMx; k += blockDim.x) {
        const int r = k / kMx, x = x0 + k % kMx, y = y0 + (r & 7), z = z0 + (r >> 3);
        if (x > x1 || y > y1 || z > z1) continue;
        const int e = best[r * kRow + k % kMx];
        diam[g.lin(x, y, z)] = e > 0 ? 2.0 * __dsqrt_rn((double)e) - 1.0 : 0.0;
    }
}

}  // namespace lbm

using namespace lbm;

static lbm_status check_n(const int32_t n[3]) {
    LBM_REQUIRE(n, LBM_E_INVAL, "null size");
    LBM_REQUIRE(n[0] >= 1 && n[1] >= 1 && n[2] >= 1 && n[0] <= kMaxEdge && n[1] <= kMaxEdge &&
                    n[2] <= kMaxEdge,
                LBM_E_INVAL, "sizes must lie in [1, %d]", kMaxEdge);
    return LBM_OK;
}

namespace lbm {
size_t label_ws_bytes_n(const int32_t n[3]) {
    Grid g = make_grid(n);
    Carver c(nullptr);
    c.take<unsigned long long>(4);
    c.take<uint8_t>(g.nvox());
    c.take<uint8_t>(g.nvox());
    return c.off;
}
size_t diam_ws_bytes_n(const int32_t n[3]) {
    Grid g = make_grid(n);
    Carver c(nullptr);
    c.take<unsigned long long>(4);
    const size_t cells = (size_t)((g.nx + kCell - 1) / kCell) * ((g.ny + kCell - 1) / kCell) *
                         ((g.nz + kCell - 1) / kCell);
    Carver chords = c;
    c.take<int32_t>(g.nvox());
    c.take<int32_t>(g.nvox());
    c.take<CellInfo>(cells);
    chords.take<uint32_t>((size_t)ChordWords(g).total());
    // never below the 12 bytes a voxel that this workspace has always asked for
    return std::max({c.off, chords.off, 12 * (size_t)g.nvox()});
}
}  // namespace lbm

namespace lbm {
// The labelling passes on scratch holding 4 counters and two voxel flag arrays (cleared by
// the kernels that need them), then the stats (host sync).
static lbm_status label_run(const Grid &g, const uint8_t *pore, int32_t *label, uint8_t *transport,
                            lbm_label_stats *stats_h, unsigned long long *counts, uint8_t *fin,
                            uint8_t *fout, hipStream_t s) {
    const int64_t nv = g.nvox();
    k_ccl_tile<<<dim3((unsigned)g.nseg, (unsigned)((g.ny + kTy - 1) / kTy),
                      (unsigned)((g.nz + kTz - 1) / kTz)),
                 kTileWaves * 64, 0, s>>>(g, pore, label, fin, fout, counts);
    LBM_CHECK_LAUNCH();
    k_ccl_border<<<row_grid(g), 256, 0, s>>>(g, pore, label);
    LBM_CHECK_LAUNCH();
    if (g.nseg > 1) {
        const int64_t nb = (int64_t)(g.nseg - 1) * g.ny * g.nz;
        k_ccl_cross<<<(unsigned)((nb + 255) / 256), 256, 0, s>>>(g, pore, label);
        LBM_CHECK_LAUNCH();
    }
    k_ccl_faces<<<(unsigned)(((int64_t)g.ny * g.nz + 255) / 256), 256, 0, s>>>(g, label, fin, fout);
    LBM_CHECK_LAUNCH();
    k_ccl_finish<<<(unsigned)std::min<int64_t>((nv + 1023) / 1024, kFinishBlocks), 256, 0, s>>>(
        nv, label, fin, fout, transport, counts);
    LBM_CHECK_LAUNCH();
    unsigned long long h[3];
    LBM_TRY_HIP(hipMemcpyAsync(h, counts, sizeof(h), hipMemcpyDeviceToHost, s));
    LBM_TRY_HIP(hipStreamSynchronize(s));
    stats_h->n_pore = (int64_t)h[0];
    stats_h->n_transport = (int64_t)h[1];
    stats_h->n_components = (int64_t)h[2];
    stats_h->porosity = (double)h[0] / (double)nv;
    stats_h->connectivity = h[0] ? (double)h[1] / (double)h[0] : 0.0;
    return LBM_OK;
}

// Scratch of lbm_label_noalloc: 256 bytes of counters and the two face-flag arrays of a
// volume of up to LBM_LABEL_NOALLOC_MAX_VOXELS voxels (32 MiB + 256 B in all), one copy per
// device for the life of the process.  Host code uses the per-device address from
// hipGetSymbolAddress, never the symbol itself.
constexpr int64_t kNoallocVox = LBM_LABEL_NOALLOC_MAX_VOXELS;
static __device__ __align__(256) uint8_t scratch[256 + 2 * kNoallocVox];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices];

static lbm_status scratch_address(void **out) {
    int dev = -1;
    LBM_TRY_HIP(hipGetDevice(&dev));
    LBM_REQUIRE(dev >= 0 && dev < kMaxDevices, LBM_E_DEVICE, "device %d beyond the scratch table", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        LBM_TRY_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        LBM_REQUIRE(p, LBM_E_DEVICE, "no address for the scratch array on device %d", dev);
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return LBM_OK;
}
}  // namespace lbm

extern "C" lbm_status lbm_label(const int32_t n[3], const uint8_t *pore, int32_t *label,
                                uint8_t *transport, lbm_label_stats *stats_h, void *workspace,
                                size_t ws_bytes, void *stream) {
    lbm_status st = check_n(n);
    if (st != LBM_OK) return st;
    LBM_REQUIRE(pore && label && stats_h && workspace, LBM_E_INVAL, "lbm_label: null argument");
    LBM_REQUIRE(ws_bytes >= label_ws_bytes_n(n), LBM_E_NOMEM, "lbm_label: workspace too small");
    st = check_device();
    if (st != LBM_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Grid g = make_grid(n);
    Carver c(workspace);
    unsigned long long *counts = c.take<unsigned long long>(4);
    uint8_t *fin = c.take<uint8_t>(g.nvox());
    uint8_t *fout = c.take<uint8_t>(g.nvox());
    return label_run(g, pore, label, transport, stats_h, counts, fin, fout, s);
}

extern "C" lbm_status lbm_label_noalloc(const int32_t n[3], const uint8_t *pore, int32_t *label,
                                        uint8_t *transport, lbm_label_stats *stats_h,
                                        void *stream) {
    lbm_status st = check_n(n);
    if (st != LBM_OK) return st;
    LBM_REQUIRE(pore && label && stats_h, LBM_E_INVAL, "lbm_label_noalloc: null argument");
    const Grid g = make_grid(n);
    LBM_REQUIRE(g.nvox() <= kNoallocVox, LBM_E_NOMEM,
                "lbm_label_noalloc: %lld voxels exceed its scratch of %lld voxels",
                (long long)g.nvox(), (long long)kNoallocVox);
    st = check_device();
    if (st != LBM_OK) return st;
    void *base = nullptr;
    st = scratch_address(&base);
    if (st != LBM_OK) return st;
    uint8_t *b = static_cast<uint8_t *>(base);
    return label_run(g, pore, label, transport, stats_h, reinterpret_cast<unsigned long long *>(b),
                     b + 256, b + 256 + g.nvox(), static_cast<hipStream_t>(stream));
}

extern "C" lbm_status lbm_pore_diameter(const int32_t n[3], const uint8_t *pore, int32_t method,
                                        double *diam, void *workspace, size_t ws_bytes,
                                        void *stream) {
    lbm_status st = check_n(n);
    if (st != LBM_OK) return st;
    LBM_REQUIRE(pore && diam && workspace, LBM_E_INVAL, "lbm_pore_diameter: null argument");
    LBM_REQUIRE(method == LBM_PSD_CHORD13 || method == LBM_PSD_MIS, LBM_E_INVAL,
                "unknown pore-size method %d", method);
    LBM_REQUIRE(ws_bytes >= diam_ws_bytes_n(n), LBM_E_NOMEM, "lbm_pore_diameter: workspace too small");
    st = check_device();
    if (st != LBM_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Grid g = make_grid(n);
    const int64_t nv = g.nvox();
    Carver c(workspace);
    int *emax_d = reinterpret_cast<int *>(c.take<unsigned long long>(4));
    if (method == LBM_PSD_CHORD13) {
        uint32_t *words = c.take<uint32_t>((size_t)ChordWords(g).total());
        // word and row counts differ by direction: a grid-stride loop over at most this many
        const unsigned nb = (unsigned)std::min<int64_t>((nv / 32 + 255) / 256 + 16, 4096);
        k_chord_bits<<<dim3(nb, 13), 256, 0, s>>>(g, pore, words);
        LBM_CHECK_LAUNCH();
        k_chords<<<row_grid(g), 256, 0, s>>>(g, pore, words, std::sqrt(2.0), std::sqrt(3.0), diam);
        LBM_CHECK_LAUNCH();
        LBM_TRY_HIP(hipStreamSynchronize(s));
        return LBM_OK;
    }
    // maximum inscribed sphere; the largest E stays on the device until the end, where it
    // also tells a domain without solid voxels (E infinite) from the others
    const int ncx = (g.nx + kCell - 1) / kCell, ncy = (g.ny + kCell - 1) / kCell,
              ncz = (g.nz + kCell - 1) / kCell;
    int32_t *a = c.take<int32_t>(nv);
    int32_t *b = c.take<int32_t>(nv);
    CellInfo *info = c.take<CellInfo>((size_t)ncx * ncy * ncz);
    const int ll = lane_log(g);
    const int64_t rows = kRows << (6 - ll);
    const unsigned row_blocks = (unsigned)(((int64_t)g.ny * g.nz + rows - 1) / rows);
    if (ll == 6) {
        k_edt_x<6><<<row_blocks, 256, 0, s>>>(g, ll, pore, a, emax_d);
        LBM_CHECK_LAUNCH();
        k_edt_axis<1, 6><<<row_grid(g), 256, 0, s>>>(g, ll, a, b);
        LBM_CHECK_LAUNCH();
        k_edt_axis<2, 6><<<row_grid(g), 256, 0, s>>>(g, ll, b, a);
    } else {
        k_edt_x<-1><<<row_blocks, 256, 0, s>>>(g, ll, pore, a, emax_d);
        LBM_CHECK_LAUNCH();
        const dim3 grid(1, (unsigned)((g.ny + rows - 1) / rows), (unsigned)g.nz);
        k_edt_axis<1, -1><<<grid, 256, 0, s>>>(g, ll, a, b);
        LBM_CHECK_LAUNCH();
        k_edt_axis<2, -1><<<grid, 256, 0, s>>>(g, ll, b, a);
    }
    LBM_CHECK_LAUNCH();
    uint32_t *list = reinterpret_cast<uint32_t *>(b);
    k_mis_centres<<<dim3((unsigned)ncx, (unsigned)ncy, (unsigned)ncz), 512, 0, s>>>(g, a, emax_d, list,
                                                                                   info);
    LBM_CHECK_LAUNCH();
    k_mis_cover<<<dim3((unsigned)((g.nx + kMx - 1) / kMx), (unsigned)((g.ny + kMy - 1) / kMy),
                       (unsigned)((g.nz + kMz - 1) / kMz)),
                  512, 0, s>>>(g, ncx, ncy, ncz, emax_d, list, info, diam);
    LBM_CHECK_LAUNCH();
    int emax = 0;
    LBM_TRY_HIP(hipMemcpyAsync(&emax, emax_d, sizeof(int), hipMemcpyDeviceToHost, s));
    LBM_TRY_HIP(hipStreamSynchronize(s));
    LBM_REQUIRE(emax < kInf, LBM_E_INVAL, "the domain holds no solid voxel: no distance map");
    return LBM_OK;
}
