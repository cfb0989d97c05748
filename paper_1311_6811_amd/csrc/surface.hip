// The step after the posterior (Sec. 2.2.2, last paragraph; Sec. 3.3.3 steps
// d and e): smoothing of the occupancy probabilities, thresholding, and removal
// of the voxels inside the body, leaving the surface voxels as a compact list.
//   smooth_kernel          3x3x3 mean over the in-grid neighbours and the
//                          threshold in one traversal (the paper merges
//                          smoothing with voxel generation to save a round
//                          trip through memory)
//   surface_flag_kernel    surface flag of every voxel (occupied, with an
//                          unoccupied or out-of-grid face neighbour) and, per
//                          block of kSurfBlock consecutive voxels, their count
//                          (surface_flag_words_kernel: the same, four voxels
//                          per lane, when rows are whole 4-byte words)
//   surface_scan_kernel    (grids of more than kScanMin blocks) the block
//                          offsets: exclusive prefix of the counts, one
//                          workgroup
//   surface_write          the flagged voxels' linear indices at their place
//                          in the ascending list (block offset = sum of the
//                          earlier blocks' counts, summed by each block itself
//                          on smaller grids)
// The paper keeps inner-voxel removal on the CPU; here it is a deterministic
// two-kernel stream compaction over a flag grid.
#include "kernels_common.h"

namespace psfs {
namespace {

using dev::f32x4;
using dev::xcd_remap;

constexpr int kPieceY = 2, kPieceZ = 2;             // rows and planes per smoothing lane (smooth4_kernel)
constexpr int kTileY = 4;                           // rows per smoothing wave
constexpr int kTileZ = 2;                           // planes per smoothing wave
constexpr int kSurfBlock = 4096;                    // voxels per compaction block (16 per lane)
constexpr int kPerLane = kSurfBlock / 256;
constexpr int kScanThreads = 1024;
constexpr int kScanMin = 4096;                      // more blocks: offsets from surface_scan_kernel

__device__ __forceinline__ uint32_t byte_at(uint32_t w, int b) { return (w >> (8 * b)) & 0xffu; }

// A smoothing launch is as wide as kSmoothWide workgroups at most: an axis of
// 2^32 lanes or more is refused, which thin grids of many planes reach (1 x 1 x 2^25
// voxels).
constexpr int64_t kSmoothWide = int64_t(1) << 20;

// Workgroup of a smoothing launch; those past the last tile have nothing to do.
__device__ __forceinline__ uint32_t smooth_group() { return blockIdx.y * gridDim.x + blockIdx.x; }

// 3x3x3 mean over the in-grid neighbours and threshold. A wave owns a tile of
// 64 x-columns (one per lane) by TY rows by TZ planes. It loads the x-windows
// of the TY + 2 rows by TZ + 2 planes it needs at clamped in-grid addresses, all
// before the first is used (a row of the wave per load): with a branch around
// each out-of-grid row the wave waited for one row after another: 13.1 us at
// 128^3, now 8.6 us (rows that are not whole 16-byte pieces). The tiles of one
// XCD form one z-slab, so that its L2 serves the neighbours' rows. Then each row's 3 x 3 window sum (rows dy = -1..1, in
// each row dx = -1..1) and the sum of three planes; out-of-grid cells are left
// out and the sum is divided by the number of in-grid cells. Every voxel's
// additions run in one fixed order.
template <int TY, int TZ>
__global__ __launch_bounds__(256) void smooth_kernel(SurfArgs a)
{
    const uint32_t nxb = (static_cast<uint32_t>(a.nx) + 63) / 64, nyb = (static_cast<uint32_t>(a.ny) + TY - 1) / TY;
    const uint32_t per_z = (nxb * nyb + 3) / 4, nzb = (static_cast<uint32_t>(a.nz) + TZ - 1) / TZ;
    if (smooth_group() >= per_z * nzb) return;
    const uint32_t b = static_cast<uint32_t>(xcd_remap(smooth_group(), static_cast<int64_t>(per_z) * nzb)), bz = b / per_z;
    // the wave's tile and rows in scalar registers (tile counts are below 2^31)
    const uint32_t tile = (b - bz * per_z) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (tile >= nxb * nyb) return;                                  // whole waves
    const int y0 = static_cast<int>(tile / nxb) * TY;
    const int x = static_cast<int>(tile % nxb) * 64 + static_cast<int>(threadIdx.x & 63);
    if (x >= a.nx) return;
    const int z0 = static_cast<int>(bz) * TZ;
    const int64_t plane = static_cast<int64_t>(a.nx) * a.ny;
    const bool xl = x > 0, xr = x + 1 < a.nx;
    const uint32_t c0 = static_cast<uint32_t>(x), cl = xl ? c0 - 1 : c0, cr = xr ? c0 + 1 : c0;
    float v[TZ + 2][TY + 2][3];
#pragma unroll
    for (int q = 0; q < TZ + 2; ++q) {
        const int z = min(max(z0 - 1 + q, 0), a.nz - 1);
#pragma unroll
        for (int r = 0; r < TY + 2; ++r) {
            const int y = min(max(y0 - 1 + r, 0), a.ny - 1);
            const float *p = a.post + (z * plane + static_cast<int64_t>(y) * a.nx);
            v[q][r][0] = p[cl];
            v[q][r][1] = p[c0];
            v[q][r][2] = p[cr];
        }
    }
    // sum of the 3 x 3 window of every output row of the tile in plane z0 - 1 + q
    float w[TZ + 2][TY];
#pragma unroll
    for (int q = 0; q < TZ + 2; ++q) {
        const int z = z0 - 1 + q;
        const bool zin = z >= 0 && z < a.nz;
        float row[TY + 2];
#pragma unroll
        for (int r = 0; r < TY + 2; ++r) {
            float t = v[q][r][1];
            t = xl ? v[q][r][0] + t : t;
            t = xr ? t + v[q][r][2] : t;
            row[r] = t;
        }
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const int y = y0 + r;
            float s = 0.0f;
            s = y > 0 ? s + row[r] : s;
            s += row[r + 1];
            s = y + 1 < a.ny ? s + row[r + 2] : s;
            w[q][r] = zin ? s : 0.0f;
        }
    }
    const int cx = xl + 1 + xr;
#pragma unroll
    for (int q = 0; q < TZ; ++q) {
        const int z = z0 + q;
        if (z >= a.nz) break;
        const int cz = (z > 0) + 1 + (z + 1 < a.nz);
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const int y = y0 + r;
            if (y >= a.ny) break;
            const int c = cx * ((y > 0) + 1 + (y + 1 < a.ny)) * cz;
            const float m = ((w[q][r] + w[q + 1][r]) + w[q + 2][r]) / static_cast<float>(c);
            const int64_t row = z * plane + static_cast<int64_t>(y) * a.nx;
            if (a.smoothed) (a.smoothed + row)[c0] = m;
            (a.occ + row)[c0] = m > a.tau ? 1 : 0;
        }
    }
}

// The value of lane l - 1 / l + 1 (0 in the wave's first / last lane).
__device__ __forceinline__ float from_left(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float from_right(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, false));
}

// smooth_kernel for rows of whole 16-byte pieces (nx a multiple of 4, arrays
// aligned): a lane owns 4 voxels of TY rows by TZ planes, groups of LX lanes a
// span of 4 LX voxels, so a row of the tile is one 16-byte load per lane. The
// x-neighbours come from the adjacent lanes, at a group's ends from a load of
// their own. The same additions in the same order. Bound by the accesses of
// its loads: a wave of smooth_kernel makes 14 64-byte accesses per row of 64
// voxels, here 16 to 18 serve 256; 7.6 us at 128^3 (1 x 2, 2 x 1 and 1 x 4 rows x
// planes per lane: 7.8, 8.0, 7.4 us), of which 19 MB take 3.7 us at the copy rate.
template <int LX, int TY, int TZ>
__global__ __launch_bounds__(256) void smooth4_kernel(SurfArgs a)
{
    constexpr int kRows = 64 / LX * TY;                 // rows of a wave
    const uint32_t nx = static_cast<uint32_t>(a.nx), ny = static_cast<uint32_t>(a.ny), nz = static_cast<uint32_t>(a.nz);
    const uint32_t nxb = (nx + 4 * LX - 1) / (4 * LX), nyb = (ny + kRows - 1) / kRows;
    const uint32_t per_z = (nxb * nyb + 3) / 4, nzb = (nz + TZ - 1) / TZ;
    if (smooth_group() >= per_z * nzb) return;
    const uint32_t b = static_cast<uint32_t>(xcd_remap(smooth_group(), static_cast<int64_t>(per_z) * nzb)), bz = b / per_z;
    const uint32_t tile = (b - bz * per_z) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (tile >= nxb * nyb) return;                      // whole waves
    const uint32_t lane = threadIdx.x & 63, lx = lane % LX, ly = lane / LX;
    const uint32_t ty = tile / nxb, x = (tile - ty * nxb) * (4 * LX) + 4 * lx, y0 = ty * kRows + ly * TY, z0 = bz * TZ;
    const bool in = x < nx && y0 < ny;                  // the others load their clamped neighbours' values
    const uint32_t xc = x < nx ? x : nx - 4;
    const uint32_t plane = nx * ny;
    const bool first = lx == 0, last = lx == LX - 1;
    const bool xl = x > 0, xr = x + 4 < nx;             // neighbours beyond the lane's 4 voxels lie in the grid
    const bool ends = nx > 4 * LX;                      // a group's ends can lie inside the grid
    const uint32_t xe = first ? (xl ? xc - 1 : xc) : (xr ? xc + 4 : xc);
    f32x4 v[TZ + 2][TY + 2];
    float edge[TZ + 2][TY + 2];
#pragma unroll
    for (int q = 0; q < TZ + 2; ++q) {
        const uint32_t z = min(max(static_cast<int>(z0) - 1 + q, 0), static_cast<int>(nz) - 1);
        const float *p = a.post + static_cast<int64_t>(z) * plane;
#pragma unroll
        for (int r = 0; r < TY + 2; ++r) {
            const uint32_t y = min(max(static_cast<int>(y0) - 1 + r, 0), static_cast<int>(ny) - 1);
            v[q][r] = *reinterpret_cast<const f32x4 *>(p + (y * nx + xc));
            edge[q][r] = 0.0f;
            if (ends && (first || last)) edge[q][r] = p[y * nx + xe];
        }
    }
    f32x4 w[TZ + 2][TY];
#pragma unroll
    for (int q = 0; q < TZ + 2; ++q) {
        const int z = static_cast<int>(z0) - 1 + q;
        const bool zin = z >= 0 && z < static_cast<int>(nz);
        f32x4 row[TY + 2];
#pragma unroll
        for (int r = 0; r < TY + 2; ++r) {
            const f32x4 c = v[q][r];
            const float fl = from_left(c.w), fr = from_right(c.x);
            const float l = first ? edge[q][r] : fl, g = last ? edge[q][r] : fr;
            f32x4 t = c;
            t.x = xl ? l + t.x : t.x;
            t.y = c.x + t.y;
            t.z = c.y + t.z;
            t.w = c.z + t.w;
            t.x = t.x + c.y;
            t.y = t.y + c.z;
            t.z = t.z + c.w;
            t.w = xr ? t.w + g : t.w;
            row[r] = t;
        }
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const uint32_t y = y0 + r;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float s = 0.0f;
                s = y > 0 ? s + row[r][e] : s;
                s += row[r + 1][e];
                s = y + 1 < ny ? s + row[r + 2][e] : s;
                w[q][r][e] = zin ? s : 0.0f;
            }
        }
    }
    if (!in) return;
#pragma unroll
    for (int q = 0; q < TZ; ++q) {
        const uint32_t z = z0 + q;
        if (z >= nz) break;
        const int cz = (z > 0) + 1 + (z + 1 < nz);
#pragma unroll
        for (int r = 0; r < TY; ++r) {
            const uint32_t y = y0 + r;
            if (y >= ny) break;
            const int cyz = ((y > 0) + 1 + (y + 1 < ny)) * cz;
            f32x4 m;
            uint32_t o = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int cx = (e > 0 || xl) + 1 + (e < 3 || xr);
                m[e] = ((w[q][r][e] + w[q + 1][r][e]) + w[q + 2][r][e]) / static_cast<float>(cx * cyz);
                o |= (m[e] > a.tau ? 1u : 0u) << (8 * e);
            }
            const int64_t base = static_cast<int64_t>(z) * plane;
            if (a.smoothed) *reinterpret_cast<f32x4 *>(a.smoothed + base + (y * nx + x)) = m;
            *reinterpret_cast<uint32_t *>(a.occ + base + (y * nx + x)) = o;
        }
    }
}

// Surface flags of one compaction block and its count. Lane l of wave w
// tests voxels base + 256 r + 64 w + l (coalesced neighbour loads); the
// lane's (i, j, k) is divided out once and then advanced by 256 voxels per
// step with the carries the host precomputed.
__global__ __launch_bounds__(256) void surface_flag_kernel(SurfArgs a)
{
    __shared__ int part[4];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kSurfBlock;
    const int64_t v0 = base + threadIdx.x;
    const int64_t plane = static_cast<int64_t>(a.nx) * a.ny;
    int k = static_cast<int>(v0 / plane);
    const int64_t rem = v0 - static_cast<int64_t>(k) * plane;
    int j = static_cast<int>(rem / a.nx);
    int i = static_cast<int>(rem - static_cast<int64_t>(j) * a.nx);
    int c = 0;
#pragma unroll
    for (int r = 0; r < kPerLane; ++r) {
        const int64_t v = v0 + 256 * r;
        if (v < a.nvox) {
            // all seven loads at in-grid addresses (a face on the grid's border
            // reads the voxel itself, the border test decides there), issued
            // together rather than one after another
            const bool border = (i == 0) | (i + 1 == a.nx) | (j == 0) | (j + 1 == a.ny) | (k == 0) | (k + 1 == a.nz);
            const uint8_t o = a.occ[v];
            const uint8_t xm = a.occ[i > 0 ? v - 1 : v], xp = a.occ[i + 1 < a.nx ? v + 1 : v];
            const uint8_t ym = a.occ[j > 0 ? v - a.nx : v], yp = a.occ[j + 1 < a.ny ? v + a.nx : v];
            const uint8_t zm = a.occ[k > 0 ? v - plane : v], zp = a.occ[k + 1 < a.nz ? v + plane : v];
            const bool hole = (xm == 0) | (xp == 0) | (ym == 0) | (yp == 0) | (zm == 0) | (zp == 0);
            const bool surf = (o != 0) & (border | hole);
            a.flags[v] = surf ? 1 : 0;
            c += surf;
        }
        i += a.step_i;
        if (i >= a.nx) {
            i -= a.nx;
            ++j;
        }
        j += a.step_j;
        if (j >= a.ny) {
            j -= a.ny;
            ++k;
        }
        k += a.step_k;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) a.counts[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// Surface flags four voxels at a time, when nx is a multiple of 4 and the
// occupancy and flag arrays are 4-byte aligned: lane l tests the four voxels of
// word g = block * 1024 + l (one row, one plane). Their x-neighbours are in the
// same word or in the adjacent words of the row, their y- and z-neighbours in
// the words nx / 4 and nx * ny / 4 away; seven word loads at clamped in-grid
// addresses (the border tests decide for faces on the grid's border), one word
// store of four flags. Bound by latency: a lane with four words, one after
// another, and 64-bit divisions took 5.9 us at 128^3, this 4.5-5.2 us.
__global__ __launch_bounds__(kSurfBlock / 4) void surface_flag_words_kernel(SurfArgs a)
{
    constexpr int kWaves = kSurfBlock / 4 / 64;
    __shared__ int part[kWaves];
    const uint32_t *occ = reinterpret_cast<const uint32_t *>(a.occ);
    uint32_t *flags = reinterpret_cast<uint32_t *>(a.flags);
    // word counts are below 2^29: 32-bit arithmetic
    const uint32_t nwords = static_cast<uint32_t>(a.nvox / 4), rw = static_cast<uint32_t>(a.nx / 4);
    const uint32_t pw = rw * static_cast<uint32_t>(a.ny);
    const uint32_t block = static_cast<uint32_t>(xcd_remap(blockIdx.x, a.nblocks));
    const uint32_t g = block * (kSurfBlock / 4) + threadIdx.x;
    int c = 0;
    if (g < nwords) {
        const uint32_t k = g / pw, rem = g - k * pw, j = rem / rw, i0 = 4 * (rem - j * rw);
        const uint32_t C = occ[g];
        const uint32_t L = occ[i0 > 0 ? g - 1 : g], R = occ[i0 + 4 < static_cast<uint32_t>(a.nx) ? g + 1 : g];
        const uint32_t YM = occ[j > 0 ? g - rw : g], YP = occ[j + 1 < static_cast<uint32_t>(a.ny) ? g + rw : g];
        const uint32_t ZM = occ[k > 0 ? g - pw : g], ZP = occ[k + 1 < static_cast<uint32_t>(a.nz) ? g + pw : g];
        const bool border_yz = (j == 0) | (j + 1 == static_cast<uint32_t>(a.ny)) | (k == 0) |
                               (k + 1 == static_cast<uint32_t>(a.nz));
        uint32_t word = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t o = byte_at(C, b);
            const uint32_t xm = b > 0 ? byte_at(C, b - 1) : byte_at(L, 3);
            const uint32_t xp = b < 3 ? byte_at(C, b + 1) : byte_at(R, 0);
            const bool border = border_yz | (b == 0 && i0 == 0) | (b == 3 && i0 + 4 == static_cast<uint32_t>(a.nx));
            const uint32_t ym = byte_at(YM, b), yp = byte_at(YP, b), zm = byte_at(ZM, b), zp = byte_at(ZP, b);
            const bool hole = (xm == 0) | (xp == 0) | (ym == 0) | (yp == 0) | (zm == 0) | (zp == 0);
            const bool surf = (o != 0) & (border | hole);
            word |= (surf ? 1u : 0u) << (8 * b);
            c += surf;
        }
        flags[g] = word;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x < 64) {
        int t = threadIdx.x < kWaves ? part[threadIdx.x] : 0;
#pragma unroll
        for (int d = kWaves / 2; d > 0; d >>= 1) t += __shfl_xor(t, d, 64);
        if (threadIdx.x == 0) a.counts[block] = t;
    }
}

// Lane l of a compaction block owns its 16 consecutive voxels
// base + 16 l .. base + 16 l + 15 (one 16-byte load of flags).
__device__ __forceinline__ uint32_t lane_flags(const SurfArgs &a, int64_t base)
{
    const int64_t v = base + 16 * static_cast<int64_t>(threadIdx.x);
    uint32_t bits = 0;
    if (v + 16 <= a.nvox) {
        const uint4 w = *reinterpret_cast<const uint4 *>(a.flags + v);
        const uint32_t word[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < 16; ++q)
            if ((word[q >> 2] >> (8 * (q & 3))) & 0xffu) bits |= 1u << q;
    } else {
        for (int q = 0; q < 16 && v + q < a.nvox; ++q)
            if (a.flags[v + q]) bits |= 1u << q;
    }
    return bits;
}

// Inclusive sum over the block's 256 lanes in lane order (wave scans + the
// totals of the waves before).
__device__ __forceinline__ int block_inclusive_scan(int x, int *wave_tot)
{
    const int lane = static_cast<int>(threadIdx.x & 63), w = static_cast<int>(threadIdx.x >> 6);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) wave_tot[w] = x;
    __syncthreads();
    for (int q = 0; q < w; ++q) x += wave_tot[q];
    return x;
}

// Exclusive prefix of the block counts, written over them as offsets, and the
// total: one workgroup; thread t owns a contiguous range of blocks, so the
// additions run in block order within a range and in thread order across the
// ranges (offsets are below nvox < 2^31).
__global__ __launch_bounds__(kScanThreads) void surface_scan_kernel(SurfArgs a)
{
    __shared__ int64_t part[kScanThreads];
    const int t = static_cast<int>(threadIdx.x);
    const int64_t per = (static_cast<int64_t>(a.nblocks) + kScanThreads - 1) / kScanThreads;
    const int64_t lo = t * per < a.nblocks ? t * per : a.nblocks;
    const int64_t hi = lo + per < a.nblocks ? lo + per : a.nblocks;
    int64_t s = 0;
    for (int64_t q = lo; q < hi; ++q) s += a.counts[q];
    part[t] = s;
    __syncthreads();
    for (int d = 1; d < kScanThreads; d <<= 1) {
        const int64_t add = t >= d ? part[t - d] : 0;
        __syncthreads();
        part[t] += add;
        __syncthreads();
    }
    int64_t run = part[t] - s;
    for (int64_t q = lo; q < hi; ++q) {
        const int32_t c = a.counts[q];
        a.counts[q] = static_cast<int32_t>(run);
        run += c;
    }
    if (t == kScanThreads - 1) *a.count = part[t];
}

// Block b's offset summed by the block itself over the earlier blocks' counts
// (and, in block 0, the total into *count); every thread of the block calls it.
__device__ __forceinline__ int64_t own_block_offset(const SurfArgs &a, int b, int64_t *red)
{
    // block 0 sums every count (its own offset is 0), the others those before them
    const int n = b == 0 ? a.nblocks : b;
    int64_t s = 0;
    for (int q = static_cast<int>(threadIdx.x); q < n; q += 256) s += a.counts[q];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    s = (red[0] + red[1]) + (red[2] + red[3]);
    if (b == 0) {
        if (threadIdx.x == 0) *a.count = s;
        return 0;
    }
    return s;
}

// scanned: the counts already hold the block offsets (surface_scan_kernel)
__global__ __launch_bounds__(256) void surface_write_kernel(SurfArgs a, int scanned)
{
    __shared__ int64_t red[4];
    __shared__ int wave_tot[4];
    const int b = static_cast<int>(blockIdx.x);
    const int64_t block_off = scanned ? static_cast<int64_t>(a.counts[b]) : own_block_offset(a, b, red);
    const int64_t base = static_cast<int64_t>(b) * kSurfBlock;
    uint32_t bits = lane_flags(a, base);
    const int c = __popc(bits);
    int64_t pos = block_off + (block_inclusive_scan(c, wave_tot) - c);
    const int64_t v0 = base + 16 * static_cast<int64_t>(threadIdx.x);
    while (bits) {
        const int q = __ffs(bits) - 1;
        bits &= bits - 1;
        if (pos < a.capacity) a.out[pos] = static_cast<int32_t>(v0 + q);
        ++pos;
    }
}

__global__ void zero_count_kernel(int64_t *count)
{
    if (threadIdx.x == 0) *count = 0;
}

}  // namespace

int64_t surface_blocks(int64_t nvox) { return (nvox + kSurfBlock - 1) / kSurfBlock; }

hipError_t launch_surface(const SurfArgs &a, hipStream_t s)
{
    if (a.nvox == 0) {
        hipLaunchKernelGGL(zero_count_kernel, dim3(1), dim3(64), 0, s, a.count);
        return hipGetLastError();
    }
    const bool pieces = a.nx % 4 == 0 && reinterpret_cast<uintptr_t>(a.post) % 16 == 0 &&
                        reinterpret_cast<uintptr_t>(a.smoothed) % 16 == 0 && reinterpret_cast<uintptr_t>(a.occ) % 4 == 0;
    const int64_t nx = a.nx, ny = a.ny, nz = a.nz;
    auto smooth_grid = [&](int span, int rows, int tz) {
        const int64_t tiles = ((nx + span - 1) / span) * ((ny + rows - 1) / rows);
        const int64_t groups = (tiles + 3) / 4 * ((nz + tz - 1) / tz);
        return dim3(static_cast<unsigned>(groups < kSmoothWide ? groups : kSmoothWide),
                    static_cast<unsigned>((groups + kSmoothWide - 1) / kSmoothWide));
    };
    if (pieces && a.nx > 128)
        hipLaunchKernelGGL((smooth4_kernel<64, kPieceY, kPieceZ>), smooth_grid(256, kPieceY, kPieceZ), dim3(256), 0, s, a);
    else if (pieces && a.nx > 64)
        hipLaunchKernelGGL((smooth4_kernel<32, kPieceY, kPieceZ>), smooth_grid(128, 2 * kPieceY, kPieceZ), dim3(256), 0, s, a);
    else if (pieces)
        hipLaunchKernelGGL((smooth4_kernel<16, kPieceY, kPieceZ>), smooth_grid(64, 4 * kPieceY, kPieceZ), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((smooth_kernel<kTileY, kTileZ>), smooth_grid(64, kTileY, kTileZ), dim3(256), 0, s, a);
    const bool words = a.nx % 4 == 0 && reinterpret_cast<uintptr_t>(a.occ) % 4 == 0 &&
                       reinterpret_cast<uintptr_t>(a.flags) % 4 == 0;
    if (words)
        hipLaunchKernelGGL(surface_flag_words_kernel, dim3(static_cast<unsigned>(a.nblocks)), dim3(kSurfBlock / 4), 0, s, a);
    else
        hipLaunchKernelGGL(surface_flag_kernel, dim3(static_cast<unsigned>(a.nblocks)), dim3(256), 0, s, a);
    const int scanned = a.nblocks > kScanMin ? 1 : 0;
    if (scanned) hipLaunchKernelGGL(surface_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, a);
    hipLaunchKernelGGL(surface_write_kernel, dim3(static_cast<unsigned>(a.nblocks)), dim3(256), 0, s, a, scanned);
    return hipGetLastError();
}

}  // namespace psfs
