// One-frame nearest fusion from pixel boxes staged in LDS, shared by the
// single-frame kernels (forward.hip) and the batch (batch.hip).
//
// A workgroup of kSBThreads lanes fuses kSBStack blocks of kSBX x kSBY x kSBZ
// voxels, one upon the other, a lane one column of kSBDepth voxels, kSBChunk of
// them at a time. Per view, the voxel centres of the stack
// project into the hull of its 8 projected corner centres (the depth is affine
// and positive at every corner, so on the stack the projection is continuous
// and maps the box into that hull); the pixel box around the hull, widened by a
// bound on the FP32 rounding of the per-voxel projection, holds every pixel a
// voxel-view of the stack reads. The boxes of as many views as fit the arena are
// copied into LDS at once (direct-to-LDS loads, pixels outside the image as 0)
// and one barrier waits for the group. Views whose box does not fit the arena,
// or whose corners are not clearly in front of the camera, are gathered
// directly; views whose box misses the image are skipped (every voxel-view of
// them adds 0). Same per-voxel projection arithmetic, pixel rule and view order
// as fuse_column: the posteriors are bit-identical.
//
// The column kernels are bound by the L1's accesses (one per 4 lanes and 64-byte
// chunk, 0.63 per voxel-view: 200 us at 256^3 x 12 views of 1280x720, where a
// variant without its gathers takes 93); here the L1 serves 16-byte pieces and
// the scattered reads go to LDS, and what bounds it is the arithmetic and the
// waits of each group. Two blocks share a workgroup's boxes and row sums: one
// block 140 us, two 120, three 121 and four 127. Chunks of 4 voxels whose Z is made
// anew keep the registers (79) and the arena (26 KB) small enough for six
// workgroups per CU, which hide each one's waits: 115 us (16 voxels at once 143).
#pragma once

#include "kernels_common.h"

namespace psfs {
namespace dev {

constexpr int kSBX = 16, kSBY = 16, kSBZ = 8;
constexpr int kSBThreads = 256;
constexpr int kSBStack = 2, kSBDepth = kSBStack * kSBZ;
constexpr int kSBChunk = 4;
static_assert(kSBDepth % kSBChunk == 0, "whole chunks");
constexpr int kSArena = 6400;                       // staged floats per workgroup: 26 KB
static_assert(kSArena % 4 == 0, "whole 16-byte pieces");
static_assert(kSBThreads == kSBX * kSBY, "a lane takes one column of the stack");

struct __align__(16) SBox {
    int x0, y0, w, area;                            // first pixel, row length (pitch) and floats in LDS
    int mode;                                       // kMiss .. kDirect
    int pieces;                                     // staged in 16-byte pieces (else pixel by pixel)
};
// kMiss: misses the image. kInside: staged, every pixel of it in the image.
// kEdge: staged, reaches past the image. kDirect: gathered from the map.
enum { kMiss, kInside, kEdge, kDirect };

// Voxel centre coordinate, as every fusion path computes it.
__device__ __forceinline__ float voxel_centre(float o, float h, int i)
{
    return o + h * (static_cast<float>(i) + 0.5f);
}

// Pixel boxes of every view for the stack with first voxel (i_lo, j_lo, k_lo)
// (phantom voxels past the grid edge included, so that every lane's voxel
// lies in the hull). Lanes 8v .. 8v+7 of the first two waves take the corners
// of view v in FP64 from the FP32 centres the voxel lanes use; lane 8v writes
// boxes[v]. The FP32 evaluation of floor's argument for a voxel (three
// roundings in each of the numerator and the depth, a reciprocal of 1 ulp and
// a product) is within 1.8e-7 (S_u + |u| S_c) / c + 1.8e-7 |u| of the exact
// value, with S the sum of the absolute terms of a row: over the stack S is
// largest and c smallest at a corner. The box is widened by 2^-6 px plus five
// times that bound.
template <class Views>
__device__ __forceinline__ void block_boxes(const Views &views, int n, const GridDesc &a, int i_lo, int j_lo,
                                            int k_lo, SBox *boxes)
{
    const int t = static_cast<int>(threadIdx.x);
    if (t >= 8 * kMaxViews) return;                 // whole waves: the shuffles need every lane
    const int v = (t >> 3) < n ? (t >> 3) : 0;
    const int corner = t & 7;
    const ViewGeom &g = views(v);
    const double X = voxel_centre(a.ox, a.h, i_lo + ((corner & 1) ? kSBX - 1 : 0));
    const double Y = voxel_centre(a.oy, a.h, j_lo + ((corner & 2) ? kSBY - 1 : 0));
    const double Z = voxel_centre(a.oz, a.h, k_lo + ((corner & 4) ? kSBDepth - 1 : 0));
    double row[3], sum[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const double t0 = static_cast<double>(g.P[4 * q]) * X, t1 = static_cast<double>(g.P[4 * q + 1]) * Y;
        const double t2 = static_cast<double>(g.P[4 * q + 2]) * Z, t3 = static_cast<double>(g.P[4 * q + 3]);
        row[q] = (t0 + t1) + (t2 + t3);
        sum[q] = (fabs(t0) + fabs(t1)) + (fabs(t2) + fabs(t3));
    }
    const double c = row[2];
    // NaN fails every comparison below; the 2^20 limits keep the conversions exact
    bool ok = c > 1e-4 * sum[2] && sum[2] < 1e30;
    const double u = ok ? row[0] / c : 0.0, w = ok ? row[1] / c : 0.0;
    ok = ok && fabs(u) < 1048576.0 && fabs(w) < 1048576.0;
    double umin = u, umax = u, wmin = w, wmax = w, cmin = ok ? c : -1.0;
    double su = sum[0], sw = sum[1], sc = sum[2], au = fabs(u), aw = fabs(w);
#pragma unroll
    for (int m = 1; m <= 4; m <<= 1) {
        umin = fmin(umin, __shfl_xor(umin, m, 64));
        umax = fmax(umax, __shfl_xor(umax, m, 64));
        wmin = fmin(wmin, __shfl_xor(wmin, m, 64));
        wmax = fmax(wmax, __shfl_xor(wmax, m, 64));
        cmin = fmin(cmin, __shfl_xor(cmin, m, 64));
        su = fmax(su, __shfl_xor(su, m, 64));
        sw = fmax(sw, __shfl_xor(sw, m, 64));
        sc = fmax(sc, __shfl_xor(sc, m, 64));
        au = fmax(au, __shfl_xor(au, m, 64));
        aw = fmax(aw, __shfl_xor(aw, m, 64));
    }
    if ((t >> 3) >= n || corner != 0) return;
    SBox b{0, 0, 0, 0, kDirect, 0};
    if (cmin > 0.0) {
        const double mu = 0.015625 + 9e-7 * ((su + au * sc) / cmin + au);
        const double mw = 0.015625 + 9e-7 * ((sw + aw * sc) / cmin + aw);
        if (mu < 0.25 && mw < 0.25) {
            const int x0 = static_cast<int>(floor(umin - mu)), x1 = static_cast<int>(floor(umax + mu));
            const int y0 = static_cast<int>(floor(wmin - mw)), y1 = static_cast<int>(floor(wmax + mw));
            // pieces of four pixels from a multiple of 4 on: each lies in the image
            // or outside it when the rows are whole pieces or the box ends before
            // the row's last piece
            const bool pieces = (g.W & 3) == 0 || x1 + 3 < g.W;
            const int xa = pieces ? x0 & ~3 : x0;
            const int bw = pieces ? (x1 - xa + 4) & ~3 : x1 - xa + 1, bh = y1 - y0 + 1;
            const bool inside = x0 >= 0 && y0 >= 0 && x1 < g.W && y1 < g.H;
            // a kEdge entry is computed from y w + x in FP32, exact below 2^24: rows past
            // 56000 of a box 300 pixels wide are not
            const float rows = static_cast<float>(max(-y0, y1) + 1), cols = static_cast<float>(max(-xa, x1));
            const bool exact = inside || fmaf(rows, static_cast<float>(bw), cols) < 16777216.0f;
            if (x1 < 0 || x0 >= g.W || y1 < 0 || y0 >= g.H)
                b.mode = kMiss;
            else if (exact && bw <= kSArena && bh <= kSArena && bw * bh <= kSArena)
                b = SBox{xa, y0, bw, bw * bh, inside ? kInside : kEdge, pieces};
        }
    }
    boxes[v] = b;
}

__device__ __forceinline__ SBox read_sbox(const SBox *boxes, int v)
{
    SBox b;
    b.x0 = __builtin_amdgcn_readfirstlane(boxes[v].x0);
    b.y0 = __builtin_amdgcn_readfirstlane(boxes[v].y0);
    b.w = __builtin_amdgcn_readfirstlane(boxes[v].w);
    b.area = __builtin_amdgcn_readfirstlane(boxes[v].area);
    b.mode = __builtin_amdgcn_readfirstlane(boxes[v].mode);
    b.pieces = __builtin_amdgcn_readfirstlane(boxes[v].pieces);
    return b;
}

// Starts copying a view's box into LDS: direct-to-LDS loads of 16-byte pieces
// (addresses of whole pixels, 4-byte aligned) or of single pixels; one wave
// instruction per 64 consecutive ones. A piece or pixel outside the image gets
// an offset past the end of the map, which loads 0. (Pixel by pixel, the address
// arithmetic made the fusion of single blocks at 256^3 x 12 views 196 us, in pieces 141 us.)
__device__ __forceinline__ void stage_sbox(const ViewGeom &g, const float *lmap, const SBox &b, float *lds)
{
    const int wave = static_cast<int>(threadIdx.x >> 6), lane = static_cast<int>(threadIdx.x & 63);
    const uint32_t W = static_cast<uint32_t>(g.W), H = static_cast<uint32_t>(g.H);
    const __amdgpu_buffer_rsrc_t rs = map_rsrc(lmap + g.map_off, W * H * 4u);
    const bool pieces = b.pieces != 0;
    const int row = pieces ? b.w >> 2 : b.w, count = pieces ? b.area >> 2 : b.area;
    const float inv = 1.0f / static_cast<float>(row);
    for (int q = wave; q * 64 < count; q += kSBThreads / 64) {
        const int e = q * 64 + lane;
        if (e < count) {
            // (e + 1/2) / row is at least 1/(2 row) from an integer and e < 2^22: exact row
            const int r = static_cast<int>((static_cast<float>(e) + 0.5f) * inv);
            const int c = e - r * row;
            const uint32_t x = static_cast<uint32_t>(b.x0 + (pieces ? 4 * c : c)), y = static_cast<uint32_t>(b.y0 + r);
            const uint32_t o = (x < W && y < H) ? (__umul24(y, W) + x) * 4u : 0xFFFFFFFFu;
            if (pieces)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(lds + q * 256), 16, o, 0, 0, 0);
            else
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(lds + q * 64), 4, o, 0, 0, 0);
        }
    }
}

template <class Views>
__device__ __forceinline__ void fuse_block(const Views &views, int n, const float *lmap, const GridDesc &a,
                                           uint32_t bi, uint32_t bj, uint32_t bk, float L0, float tau, float *post,
                                           uint8_t *occ, float *arena, SBox *boxes)
{
    const int t = static_cast<int>(threadIdx.x);
    const int i_lo = static_cast<int>(bi) * kSBX, j_lo = static_cast<int>(bj) * kSBY, k0 = static_cast<int>(bk) * kSBDepth;
    const int i = i_lo + t % kSBX, j = j_lo + t / kSBX;
    block_boxes(views, n, a, i_lo, j_lo, k0, boxes);
    const float X = voxel_centre(a.ox, a.h, i), Y = voxel_centre(a.oy, a.h, j);
    float L[kSBDepth];
#pragma unroll
    for (int kk = 0; kk < kSBDepth; ++kk) L[kk] = L0;
    __syncthreads();                                // boxes visible

    // The views are taken in groups whose boxes fit the arena together: their
    // boxes are staged at once (each wave derives the same offsets) and one
    // barrier waits for them. A kDirect view takes no room.
    for (int v0 = 0; v0 < n;) {
        int v1 = v0, off = 0;
        for (; v1 < n; ++v1) {
            const SBox b = read_sbox(boxes, v1);
            if (b.mode != kInside && b.mode != kEdge) continue;
            if (off + b.area > kSArena) break;
            stage_sbox(views(v1), lmap, b, arena + off);
            off += (b.area + 3) & ~3;               // 16-byte pieces start aligned
        }
        __syncthreads();                            // every wave's loads have landed
        off = 0;
        for (int v = v0; v < v1; ++v) {
            const SBox b = read_sbox(boxes, v);
            if (b.mode == kMiss) continue;
            const ViewGeom &g = views(v);
            const float ax = fmaf(g.P[0], X, fmaf(g.P[1], Y, g.P[3]));
            const float bx = fmaf(g.P[4], X, fmaf(g.P[5], Y, g.P[7]));
            const float cx = fmaf(g.P[8], X, fmaf(g.P[9], Y, g.P[11]));
            const __amdgpu_buffer_rsrc_t rs = map_rsrc(lmap + g.map_off, static_cast<uint32_t>(g.W) * static_cast<uint32_t>(g.H) * 4u);
            const float wf = static_cast<float>(b.w);
            const float od = static_cast<float>(b.y0) * wf + static_cast<float>(b.x0);
            const float emax = static_cast<float>(b.area - 1);
            const int base = off - (b.y0 * b.w + b.x0);
#pragma unroll
            for (int h = 0; h < kSBDepth; h += kSBChunk) {
                float Z[kSBChunk], val[kSBChunk];
#pragma unroll
                for (int kk = 0; kk < kSBChunk; ++kk) Z[kk] = voxel_centre(a.oz, a.h, k0 + h + kk);
                if (b.mode == kDirect) {
                    uint32_t o[kSBChunk];
                    nearest_offsets<kSBChunk, 4>(g, ax, bx, cx, Z, false, o);
#pragma unroll
                    for (int kk = 0; kk < kSBChunk; ++kk) val[kk] = map_load(rs, o[kk]);
                } else {
                    int e[kSBChunk];
                    if (b.mode == kInside) {
                        // box entry (y - y0) w + (x - x0), x and y in the image:
                        // truncation is the floor (a read past the LDS gives 0)
#pragma unroll
                        for (int kk = 0; kk < kSBChunk; ++kk) {
                            const float r = __builtin_amdgcn_rcpf(fmaf(g.P[10], Z[kk], cx));
                            const uint32_t x = static_cast<uint32_t>(fmaf(g.P[2], Z[kk], ax) * r);
                            const uint32_t y = static_cast<uint32_t>(fmaf(g.P[6], Z[kk], bx) * r);
                            e[kk] = static_cast<int>(__umul24(y, static_cast<uint32_t>(b.w)) + x) + base;
                        }
                    } else {
                        // exact in FP32 (integers below 2^24, block_boxes); the clamp keeps a read in the box
#pragma unroll
                        for (int kk = 0; kk < kSBChunk; ++kk) {
                            const float r = __builtin_amdgcn_rcpf(fmaf(g.P[10], Z[kk], cx));
                            const float x = floorf(fmaf(g.P[2], Z[kk], ax) * r);
                            const float y = floorf(fmaf(g.P[6], Z[kk], bx) * r);
                            e[kk] = off + static_cast<int>(__builtin_amdgcn_fmed3f(fmaf(y, wf, x - od), 0.0f, emax));
                        }
                    }
#pragma unroll
                    for (int kk = 0; kk < kSBChunk; ++kk) val[kk] = arena[e[kk]];
                }
#pragma unroll
                for (int kk = 0; kk < kSBChunk; ++kk) L[h + kk] += val[kk];
            }
            if (b.mode != kDirect) off += (b.area + 3) & ~3;
        }
        v0 = v1;
        if (v0 < n) __syncthreads();                // the group's reads are done
    }
    if (i >= a.nx || j >= a.ny) return;
    const int64_t plane = static_cast<int64_t>(a.nx) * a.ny;
    int64_t idx = (static_cast<int64_t>(k0) * a.ny + j) * a.nx + i;
#pragma unroll
    for (int kk = 0; kk < kSBDepth; ++kk, idx += plane) {
        if (k0 + kk < a.nz) {
            const float p = sigmoid_fast(L[kk]);
            post[idx] = p;
            if (occ) occ[idx] = p > tau ? 1 : 0;
        }
    }
}

template <class T>
__host__ __device__ int64_t block_count(const T &a)
{
    return static_cast<int64_t>((a.nx + kSBX - 1) / kSBX) * ((a.ny + kSBY - 1) / kSBY) * ((a.nz + kSBDepth - 1) / kSBDepth);
}

}  // namespace dev
}  // namespace psfs
