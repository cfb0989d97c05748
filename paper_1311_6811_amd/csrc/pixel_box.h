// Bilinear sampling of voxel blocks from pixel boxes staged in LDS, shared by
// the bilinear reconstruction (forward.hip) and the differentiable pass
// (diff.hip). The argument structs (BilinearArgs, DiffArgs) name their views,
// FP64 camera matrices Pd, maps and grid alike.
#pragma once

#include "kernels_common.h"

namespace psfs {
namespace dev {

constexpr int kBoxThreads = 256;        // lanes of a workgroup that works from pixel boxes

// Projection rows of view v at an FP64 voxel column (X, Y), from the camera
// matrix widened on the host (kernel arguments: scalar operands of the FMAs).
template <class Args>
__device__ __forceinline__ Proj64 proj64_view(const Args &a, int v, double X, double Y)
{
    const double *P = a.Pd[v];
    Proj64 p;
    p.ax = fma(P[0], X, fma(P[1], Y, P[3]));
    p.bx = fma(P[4], X, fma(P[5], Y, P[7]));
    p.cx = fma(P[8], X, fma(P[9], Y, P[11]));
    p.pz0 = P[2];
    p.pz1 = P[6];
    p.pz2 = P[10];
    return p;
}

// Pixel box [x0, x0+w) x [y0, y0+h) holding both bilinear taps in x and y of
// every voxel centre of the workgroup's voxel box, for every view: the
// projection maps the box into the hull of its 8 projected corners (all in
// front of the camera), widened by 1e-6 px for the lanes' own FP64 rounding.
// Lanes 8v..8v+7 project the corners of view v; the box is stored in LDS.
// ok = 0 when a corner is not in front or the box exceeds `cap` floats; kMissed when
// no pixel of it lies in the image, so that every sample is 0.
struct PixBox {
    int x0, y0, w, h, ok;
    int pieces;                         // staged in 16-byte pieces (else pixel by pixel)
};
constexpr int kMissed = 2;

// Floats that a staged box takes: the next one starts at a whole piece.
__device__ __forceinline__ int box_floats(const PixBox &b) { return (b.w * b.h + 3) & ~3; }

// First voxel (bi, bj, kb) of an EX x EY x EZ block. pieces: boxes are widened to
// pieces of four pixels from a multiple of 4 on where each piece then lies in the
// image or outside it (the rows are whole pieces, or the box ends before the
// row's last one) and the box still fits. sampling: boxes that miss the image are
// marked, for passes that only add the samples.
template <int EX, int EY, int EZ, class Args>
__device__ __forceinline__ void compute_boxes(const Args &a, int bi, int bj, int kb, int cap, bool pieces, bool sampling,
                                              PixBox *boxes)
{
    for (int t0 = 0; t0 < 8 * a.n; t0 += kBoxThreads) {
        const int t = t0 + static_cast<int>(threadIdx.x);
        const int v = t < 8 * a.n ? t >> 3 : 0;
        const int corner = t & 7;
        const double X = centre64(a.ox, a.h, corner & 1 ? bi + EX - 1 : bi);
        const double Y = centre64(a.oy, a.h, corner & 2 ? bj + EY - 1 : bj);
        const double Z = centre64(a.oz, a.h, corner & 4 ? kb + EZ - 1 : kb);
        const Proj64 p = proj64_view(a, v, X, Y);
        const double c = fma(p.pz2, Z, p.cx);
        double ok = c > 0.0 ? 1.0 : 0.0;
        const double u = fma(p.pz0, Z, p.ax) / c, w = fma(p.pz1, Z, p.bx) / c;
        double umin = u, umax = u, wmin = w, wmax = w;
#pragma unroll
        for (int m = 1; m <= 4; m <<= 1) {
            umin = fmin(umin, __shfl_xor(umin, m, 64));
            umax = fmax(umax, __shfl_xor(umax, m, 64));
            wmin = fmin(wmin, __shfl_xor(wmin, m, 64));
            wmax = fmax(wmax, __shfl_xor(wmax, m, 64));
            ok = fmin(ok, __shfl_xor(ok, m, 64));
        }
        if (t < 8 * a.n && corner == 0) {
            PixBox b{0, 0, 0, 0, 0, 0};
            // NaN or huge coordinates fail these range tests
            if (ok > 0.5 && umin > -1e6 && umax < 1e6 && wmin > -1e6 && wmax < 1e6) {
                b.x0 = static_cast<int>(floor(umin - 1e-6));
                b.y0 = static_cast<int>(floor(wmin - 1e-6));
                b.w = static_cast<int>(floor(umax + 1e-6)) + 2 - b.x0;
                b.h = static_cast<int>(floor(wmax + 1e-6)) + 2 - b.y0;
                // sides are checked before the product so it cannot overflow
                b.ok = (b.w > 0 && b.h > 0 && b.w <= cap && b.h <= cap && b.w * b.h <= cap) ? 1 : 0;
                const int x1 = b.x0 + b.w - 1, xa = b.x0 & ~3, wa = (x1 - xa + 4) & ~3, W = a.view[v].W;
                if (pieces && b.ok && ((W & 3) == 0 || x1 + 3 < W) && wa <= cap && wa * b.h <= cap) {
                    b.x0 = xa;
                    b.w = wa;
                    b.pieces = 1;
                }
                if (sampling && (x1 < 0 || b.x0 >= W || b.y0 + b.h <= 0 || b.y0 >= a.view[v].H)) b.ok = kMissed;
            }
            boxes[v] = b;
        }
    }
}

__device__ __forceinline__ PixBox read_box(const PixBox *boxes, int v)
{
    PixBox b;
    b.x0 = __builtin_amdgcn_readfirstlane(boxes[v].x0);
    b.y0 = __builtin_amdgcn_readfirstlane(boxes[v].y0);
    b.w = __builtin_amdgcn_readfirstlane(boxes[v].w);
    b.h = __builtin_amdgcn_readfirstlane(boxes[v].h);
    b.ok = __builtin_amdgcn_readfirstlane(boxes[v].ok);
    b.pieces = __builtin_amdgcn_readfirstlane(boxes[v].pieces);
    return b;
}

// Element e of a box, row-major: r = e / w without an integer division
// ((e + 1/2) / w is at least 1/(2w) away from an integer for e < 2^22).
__device__ __forceinline__ void box_rc(int e, int w, float inv_w, int &r, int &c)
{
    r = static_cast<int>((static_cast<float>(e) + 0.5f) * inv_w);
    c = e - r * w;
}

// Starts copying a view's map over the box into LDS (direct-to-LDS loads of
// 16-byte pieces or of single pixels, one wave instruction per 64 consecutive
// ones); a pixel outside the image gets an offset past the end of the map, which
// loads 0. The values are there after the workgroup's next barrier. (Pixel by pixel
// against in pieces: bilinear fusion 128^3 x 8 views of 640x480 33.9 / 30.3 us, 160^3 x 8
// of 1280x720 65 / 51, 224^3 x 12 182 / 158; differentiable forward 58 / 54, 121 / 106,
// 271 / 248.)
__device__ __forceinline__ void stage_box_async(float *lds, const PixBox &b, const float *map, int W, int H)
{
    const bool pieces = b.pieces != 0;
    const int row = pieces ? b.w >> 2 : b.w, count = row * b.h;
    const float inv_w = 1.0f / static_cast<float>(row);
    const __amdgpu_buffer_rsrc_t rs = map_rsrc(map, static_cast<uint32_t>(W) * static_cast<uint32_t>(H) * 4u);
    const int wave = static_cast<int>(threadIdx.x >> 6), lane = static_cast<int>(threadIdx.x & 63);
    for (int q = wave; q * 64 < count; q += kBoxThreads / 64) {
        const int e = q * 64 + lane;
        if (e < count) {
            int r, c;
            box_rc(e, row, inv_w, r, c);
            const uint32_t x = static_cast<uint32_t>(b.x0 + (pieces ? 4 * c : c)), y = static_cast<uint32_t>(b.y0 + r);
            const bool in = x < static_cast<uint32_t>(W) && y < static_cast<uint32_t>(H);
            const uint32_t o = in ? (__umul24(y, static_cast<uint32_t>(W)) + x) * 4u : 0xFFFFFFFFu;
            if (pieces)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(lds + q * 256),
                                                         16, o, 0, 0, 0);
            else
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(lds + q * 64), 4,
                                                         o, 0, 0, 0);
        }
    }
}

// The views of [v_lo, v_hi) whose box has the given `ok`, as bits.
__device__ __forceinline__ uint32_t views_with(const PixBox *boxes, int v_lo, int v_hi, int ok)
{
    static_assert(kMaxViews <= 32, "a bit per view");
    const int v = v_lo + static_cast<int>(threadIdx.x & 63);
    return static_cast<uint32_t>(__ballot(v < v_hi && boxes[v < v_hi ? v : v_lo].ok == ok)) << v_lo;
}

// Bits [v0, v1).
__device__ __forceinline__ uint32_t view_range(int v0, int v1)
{
    return static_cast<uint32_t>((uint64_t(1) << v1) - (uint64_t(1) << v0));
}

// Starts staging the boxes of the views `boxed` from v0 on that fit the CAP floats
// of `arena` together, one after another; returns the first view that is left for
// the next group (v_hi when there is none).
template <int CAP, class Args>
__device__ __forceinline__ int stage_group(const Args &a, int v0, int v_hi, uint32_t boxed, const PixBox *boxes, float *arena)
{
    int off = 0;
    for (uint32_t m = boxed & view_range(v0, v_hi); m; m &= m - 1) {
        const int v = __builtin_ctz(m);
        const PixBox box = read_box(boxes, v);
        if (off + box.w * box.h > CAP) return v;
        stage_box_async(arena + off, box, a.lmap + a.view[v].map_off, a.view[v].W, a.view[v].H);
        off += box_floats(box);
    }
    return v_hi;
}

// L[kk] += the bilinear sample of every view, in view order, at the lane's
// KZ voxels (Xd, Yd, slice kb + kk) of the workgroup's 16 x 16 x KZ voxel
// block. The views are taken in groups whose boxes fit the CAP floats of
// `arena` together: their boxes are loaded at once, and one barrier waits for
// the group. A view without a valid box is sampled from its map; one whose box
// misses the image is passed over (staged and sampled as zeros, 200^3 voxels whose
// 8 views mostly look past them took 109 us, column by column 95).
template <Taps T, int KZ, int CAP, class Args>
__device__ __forceinline__ void add_bilinear(const Args &a, double Xd, double Yd, int kb, float *arena,
                                             const PixBox *boxes, float (&L)[KZ])
{
    const uint32_t boxed = views_with(boxes, 0, a.n, 1), sampled = boxed | views_with(boxes, 0, a.n, 0);
    for (int v0 = 0; v0 < a.n;) {
        const int v1 = stage_group<CAP>(a, v0, a.n, boxed, boxes, arena);
        __syncthreads();                    // every wave's loads have landed
        int off = 0;
        for (uint32_t m = sampled & view_range(v0, v1); m; m &= m - 1) {
            const int v = __builtin_ctz(m);
            const ViewGeom &g = a.view[v];
            const Proj64 p = proj64_view(a, v, Xd, Yd);
            if (boxed >> v & 1) {
                const PixBox box = read_box(boxes, v);
                // box element of tap (x0, y0): (y0 - box.y0) w + (x0 - box.x0),
                // exact in FP64 (integers far below 2^53). Every voxel centre
                // of the workgroup is in front of the camera and has both taps
                // in the box (taps outside the image read the 0s the staging
                // wrote there); the clamp only keeps the reads in the box.
                const double wd = static_cast<double>(box.w);
                const double od = static_cast<double>(box.y0) * wd + static_cast<double>(box.x0);
                const int emax = box.w * box.h - box.w - 2;
#pragma unroll
                for (int kk = 0; kk < KZ; ++kk) {
                    const double Zd = centre64(a.oz, a.h, kb + kk);
                    Tap4 t;
                    project64_front<T>(p, Zd, t);
                    const int e = min(max(static_cast<int>(fma(t.y0, wd, t.x0 - od)), 0), emax);
                    const float *s = arena + off + e;
                    const float top = fmaf(t.fx, s[1] - s[0], s[0]);
                    const float bot = fmaf(t.fx, s[box.w + 1] - s[box.w], s[box.w]);
                    L[kk] += fmaf(t.fy, bot - top, top);
                }
                off += box_floats(box);
            } else {
#pragma unroll
                for (int kk = 0; kk < KZ; ++kk) {
                    const double Zd = centre64(a.oz, a.h, kb + kk);
                    Tap4 t;
                    if (!project64<T>(p, Zd, t)) continue;
                    L[kk] += bilinear_sample(a.lmap + g.map_off, g.W, g.H, t.x0, t.y0, t.fx, t.fy);
                }
            }
        }
        v0 = v1;
        if (v0 < a.n) __syncthreads();      // the group's reads are done
    }
}

}  // namespace dev
}  // namespace psfs
