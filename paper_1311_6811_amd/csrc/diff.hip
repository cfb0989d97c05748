// Differentiable variant of the occupancy pass for gfx950.
//
// Forward: every view's log(2*SLM) map (Eq. 1-2) is sampled bilinearly at the
// projected voxel centre and summed into the logit of Eq. 3-9's posterior,
// L = logit(prior) + sum_k l~_k; the loss is the mean binary cross-entropy
// with logits, softplus(L) - y*L, over a box of voxels.
//
// Backward (hand-written adjoint, projections recomputed, not stored):
//   g_v = dLoss/dL_v = grad_loss * (sigmoid(L_v) - y_v) / |region|
//   adjoint map:  Abar_k[tap] += g_v * w_tap         (w = bilinear weights)
//   camera:       dLoss/dP_k = sum_v g_v * (dl~/du du/dP + dl~/dv dv/dP), with
//                 u = a/c, v = b/c, (a,b,c) = P [X;1]:
//                 du/dP_row0 = X~/c, dv/dP_row1 = X~/c, d(u,v)/dP_row2 = -(u,v) X~/c
//   pixel chain:  dlog(2*SLM)/dd = -sigmoid(d) with d = log N - log u, and
//                 dd/dmu_c = (I_c - mu_c)/v_c,
//                 dd/dv_c = (I_c - mu_c)^2/(2 v_c^2) - 1/(2 v_c).
// Reductions of the loss and of the camera gradients run in a fixed order
// (per lane, a fixed wavefront butterfly, waves in order, workgroups in order
// in FP64). The adjoint maps are accumulated in fixed point: every term
// g_v * w satisfies |g_v * w| <= G = |grad_loss| / |region|, so it is rounded
// to a multiple of 2^-E with 2^E * G <= 2^19; a workgroup's terms for one
// pixel (at most 2048) then fit in int32 in LDS (integer LDS atomics, much
// faster than FP32 ones on this GPU) and the global sums fit in int64 (at most
// 2^31 terms). Integer sums do not depend on order, so all outputs are
// reproducible bit for bit; the rounding error per term is <= 2^-20 G.
#include <algorithm>

#include "pixel_box.h"

namespace psfs {
namespace {

using namespace dev;

constexpr int kBlock = kBoxThreads;
constexpr int kWaves = kBlock / 64;
constexpr int kBoxCap = 4096;           // floats of one view's pixel box staged in LDS (backward)
constexpr int kBwdBlocks = 1024;        // workgroups of the backward (four per CU): smaller grids split their views
constexpr int kFwdArena = 7500;         // floats of the forward's staged boxes
constexpr int kStageIters = kBoxCap / kBlock;

struct Coords {
    int i, j, kb;                       // lane column, first slice of the workgroup
    int bi, bj;                         // first column of the workgroup
};

__device__ __forceinline__ bool in_region(const DiffArgs &a, int i, int j, int k)
{
    return i >= a.sub[0] && i < a.sub[1] && j >= a.sub[2] && j < a.sub[3] && k >= a.sub[4] && k < a.sub[5];
}

__device__ __forceinline__ float softplusf(float x)
{
    return fmaxf(x, 0.0f) + log1pf(expf(-fabsf(x)));
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}

// Exponent E of the adjoint fixed point (see the file comment); 0 when G is
// 0 or not finite (every term is then 0 or the input invalid).
// Two's-complement int32 as the uint64 addend of a signed int64 sum.
__device__ __forceinline__ unsigned long long widen(int q)
{
    return static_cast<unsigned long long>(static_cast<long long>(q));
}

__device__ __forceinline__ int adjoint_exponent(float grad_loss, float inv_count)
{
    const float G = fabsf(grad_loss) * inv_count;
    if (!(G > 0.0f) || !isfinite(G)) return 0;
    int e;
    frexpf(G, &e);                      // G < 2^e
    return 19 - e;
}

// Workgroup of either pass = 16 x 16 voxel columns x kFZ slices, a lane one
// column and its kFZ voxels. Its views' pixel boxes hold ~0.7 pixels per
// voxel at 128^3 x 8 views of 640x480 (~0.9 for 8 x 8 x 16 or 8 x 8 x 32
// blocks), and the per-view work (box, barriers, projection rows) is shared
// by 2048 voxels. The forward's waves are 16 x 4 columns (lane t: column
// (t % 16, t / 16)); the backward's are 8 x 8 columns (wave w, lane l: column
// (8 (w & 1) + l % 8, 8 (w >> 1) + l / 8)), so that fewer of its lanes lie on
// one viewing ray of a ring camera, where they would add into the same
// pixels of the adjoint box (same-address LDS atomics).
constexpr int kFX = 16, kFY = 16, kFZ = 8;

template <bool SQUARE_WAVES>
__device__ __forceinline__ Coords block_coords(int nx, int ny, int nz)
{
    const int ntx = (nx + kFX - 1) / kFX, nty = (ny + kFY - 1) / kFY;
    const int64_t ntile = static_cast<int64_t>(ntx) * nty;
    const int64_t nb = ntile * ((nz + kFZ - 1) / kFZ);
    const int64_t b = xcd_remap(blockIdx.x, nb);
    const int64_t zc = b / ntile;
    const int t = static_cast<int>(b - zc * ntile);
    const int tyi = t / ntx, txi = t - tyi * ntx;
    const int w = static_cast<int>(threadIdx.x >> 6), l = static_cast<int>(threadIdx.x & 63);
    Coords c;
    c.bi = txi * kFX;
    c.bj = tyi * kFY;
    if (SQUARE_WAVES) {
        c.i = c.bi + 8 * (w & 1) + (l & 7);
        c.j = c.bj + 8 * (w >> 1) + (l >> 3);
    } else {
        c.i = c.bi + static_cast<int>(threadIdx.x % kFX);
        c.j = c.bj + static_cast<int>(threadIdx.x / kFX);
    }
    c.kb = static_cast<int>(zc) * kFZ;
    return c;
}

// Copies a view's map over the box into LDS; pixels outside the image read as
// 0. All loads of a lane are issued before its LDS stores. NP passes of the
// workgroup cover boxes of up to NP * kBlock pixels.
template <int NP>
__device__ __forceinline__ void stage_box_n(float *lds, const PixBox &b, const float *map, int W, int H)
{
    const int area = b.w * b.h;
    const float inv_w = 1.0f / static_cast<float>(b.w);
    float vals[NP];
#pragma unroll
    for (int t = 0; t < NP; ++t) {
        const int e = static_cast<int>(threadIdx.x) + t * kBlock;
        vals[t] = 0.0f;
        if (e < area) {
            int r, c;
            box_rc(e, b.w, inv_w, r, c);
            const int x = b.x0 + c, y = b.y0 + r;
            if (x >= 0 && x < W && y >= 0 && y < H) vals[t] = map[static_cast<int64_t>(y) * W + x];
        }
    }
#pragma unroll
    for (int t = 0; t < NP; ++t) {
        const int e = static_cast<int>(threadIdx.x) + t * kBlock;
        if (e < area) lds[e] = vals[t];
    }
}

// stage_box_n with as few passes as the (workgroup-uniform) box needs: most
// boxes of the 8x8-column workgroups hold under 1024 pixels.
__device__ __forceinline__ void stage_box(float *lds, const PixBox &b, const float *map, int W, int H)
{
    const int area = b.w * b.h;
    if (area <= 4 * kBlock)
        stage_box_n<4>(lds, b, map, W, H);
    else if (area <= 8 * kBlock)
        stage_box_n<8>(lds, b, map, W, H);
    else
        stage_box_n<kStageIters>(lds, b, map, W, H);
}

__global__ __launch_bounds__(kBlock) void diff_fwd_kernel(DiffArgs a)
{
    __shared__ __align__(16) float arena[kFwdArena];
    __shared__ PixBox boxes[kMaxViews];
    const Coords q = block_coords<false>(a.nx, a.ny, a.nz);
    compute_boxes<kFX, kFY, kFZ>(a, q.bi, q.bj, q.kb, kFwdArena, true, true, boxes);
    const double Xd = centre64(a.ox, a.h, q.i), Yd = centre64(a.oy, a.h, q.j);
    float L[kFZ];
#pragma unroll
    for (int kk = 0; kk < kFZ; ++kk) L[kk] = a.L0;
    __syncthreads();
    add_bilinear<Taps::kDifferentiable, kFZ, kFwdArena>(a, Xd, Yd, q.kb, arena, boxes, L);

    double part = 0.0;
    if (q.i < a.nx && q.j < a.ny) {
#pragma unroll
        for (int kk = 0; kk < kFZ; ++kk) {
            const int k = q.kb + kk;
            if (k >= a.nz) continue;
            const int64_t idx = (static_cast<int64_t>(k) * a.ny + q.j) * a.nx + q.i;
            a.logits[idx] = L[kk];
            if (in_region(a, q.i, q.j, k)) {
                const float y = static_cast<float>(a.labels[idx]);
                part += static_cast<double>(softplusf(L[kk]) - y * L[kk]);
            }
        }
    }
    part = wave_sum(part);
    __shared__ double wsum[kWaves];
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < kWaves; ++w) s += wsum[w];
        a.loss_part[blockIdx.x] = s;
    }
}

// loss = inv_count * sum of the workgroup partials, in a fixed order: thread
// t adds partials t + 256 q (eight loads in flight at a time), then the
// wave butterfly of wave_sum, then the four waves in order.
__global__ __launch_bounds__(256) void loss_finalize_kernel(const double *part, int64_t nparts, float inv_count, float *loss)
{
    __shared__ double wsum[4];
    double s = 0.0;
    for (int64_t b0 = 0; b0 < nparts; b0 += 8 * 256) {
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t b = b0 + threadIdx.x + 256 * q;
            v[q] = b < nparts ? part[b] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) s += v[q];
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) *loss = static_cast<float>(((wsum[0] + wsum[1]) + (wsum[2] + wsum[3])) * static_cast<double>(inv_count));
}

__global__ __launch_bounds__(256) void zero_kernel(float *p, int64_t n4)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n4; i += stride)
        reinterpret_cast<f32x4 *>(p)[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
}

// A lane's sums over its voxels of one view: g_r and g_r Z for the rows r of P.
struct CamSums {
    float su = 0.0f, suz = 0.0f, sv = 0.0f, svz = 0.0f, sc = 0.0f, scz = 0.0f;
};

// Fixed-point terms of one voxel's four taps.
struct TapTerms {
    int q00, q10, q01, q11;
};

__device__ __forceinline__ TapTerms tap_terms(float gk, float fx, float fy, float qscale)
{
    return TapTerms{static_cast<int>(rintf(gk * (1.0f - fx) * (1.0f - fy) * qscale)),
                    static_cast<int>(rintf(gk * fx * (1.0f - fy) * qscale)),
                    static_cast<int>(rintf(gk * (1.0f - fx) * fy * qscale)), static_cast<int>(rintf(gk * fx * fy * qscale))};
}

__device__ __forceinline__ void add_camera_terms(CamSums &s, float gk, const Tap4 &t, float Z, float l00, float l10,
                                                 float l01, float l11)
{
    const float dldu = (1.0f - t.fy) * (l10 - l00) + t.fy * (l11 - l01);
    const float dldv = (1.0f - t.fx) * (l01 - l00) + t.fx * (l11 - l10);
    const float gu = gk * dldu * t.rc, gw = gk * dldv * t.rc;
    const float gc = -(gu * t.u + gw * t.v);
    s.su += gu; s.suz = fmaf(gu, Z, s.suz);
    s.sv += gw; s.svz = fmaf(gw, Z, s.svz);
    s.sc += gc; s.scz = fmaf(gc, Z, s.scz);
}

// Whether a voxel's adjoint terms can round to anything but 0 (NaN: yes):
// every tap weight is at most 1 and rintf(0.5) is 0.
__device__ __forceinline__ bool scatters(float gk, float qscale) { return !(fabsf(gk) * qscale <= 0.5f); }

// The lane's voxels of one view, from the view's box staged
// at `map_box`; with SCATTER their adjoint terms go to `adj_box`. As in the
// forward kernel there are no per-voxel depth or range tests: a voxel whose
// taps all fall outside the image reads four 0s, adds 0 to the camera sums and
// scatters only into box pixels outside the image, which the flush skips: the
// same as skipping it.
template <bool SCATTER>
__device__ __forceinline__ void box_voxels(const DiffArgs &a, const Proj64 &p, const PixBox &box, const float *map_box,
                                           int *adj_box, int kb, const float (&gv)[kFZ], float qscale,
                                           CamSums &s)
{
    const double wd = static_cast<double>(box.w);
    const double od = static_cast<double>(box.y0) * wd + static_cast<double>(box.x0);
    const int emax = box.w * box.h - box.w - 2;
#pragma unroll
    for (int kk = 0; kk < kFZ; ++kk) {
        if (gv[kk] == 0.0f) continue;
        const double Zd = centre64(a.oz, a.h, kb + kk);
        Tap4 t;
        project64_front<Taps::kDifferentiable>(p, Zd, t);
        const int e = min(max(static_cast<int>(fma(t.y0, wd, t.x0 - od)), 0), emax);
        const float l00 = map_box[e], l10 = map_box[e + 1], l01 = map_box[e + box.w], l11 = map_box[e + box.w + 1];
        if (SCATTER) {
            const TapTerms q = tap_terms(gv[kk], t.fx, t.fy, qscale);
            atomicAdd(&adj_box[e], q.q00);
            atomicAdd(&adj_box[e + 1], q.q10);
            atomicAdd(&adj_box[e + box.w], q.q01);
            atomicAdd(&adj_box[e + box.w + 1], q.q11);
        }
        add_camera_terms(s, gv[kk], t, static_cast<float>(Zd), l00, l10, l01, l11);
    }
}

// The lane's voxels of a view without a box: taps from the map, adjoint terms
// into the global sums.
__device__ __forceinline__ void map_voxels(const DiffArgs &a, const ViewGeom &g, const Proj64 &p, int kb,
                                           const float (&gv)[kFZ], float qscale, CamSums &s)
{
    const float *map = a.lmap + g.map_off;
    unsigned long long *adj = reinterpret_cast<unsigned long long *>(a.adj) + g.map_off;
#pragma unroll
    for (int kk = 0; kk < kFZ; ++kk) {
        if (gv[kk] == 0.0f) continue;
        const double Zd = centre64(a.oz, a.h, kb + kk);
        Tap4 t;
        if (!project64<Taps::kDifferentiable>(p, Zd, t)) continue;
        if (!(t.x0 >= -1.0 && t.x0 < g.W && t.y0 >= -1.0 && t.y0 < g.H)) continue;
        const int ix = static_cast<int>(t.x0), iy = static_cast<int>(t.y0);
        const bool xin0 = ix >= 0, xin1 = ix + 1 < g.W, yin0 = iy >= 0, yin1 = iy + 1 < g.H;
        const int64_t base = static_cast<int64_t>(iy) * g.W + ix;
        const float l00 = xin0 && yin0 ? map[base] : 0.0f, l10 = xin1 && yin0 ? map[base + 1] : 0.0f;
        const float l01 = xin0 && yin1 ? map[base + g.W] : 0.0f, l11 = xin1 && yin1 ? map[base + g.W + 1] : 0.0f;
        if (scatters(gv[kk], qscale)) {
            const TapTerms q = tap_terms(gv[kk], t.fx, t.fy, qscale);
            if (xin0 && yin0) atomicAdd(adj + base, widen(q.q00));
            if (xin1 && yin0) atomicAdd(adj + base + 1, widen(q.q10));
            if (xin0 && yin1) atomicAdd(adj + base + g.W, widen(q.q01));
            if (xin1 && yin1) atomicAdd(adj + base + g.W + 1, widen(q.q11));
        }
        add_camera_terms(s, gv[kk], t, static_cast<float>(Zd), l00, l10, l01, l11);
    }
}

// dLoss/dP row r of one view = sum over the lanes' voxels of g_r (X, Y, Z, 1):
// the wave's sums of the 12 entries through its 768 floats of LDS, in a fixed
// order: lane 4e + m adds lanes 16m .. 16m+15 of entry e, then a quad
// butterfly; lane 4e writes out[e].
__device__ __forceinline__ void wave_camera_sums(const CamSums &s, float X, float Y, float *red, float *out)
{
    const int lane = static_cast<int>(threadIdx.x & 63);
    const float vals[12] = {X * s.su, Y * s.su, s.suz, s.su, X * s.sv, Y * s.sv, s.svz, s.sv, X * s.sc, Y * s.sc, s.scz, s.sc};
#pragma unroll
    for (int e = 0; e < 12; ++e) red[e * 64 + lane] = vals[e];
    wave_lds_sync();
    float t = 0.0f;
    if (lane < 48) {
        const f32x4 *src = reinterpret_cast<const f32x4 *>(red + (lane >> 2) * 64 + (lane & 3) * 16);
        const f32x4 r0 = src[0], r1 = src[1], r2 = src[2], r3 = src[3];
        t = (((r0.x + r0.y) + (r0.z + r0.w)) + ((r1.x + r1.y) + (r1.z + r1.w))) +
            (((r2.x + r2.y) + (r2.z + r2.w)) + ((r3.x + r3.y) + (r3.z + r3.w)));
    }
    t += dpp<0xb1>(t);
    t += dpp<0x4e>(t);
    if (lane < 48 && (lane & 3) == 0) out[lane >> 2] = t;
    wave_lds_sync();
}

// Adds a view's adjoint box to the global sums and clears what it read.
__device__ __forceinline__ void flush_box(const PixBox &box, int *adj_box, unsigned long long *adj, int W, int H)
{
    const int area = box.w * box.h;
    const float inv_w = 1.0f / static_cast<float>(box.w);
    for (int e = threadIdx.x; e < area; e += kBlock) {
        int r, c;
        box_rc(e, box.w, inv_w, r, c);
        const int x = box.x0 + c, y = box.y0 + r;
        const int val = adj_box[e];
        adj_box[e] = 0;
        if (x >= 0 && x < W && y >= 0 && y < H && val != 0) atomicAdd(adj + static_cast<int64_t>(y) * W + x, widen(val));
    }
}

// Workgroup (b, y): views [n y / gridDim.y, n (y + 1) / gridDim.y) of block b.
// Bound by the instructions of the FP64 projection and of the camera terms.
// Away from the body the sigmoid differs from the label by less than 2^-20, so most
// workgroups have no voxel whose term can round to something (scatters): these are
// cold and need no adjoint box, no flush and fewer barriers; their views' boxes are
// staged in groups, as in the forward, and views whose box misses the image are passed
// over. In a hot workgroup every voxel adds its four tap terms to the view's box in
// LDS (leaving out those that round to 0: 138 x 174 x 103 x 12 views, a fiftieth hot,
// 151 us against 144). Where a view's box is larger than its LDS, what is left of the
// global atomics is the surface's; there the terms of 0 are left out. Both kinds share one
// loop over the views: in two of their own the kernel is 37 KB of instructions
// against 28, and 138 x 174 x 103 x 12 takes 177 us hot against 166. Backward pass
// (zeroing, this kernel, pixel chain) at 160^3 x 8 views of 1280x720: 1706 -> 225 us;
// 224^3 x 12: 765 -> 458; 128^3 x 8 of 640x480: 94 -> 87. Grids of fewer than kBwdBlocks
// blocks split their views over gridDim.y (61 x 53 x 47 x 5 views, 96 blocks: 41 -> 26 us).
__global__ __launch_bounds__(kBlock) void diff_bwd_kernel(DiffArgs a)
{
    constexpr int kRed = 12 * 64;                       // floats of one wave's camera reduction
    constexpr int kGroup = 2 * kBoxCap - kWaves * kRed; // floats of a group's boxes
    __shared__ __align__(16) float arena[2 * kBoxCap];
    __shared__ float cam[kWaves][kMaxViews * 12];
    __shared__ PixBox boxes[kMaxViews];
    const Coords q = block_coords<true>(a.nx, a.ny, a.nz);
    const float X = a.ox + a.h * (static_cast<float>(q.i) + 0.5f);
    const float Y = a.oy + a.h * (static_cast<float>(q.j) + 0.5f);
    const double Xd = centre64(a.ox, a.h, q.i), Yd = centre64(a.oy, a.h, q.j);
    const float gl = *a.grad_loss;
    const float qscale = ldexpf(1.0f, adjoint_exponent(gl, a.inv_count));
    const int v_lo = a.n * static_cast<int>(blockIdx.y) / static_cast<int>(gridDim.y);
    const int v_hi = a.n * static_cast<int>(blockIdx.y + 1) / static_cast<int>(gridDim.y);

    float gv[kFZ];
    bool any = false, hot = false;
#pragma unroll
    for (int kk = 0; kk < kFZ; ++kk) {
        const int k = q.kb + kk;
        gv[kk] = 0.0f;
        if (q.i < a.nx && q.j < a.ny && k < a.nz && in_region(a, q.i, q.j, k)) {
            const int64_t idx = (static_cast<int64_t>(k) * a.ny + q.j) * a.nx + q.i;
            gv[kk] = gl * (sigmoidf_stable(a.logits[idx]) - static_cast<float>(a.labels[idx])) * a.inv_count;
            any = any || gv[kk] != 0.0f;
            hot = hot || scatters(gv[kk], qscale);
        }
    }
    const int wave = threadIdx.x >> 6;
    __shared__ int seen[kWaves];
    const int wave_seen = (__any(any) ? 1 : 0) | (__any(hot) ? 2 : 0);
    if ((threadIdx.x & 63) == 0) seen[wave] = wave_seen;
    __syncthreads();
    int block_seen = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) block_seen |= seen[w];
    block_seen = __builtin_amdgcn_readfirstlane(block_seen);
    const bool block_any = block_seen != 0, block_hot = (block_seen & 2) != 0;
    // a workgroup with no voxel in the loss region contributes nothing
    if (!block_any) {
        for (int e = 12 * v_lo + static_cast<int>(threadIdx.x); e < 12 * v_hi; e += kBlock)
            a.cam_part[static_cast<int64_t>(blockIdx.x) * a.n * 12 + e] = 0.0f;
        return;
    }
    // not widened to pieces: a hot box is as wide to flush, and where boxes are large fewer fit
    // a group (129^3 x 15 cold views 140 -> 135 us without, 128^3 x 8 75 both)
    compute_boxes<kFX, kFY, kFZ>(a, q.bi, q.bj, q.kb, kBoxCap, false, !block_hot, boxes);

    int *adj_box = reinterpret_cast<int *>(arena + kBoxCap);
    // the adjoint box starts at zero once; each view's flush clears the
    // entries it reads, and a view scatters only inside its own box
    if (block_hot)
        for (int e = threadIdx.x; e < kBoxCap; e += kBlock) adj_box[e] = 0;
    __syncthreads();                        // boxes visible
    const uint32_t boxed = views_with(boxes, v_lo, v_hi, 1), missed = views_with(boxes, v_lo, v_hi, kMissed);
    // each wave reduces in its own 768 floats: past the boxes of the group, or in the
    // view's staged box once it is free
    float *red = arena + (block_hot ? 0 : kGroup) + wave * kRed;
    for (int v0 = v_lo; v0 < v_hi;) {
        int v1 = v0 + 1;
        if (!block_hot) {
            v1 = stage_group<kGroup>(a, v0, v_hi, boxed, boxes, arena);
            __syncthreads();                // every wave's loads have landed
        }
        int off = 0;
        for (int v = v0; v < v1; ++v) {
            if (missed >> v & 1) {          // samples that are all 0, and finite gradients
                if ((threadIdx.x & 63) < 12) cam[wave][v * 12 + (threadIdx.x & 63)] = 0.0f;
                continue;
            }
            const ViewGeom &g = a.view[v];
            const Proj64 p = proj64_view(a, v, Xd, Yd);
            CamSums s;
            if (!(boxed >> v & 1)) {
                map_voxels(a, g, p, q.kb, gv, qscale, s);
            } else {
                const PixBox box = read_box(boxes, v);
                if (block_hot) {
                    __syncthreads();        // the previous views' flush and camera sums are done
                    stage_box(arena, box, a.lmap + g.map_off, g.W, g.H);
                    __syncthreads();
                    box_voxels<true>(a, p, box, arena, adj_box, q.kb, gv, qscale, s);
                    __syncthreads();        // every scatter into the box is done
                    flush_box(box, adj_box, reinterpret_cast<unsigned long long *>(a.adj) + g.map_off, g.W, g.H);
                } else {
                    box_voxels<false>(a, p, box, arena + off, nullptr, q.kb, gv, qscale, s);
                    off += box_floats(box);
                }
            }
            wave_camera_sums(s, X, Y, red, &cam[wave][v * 12]);
        }
        v0 = v1;
        if (!block_hot && v0 < v_hi) __syncthreads();   // the group's reads are done
    }
    __syncthreads();
    for (int e = 12 * v_lo + static_cast<int>(threadIdx.x); e < 12 * v_hi; e += kBlock) {
        float s = 0.0f;
        for (int w = 0; w < kWaves; ++w) s += cam[w][e];
        a.cam_part[static_cast<int64_t>(blockIdx.x) * a.n * 12 + e] = s;
    }
}

// The 12 camera-gradient entries of view v: gP[12v + e] = sum over the
// backward workgroups b of cam_part[b][12v + e], in FP64 and a fixed order
// (thread t adds b = t, t + 256, ...; then wave butterflies; then the four
// waves in order). Run by one 256-lane workgroup per view of the pixel chain,
// which follows the backward kernel on the stream.
__device__ __forceinline__ void camera_gradient(const ChainArgs &a, int v)
{
    __shared__ double wsum[kWaves][12];
    const int ne = a.n * 12;
    double acc[12];
#pragma unroll
    for (int e = 0; e < 12; ++e) acc[e] = 0.0;
    for (int64_t b = threadIdx.x; b < a.cam_parts; b += 256) {
        const float *row = a.cam_part + b * ne + v * 12;
#pragma unroll
        for (int e = 0; e < 12; ++e) acc[e] += static_cast<double>(row[e]);
    }
#pragma unroll
    for (int e = 0; e < 12; ++e) {
        const double w = wave_sum(acc[e]);
        if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6][e] = w;
    }
    __syncthreads();
    if (threadIdx.x < 12) {
        double sum = 0.0;
        for (int w = 0; w < kWaves; ++w) sum += wsum[w][threadIdx.x];
        a.gP[v * 12 + threadIdx.x] = static_cast<float>(sum);
    }
}

// dLoss/dmu_c and dLoss/dvar_c of one pixel from its adjoint A (the
// reciprocal of each variance once, refined to about half an ulp).
__device__ __forceinline__ void chain_pixel(float A, float i0, float i1, float i2, const float m[3], const float v[3],
                                            float k0, float gm[3], float gvv[3])
{
    const float I[3] = {i0, i1, i2};
    float t[3], rv[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        rv[c] = recip(v[c]);
        t[c] = (I[c] - m[c]) * rv[c];
    }
    const float q = fmaf(I[0] - m[0], t[0], fmaf(I[1] - m[1], t[1], (I[2] - m[2]) * t[2]));   // sum d_c^2 / v_c
    const float half_logdet = (0.5f * kLn2) * (__builtin_amdgcn_logf(v[0] * v[1]) + __builtin_amdgcn_logf(v[2]));
    const float d = (k0 - half_logdet) - 0.5f * q;
    const float s = -A * sigmoid_fast(d);           // dLoss/dd
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        gm[c] = s * t[c];
        gvv[c] = s * (0.5f * t[c] * t[c] - 0.5f * rv[c]);
    }
}

typedef long long i64x2 __attribute__((ext_vector_type(2)));

// The chain for the pixels [p0, p0 + 256) of one view (p0 a multiple of 4,
// all inside the view): each load instruction of the wave reads one
// contiguous span, the lanes regroup the inputs per pixel quad through LDS
// (as the likelihood pass does) and regroup the gradients back so that each
// store instruction writes one contiguous span.
__device__ __forceinline__ void chain_wave(const ChainView &cv, const long long *adj, double unit, float k0,
                                           int64_t p0, SlmStage &st)
{
    const int lane = static_cast<int>(threadIdx.x & 63);
    const f32x4 *mp = reinterpret_cast<const f32x4 *>(cv.mean + 3 * p0);
    const f32x4 *vp = reinterpret_cast<const f32x4 *>(cv.var + 3 * p0);
    const uint32_t *ip = reinterpret_cast<const uint32_t *>(cv.img + 3 * p0);
    const i64x2 *ap = reinterpret_cast<const i64x2 *>(adj + p0 + 4 * lane);
    f32x4 m[3], v[3];
    uint32_t w[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        m[r] = __builtin_nontemporal_load(mp + lane + 64 * r);
        v[r] = __builtin_nontemporal_load(vp + lane + 64 * r);
        w[r] = __builtin_nontemporal_load(ip + lane + 64 * r);
    }
    const i64x2 a01 = __builtin_nontemporal_load(ap), a23 = __builtin_nontemporal_load(ap + 1);
    const float A[4] = {static_cast<float>(static_cast<double>(a01.x) * unit), static_cast<float>(static_cast<double>(a01.y) * unit),
                        static_cast<float>(static_cast<double>(a23.x) * unit), static_cast<float>(static_cast<double>(a23.y) * unit)};
    f32x4 qm[3], qv[3];
    uint32_t qw[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        st.f[lane + 64 * r] = m[r];
        st.w[lane + 64 * r] = w[r];
    }
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        qm[r] = st.f[3 * lane + r];
        qw[r] = st.w[3 * lane + r];
    }
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 3; ++r) st.f[lane + 64 * r] = v[r];
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 3; ++r) qv[r] = st.f[3 * lane + r];
    wave_lds_sync();
    float mm[12], vv[12], gm[12], gvv[12];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        mm[4 * r] = qm[r].x; mm[4 * r + 1] = qm[r].y; mm[4 * r + 2] = qm[r].z; mm[4 * r + 3] = qm[r].w;
        vv[4 * r] = qv[r].x; vv[4 * r + 1] = qv[r].y; vv[4 * r + 2] = qv[r].z; vv[4 * r + 3] = qv[r].w;
    }
#pragma unroll
    for (int px = 0; px < 4; ++px) {
        const int b = 3 * px;
        chain_pixel(A[px], byte_of(qw[b / 4], b % 4), byte_of(qw[(b + 1) / 4], (b + 1) % 4),
                    byte_of(qw[(b + 2) / 4], (b + 2) % 4), mm + b, vv + b, k0, gm + b, gvv + b);
    }
    f32x4 *gmo = reinterpret_cast<f32x4 *>(cv.gmean + 3 * p0);
    f32x4 *gvo = reinterpret_cast<f32x4 *>(cv.gvar + 3 * p0);
#pragma unroll
    for (int r = 0; r < 3; ++r) st.f[3 * lane + r] = f32x4{gm[4 * r], gm[4 * r + 1], gm[4 * r + 2], gm[4 * r + 3]};
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 3; ++r) gmo[lane + 64 * r] = st.f[lane + 64 * r];
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 3; ++r) st.f[3 * lane + r] = f32x4{gvv[4 * r], gvv[4 * r + 1], gvv[4 * r + 2], gvv[4 * r + 3]};
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < 3; ++r) gvo[lane + 64 * r] = st.f[lane + 64 * r];
}

__global__ __launch_bounds__(256) void pixel_chain_kernel(ChainArgs a)
{
    __shared__ SlmStage st[4];
    if (blockIdx.x == 0) camera_gradient(a, static_cast<int>(blockIdx.y));
    const ChainView cv = a.view[blockIdx.y];
    const int wave = static_cast<int>(threadIdx.x >> 6);
    const int64_t pw = (static_cast<int64_t>(blockIdx.x) * 4 + wave) * 256;   // the wave's first pixel
    if (pw >= cv.npix) return;
    const long long *adj = reinterpret_cast<const long long *>(a.adj) + cv.map_off;
    const double unit = ldexp(1.0, -adjoint_exponent(*a.grad_loss, a.inv_count));
    if (pw + 256 <= cv.npix) {
        chain_wave(cv, adj, unit, a.k0, pw, st[wave]);
        return;
    }
    // the view's last, partial span: lane by lane
    const int64_t p0 = pw + 4 * static_cast<int64_t>(threadIdx.x & 63);
    if (p0 >= cv.npix) return;
    for (int64_t p = p0; p < cv.npix && p < p0 + 4; ++p) {
        const uint8_t *I = cv.img + 3 * p;
        const float A = static_cast<float>(static_cast<double>(adj[p]) * unit);
        chain_pixel(A, I[0], I[1], I[2], cv.mean + 3 * p, cv.var + 3 * p, a.k0, cv.gmean + 3 * p, cv.gvar + 3 * p);
    }
}

}  // namespace

int64_t diff_fwd_blocks(int nx, int ny, int nz)
{
    return static_cast<int64_t>((nx + kFX - 1) / kFX) * ((ny + kFY - 1) / kFY) * ((nz + kFZ - 1) / kFZ);
}
int64_t diff_bwd_blocks(int nx, int ny, int nz) { return diff_fwd_blocks(nx, ny, nz); }

hipError_t launch_diff_forward(const DiffArgs &a, float *loss, hipStream_t s)
{
    const int64_t nb = diff_fwd_blocks(a.nx, a.ny, a.nz);
    if (nb > 0) hipLaunchKernelGGL(diff_fwd_kernel, dim3(static_cast<unsigned>(nb)), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(loss_finalize_kernel, dim3(1), dim3(256), 0, s, a.loss_part, nb, a.inv_count, loss);
    return hipGetLastError();
}

hipError_t launch_diff_backward(const DiffArgs &a, const ChainArgs &c, int64_t map_floats, int64_t max_npix,
                                float *gP, hipStream_t s)
{
    if (map_floats > 0) {
        const int64_t n4 = map_floats / 4;
        const int64_t blocks = std::min<int64_t>((n4 + 1023) / 1024, 4096);
        hipLaunchKernelGGL(zero_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, a.adj, n4);
    }
    const int64_t nb = diff_bwd_blocks(a.nx, a.ny, a.nz);
    if (nb > 0 && a.n > 0) {
        // with few views, what every workgroup does before them outweighs a second round
        // of workgroups (640 blocks: 3 views 34.7 us in one, 40.7 in two; 13 views 51.1 / 45.3)
        const int64_t fit = a.n >= 12 ? (kBwdBlocks + nb - 1) / nb : std::max<int64_t>(kBwdBlocks / nb, 1);
        const int64_t split = std::min<int64_t>(a.n, fit);
        hipLaunchKernelGGL(diff_bwd_kernel, dim3(static_cast<unsigned>(nb), static_cast<unsigned>(split)), dim3(kBlock), 0, s, a);
    }
    if (a.n > 0) {
        // the pixel chain also sums the camera-gradient partials (camera_gradient)
        ChainArgs ca = c;
        ca.cam_part = a.cam_part;
        ca.cam_parts = nb > 0 ? nb : 0;
        ca.gP = gP;
        const int64_t quads = (max_npix + 3) / 4;
        hipLaunchKernelGGL(pixel_chain_kernel, dim3(static_cast<unsigned>((quads + 255) / 256), static_cast<unsigned>(c.n)),
                           dim3(256), 0, s, ca);
    }
    return hipGetLastError();
}

}  // namespace psfs
