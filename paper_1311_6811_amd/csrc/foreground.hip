// Learned foreground colour model for frames after the first (Eq. 1-2 use a
// uniform foreground density, as nothing is known of the foreground's colours
// at the first frame, Sec. 2.2.2). Three launches:
//   fg_zero_kernel     bin counts to 0
//   fg_hist_kernel     per workgroup an LDS histogram of the foreground pixels
//                      (mask != 0, or log(2*SLM) > 0 of the previous frame)
//                      of one view, added to the global counts with integer
//                      atomics (order-independent)
//   fg_density_kernel  log density of one colour value per bin, Laplace-
//                      smoothed: log((c + 1) / ((N + 4096) * 4096)), in FP64
#include "kernels_common.h"

namespace psfs {
namespace {

using namespace dev;

constexpr int kBins = PSFS_FG_BINS;
constexpr int kHistThreads = 1024;
constexpr int kPixPerBlock = 16 * kHistThreads;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void fg_zero_kernel(uint32_t *counts)
{
    counts[blockIdx.x * 256 + threadIdx.x] = 0u;
}

// Marks of the 16 pixels [p, p + 16) (bit e: pixel p + e is foreground), all
// inside the view.
__device__ __forceinline__ uint32_t marks16(const uint8_t *mask, const float *map, int64_t p)
{
    uint32_t bits = 0;
    if (mask) {
        u32x4 w;                                    // any alignment
        __builtin_memcpy(&w, mask + p, 16);
#pragma unroll
        for (int e = 0; e < 16; ++e) bits |= byte_u(w[e >> 2], e & 3) != 0 ? 1u << e : 0u;
    } else {
        f32x4 m[4];
        __builtin_memcpy(m, map + p, 64);
#pragma unroll
        for (int e = 0; e < 16; ++e) bits |= m[e >> 2][e & 3] > 0.0f ? 1u << e : 0u;
    }
    return bits;
}

// grid (ceil(max_npix / kPixPerBlock), views). A lane takes 16 consecutive
// pixels: its marks in one load, and where one is set the 48 image bytes in
// three (pixel by pixel, every image load waited for its mark). The large
// workgroups and the flush in bin order keep the global atomics few per cache
// line: 8 views of 640x480 12.1 -> 7.7 us (10.9 us with 4096 pixels per
// workgroup and four adjacent bins per lane). A workgroup without foreground
// adds nothing.
__global__ __launch_bounds__(kHistThreads) void fg_hist_kernel(FgArgs a)
{
    __shared__ uint32_t h[kBins];
    const SlmView &sv = a.view[blockIdx.y];
    const uint8_t *mask = a.mask[blockIdx.y];
    const float *map = a.lmap ? a.lmap + sv.map_off : nullptr;
    const int64_t p0 = static_cast<int64_t>(blockIdx.x) * kPixPerBlock + 16 * static_cast<int64_t>(threadIdx.x);
    const bool whole = p0 + 16 <= sv.npix;
    uint32_t bits = 0;
    if (whole) {
        bits = marks16(mask, map, p0);
    } else {
        for (int e = 0; e < 16 && p0 + e < sv.npix; ++e)
            if (mask ? mask[p0 + e] != 0 : map[p0 + e] > 0.0f) bits |= 1u << e;
    }
    if (__syncthreads_or(bits != 0 ? 1 : 0) == 0) return;
    uint32_t w[12];
    if (bits != 0 && whole) __builtin_memcpy(w, static_cast<const uint8_t *>(__builtin_assume_aligned(sv.img + 3 * p0, 4)), 48);
#pragma unroll
    for (int r = 0; r < kBins / kHistThreads; ++r) h[threadIdx.x + kHistThreads * r] = 0u;
    __syncthreads();
    if (bits != 0) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if (!(bits & (1u << e))) continue;
            uint32_t c[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) c[q] = whole ? byte_u(w[(3 * e + q) >> 2], (3 * e + q) & 3) : sv.img[3 * (p0 + e) + q];
            atomicAdd(&h[colour_bin(c[0], c[1], c[2])], 1u);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kBins / kHistThreads; ++r) {
        const uint32_t c = h[threadIdx.x + kHistThreads * r];
        if (c) atomicAdd(a.counts + threadIdx.x + kHistThreads * r, c);
    }
}

// Workgroup g: the densities of bins 256 g .. 256 g + 255, one per lane; each
// workgroup sums all the counts itself (16 KB from L2; integers, so every
// workgroup has the same sum). One workgroup for all bins took 10.8 us, its
// lanes 16 FP64 logarithms one after another; 16 workgroups 2.8 us.
__global__ __launch_bounds__(256) void fg_density_kernel(FgArgs a)
{
    __shared__ unsigned long long part[4];
    u32x4 c[kBins / 1024];
    unsigned long long s = 0;
#pragma unroll
    for (int r = 0; r < kBins / 1024; ++r) __builtin_memcpy(&c[r], a.counts + 4 * (threadIdx.x + 256 * r), 16);
    const int b = static_cast<int>(blockIdx.x) * 256 + static_cast<int>(threadIdx.x);
    const uint32_t own = a.counts[b];
#pragma unroll
    for (int r = 0; r < kBins / 1024; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) s += c[r][q];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    s = (part[0] + part[1]) + (part[2] + part[3]);
    const double denom = (static_cast<double>(s) + kBins) * kBins;
    a.logd[b] = static_cast<float>(log((static_cast<double>(own) + 1.0) / denom));
}

}  // namespace

hipError_t launch_foreground(const FgArgs &a, int64_t max_npix, hipStream_t s)
{
    hipLaunchKernelGGL(fg_zero_kernel, dim3(kBins / 256), dim3(256), 0, s, a.counts);
    if (a.n > 0 && max_npix > 0) {
        const dim3 g(static_cast<unsigned>((max_npix + kPixPerBlock - 1) / kPixPerBlock), static_cast<unsigned>(a.n));
        hipLaunchKernelGGL(fg_hist_kernel, g, dim3(kHistThreads), 0, s, a);
    }
    hipLaunchKernelGGL(fg_density_kernel, dim3(kBins / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace psfs
