// Host-side helpers shared by the C ABI implementation files (not part of the ABI).
#pragma once

#include <cstddef>
#include <cstdint>
#include <map>
#include <mutex>
#include <string>

#include "psfs_internal.h"

namespace psfs {
namespace host {

int fail(int status, const char *fmt, ...);
int hip_fail(hipError_t e, const char *what);
bool aligned(const void *p, size_t a);
bool finite_all(const float *v, int n);
int check_device();
int64_t padded_pixels(int width, int height);
size_t align256(size_t x);
// Whether every voxel centre of the grid projects into view g (nearest sampling:
// P pre-offset) with room for the FP32 rounding of its projection. (The column
// kernels' lanes past the grid's edge take its last voxels' place.)
bool grid_inside(const ViewGeom &g, const psfs_grid &grid);
// Whether the block tile is the better one for the one-frame nearest fusion, and
// boxes staged in LDS for the bilinear fusion.
bool block_pays(const psfs_camera *cams, int n, const psfs_grid &grid, bool step);
constexpr int kNarrowTile = 2, kShallowTile = 3;    // 8 x 16 columns of 4 voxels, 8 x 32 of 2
constexpr int kWideTile = 4;                        // 32 x 8 of 4: the two- and four-frame steps
bool small_grid(const psfs_grid &grid);
bool many_waves(const psfs_grid &grid);
bool bilinear_boxes_pay(const psfs_camera *cams, int n, const psfs_grid &grid);

// Part of the autotuners' cache keys: raised when the kernel behind a tile changes,
// so that choices timed on the older one are not applied.
constexpr int kTileRevision = 2;

// Autotuner cache (tune_cache.hip): $PSFS_AUTOTUNE_CACHE, else
// $HOME/.cache/psfs/autotune.json; callers hold tune_cache_mutex() around
// a read-modify-write.
std::string tune_cache_path();
std::mutex &tune_cache_mutex();
std::map<std::string, int> read_tune_cache(const std::string &path);
void write_tune_cache(const std::string &path, const std::map<std::string, int> &m);

}  // namespace host
}  // namespace psfs

#define PSFS_GUARD_BEGIN try {
#define PSFS_GUARD_END                                                                              \
    }                                                                                               \
    catch (const std::bad_alloc &) { return psfs::host::fail(PSFS_E_RANGE, "out of host memory"); } \
    catch (...) { return psfs::host::fail(PSFS_E_ARG, "unexpected exception"); }
