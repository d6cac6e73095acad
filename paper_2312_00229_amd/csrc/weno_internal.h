// Internal declarations shared by the host files of the library.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "weno_fwd.h"
#include "weno_zoom.h"

// Device-resident table of a batched call, written into the caller's
// workspace by weno_zoom2x_batched_plan:
//   [0, ...)                 BatchRun runs[kIoModes + count]  (the first run of each I/O mode, then the others)
//   then                     FwdJob jobs[count]       (by I/O mode, then most planes per unit, then
//                                                     largest image first)
//   then                     int64_t prefix[count+1]  (first unit of each image: a strip of one plane,
//                                                     or of a group of interleaved planes, wz_unit_planes)
//   then                     FwdParams params[count]
// A run: images of one mode with as many planes per unit, units [first, end).
struct BatchRun {
    int64_t first, end;
    int32_t image, image_end;   // its images
    int32_t planes;             // per unit (tickets)
    int32_t next;               // the mode's next run, or -1
};
constexpr size_t batch_runs_offset() { return 0; }
constexpr size_t batch_jobs_offset(int count)
{
    return batch_runs_offset() + (size_t)(wz::kIoModes + count) * sizeof(BatchRun);
}
constexpr size_t batch_prefix_offset(int count)
{
    return batch_jobs_offset(count) + (size_t)count * sizeof(wz::FwdJob);
}
constexpr size_t batch_params_offset(int count)
{
    return (batch_prefix_offset(count) + (size_t)(count + 1) * sizeof(int64_t) + 15) / 16 * 16;
}
constexpr size_t batch_table_bytes(int count)
{
    return (batch_params_offset(count) + (size_t)count * sizeof(wz::FwdParams) + 255) / 256 * 256;
}

// host helpers (weno_api.hip)
int wz_hip_error(hipError_t e, const char* what);
int wz_esize(int32_t dtype);
int wz_check_tensor(const weno_tensor_t* t);
int wz_check_params(const weno_params_t* p);
int wz_check_pair(const weno_tensor_t* src, const weno_tensor_t* dst, int factor);
void wz_byte_range(const weno_tensor_t* t, uintptr_t* lo, uintptr_t* hi);
bool wz_overlap(const weno_tensor_t* a, const weno_tensor_t* b);
int64_t wz_plane_extent(const weno_tensor_t* t);
double wz_nbw(const weno_params_t* p);
int wz_beta_mode(float beta);
int wz_device_cus();

// Planes of one image interleaved in memory (channels closer together than
// rows, as in HWC): the same strip of its planes touches the same lines.
inline bool planes_share_lines(int C, int64_t sc, int64_t sh)
{
    return C > 1 && sc < sh   /* strides are never negative */;
}

// Workgroups along x that a launch may have: the work-items of a dimension are
// counted in 32 bits, and a launch of more runs without the rest, with no error.
constexpr int64_t kMaxGridX = (1ll << 32) / wz::kBlock - 1;

// Workgroups of a plane of `strips` strips: padded to a multiple of the XCD
// count when the planes share lines (zoom2x_kernel), the padding exiting at
// once.  The busiest XCD then holds planes x grid_x / 8 of them.
inline int64_t wz_grid_blocks(int64_t strips, bool share)
{
    using namespace wz;
    const int64_t bx = (strips + kWavesPerBlock - 1) / kWavesPerBlock;
    return share ? (bx + kXcds - 1) / kXcds * kXcds : bx;
}
inline int wz_grid_x(int64_t strips, bool share) { return (int)wz_grid_blocks(strips, share); }

// Groups of an image's interleaved planes, the same strip of a group being a
// unit: no more planes than a compute unit has waves for (zoom2x_batched_kernel),
// so that few strips of many planes still reach many compute units (4 uint8 HWC
// images of 64 channels and 64 squared 105 -> 33 us).
__host__ __device__ inline int wz_unit_groups(int C, bool share) { return share ? (C + 15) / 16 : 1; }
// planes of a unit (the last group may hold fewer)
__host__ __device__ inline int wz_unit_planes(int C, bool share)
{
    const int groups = wz_unit_groups(C, share);
    return share ? (C + groups - 1) / groups : 1;
}

// Launches of one I/O mode (weno_zoom.hip, compiled once per mode): one doubling
// of a job with its beta mode, columns per lane and strip height, and a batch
// plan's images of that mode.
struct ZoomLauncher {
    hipError_t (*single)(const wz::FwdJob& jb, const wz::FwdParams& P, int beta_mode, int cols, int rows,
                         hipStream_t st);
    hipError_t (*batched)(const weno_batch_plan_t* plan, hipStream_t st);
};
template <int IO>
ZoomLauncher zoom_launcher();
