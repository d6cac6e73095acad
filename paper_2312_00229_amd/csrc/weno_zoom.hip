// The doubling's kernels and their launches, one object per I/O mode: this file
// is compiled once for each value of WENO_IO (kIo* of weno_fwd.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>

#include "weno_fwd.h"
#include "weno_internal.h"
#include "weno_zoom.h"

#ifndef WENO_IO
#error "compile with -DWENO_IO=<I/O mode>"
#endif

using namespace wz;

namespace {

// per-plane context: buffer resources over the plane's byte extent
__device__ __forceinline__ StripCtx make_ctx(const FwdJob& jb, int n, int c, float out_scale)
{
    StripCtx cx;
    cx.src = make_rsrc(jb.src + n * jb.s_n + c * jb.s_c, jb.src_extent);
    cx.dst = make_rsrc(jb.dst + n * jb.d_n + c * jb.d_c, jb.dst_extent);
    cx.s_h = (uint32_t)jb.s_h;
    cx.s_w_bytes = (uint32_t)jb.s_w;
    cx.d_h = (uint32_t)jb.d_h;
    cx.d_w = (uint32_t)jb.d_w;
    cx.H = jb.H;
    cx.W = jb.W;
    cx.src_shift = jb.src_shift;
    cx.src_h = jb.src_h;
    cx.src_w = jb.src_w;
    cx.out_scale = out_scale;
    return cx;
}

// this wave's LDS rows for staged stores
template <int COLS, int IO, int WAVES = kWavesPerBlock>
__device__ __forceinline__ float* wave_stage()
{
    if constexpr (io_out_staged(IO)) {
        __shared__ __align__(16) float rows[WAVES * stage_floats<COLS, IO>()];
        return rows + (threadIdx.x >> 6) * stage_floats<COLS, IO>();
    } else {
        return nullptr;
    }
}

// TAIL (two columns only): the launch has one-column tail strips
// (jb.tail_rows > 0) and one wave index across the planes
// Two-column kernels are held to 168 VGPRs, three waves per SIMD: strided float
// destinations would take 170 (two to four values spill).
template <int COLS, int BETA, int IO, Pace PACE, bool TAIL = false>
__global__ __launch_bounds__(kBlock, COLS == 2 ? 3 : 1) void zoom2x_kernel(FwdJob jb, FwdParams P, int rows_per_strip)
{
    // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.
    // Renumber them so that every XCD gets a contiguous range of strips
    // (whole bands of adjacent rows): the 9 halo rows a strip shares with the
    // strip above are then re-read from the same L2.  A bijection on
    // [0, gridDim.x).  The XCD of a workgroup is its linear index (plane-major)
    // mod 8, so the XCD of a strip rotates from plane to plane, which spreads
    // the planes' workgroups evenly over the XCDs.  With tail strips the grid
    // is one-dimensional and every XCD gets a contiguous range of waves, plane
    // after plane.  For images whose planes are interleaved (HWC) a row of the grid
    // is an image, a multiple of 8 workgroups per plane, and on each
    // XCD a strip's workgroups of all the planes follow each other: the lines
    // the planes share meet in one L2 while they are there, instead of reaching
    // HBM once per plane with a third of their bytes each (1080p RGB uint8:
    // writes 3.0x -> 1.0x the output, reads 4.1x -> 1.1x the input).
    const int nb = gridDim.x, b = blockIdx.x;
    const int xcd = b % kXcds, k = b / kXcds;
    const int logical = xcd * (nb / kXcds) + min(xcd, nb % kXcds) + k;
    // the wave index is the same in every lane; say so, so that strip rows and
    // buffer offsets live in SGPRs
    const int wave = __builtin_amdgcn_readfirstlane(logical * kWavesPerBlock + (threadIdx.x >> 6));
    float* const stage = wave_stage<COLS, IO>();
    if constexpr (TAIL) {
        // One wave index across the planes (gridDim.y is 1).  Per plane: the
        // two-column strips, band by band, then the one-column strips of the
        // last columns (no more than a one-column strip owns), whose bands
        // are taller so that each walks about as long as a two-column strip.
        static_assert(COLS == 2, "tail strips follow two-column strips");
        const int n2 = jb.strips_x * jb.strips_y, per_plane = n2 + jb.tail_bands;
        const int plane = wave / per_plane;
        if (plane >= jb.planes) return;  // whole wave
        const int w = wave - plane * per_plane;
        const int n = plane / jb.C, c = plane - n * jb.C;
        const StripCtx cx = make_ctx(jb, n, c, P.out_scale);
        if (w < n2) {
            const int sy = w / jb.strips_x, sx = w - sy * jb.strips_x;
            const int R0 = sy * rows_per_strip;
            zoom_strip<2, BETA, IO, PACE>(cx, P, sx * strip_own<2>(), R0, min(R0 + rows_per_strip, jb.H),
                                           stage);
        } else {
            const int R0 = (w - n2) * jb.tail_rows;
            zoom_strip<1, BETA, IO, PACE>(cx, P, jb.strips_x * strip_own<2>(), R0, min(R0 + jb.tail_rows, jb.H),
                                           stage);
        }
    } else {
        int n, c, w = wave;
        if (jb.share) {
            // image blockIdx.y; on each XCD workgroup by workgroup, plane by plane
            const int per_xcd = nb / (kXcds * jb.C);
            n = blockIdx.y;
            c = k % jb.C;
            w = __builtin_amdgcn_readfirstlane((xcd * per_xcd + k / jb.C) * kWavesPerBlock + (threadIdx.x >> 6));
        } else {
            n = blockIdx.y / jb.C;
            c = blockIdx.y - n * jb.C;
        }
        if (w >= jb.strips_x * jb.strips_y) return;  // whole wave
        const int sy = w / jb.strips_x;
        const int sx = w - sy * jb.strips_x;
        const StripCtx cx = make_ctx(jb, n, c, P.out_scale);
        const int R0 = sy * rows_per_strip;
        const int R1 = min(R0 + rows_per_strip, jb.H);
        zoom_strip<COLS, BETA, IO, PACE>(cx, P, sx * strip_own<COLS>(), R0, R1, stage);
    }
}

// Persistent kernel over the strips of many images, those of one I/O mode (a
// kernel that switched between all modes took the registers of the largest:
// 176 VGPRs, two waves per SIMD).  A unit is one strip of a plane, or of a group
// of an image's interleaved planes (wz_unit_groups).  One workgroup fills a
// compute unit (three waves per SIMD, four with one column per lane); workgroup
// g takes units g, g + grid, ..., and its waves share them out through a ticket
// in LDS, a ticket being a plane of a unit.  The table holds the images by their
// planes per unit, so the units come in runs of equal ticket counts, and a wave
// goes from run to run as its tickets pass their ends (with the largest count
// for all, a 64-channel image left 61 empty tickets in each unit of the others:
// one beside 64 planar float32 images 281 us, now 95).  The planes of a strip,
// which fill the same lines with a byte in three each, then run side by side on
// one compute unit, and the lines leave its L2 whole.  Units of more than eight
// planes, whose images may be in several groups, are dealt out so that every XCD
// gets consecutive ones: the groups of a strip then meet in one L2 (32 float32
// HWC images of 64 channels and 64 squared 545 -> 285 us; units of 3 planes
// would lose, 83 -> 103).  The work is vector issue, the same on every compute
// unit, and the images are stored largest first and in bands of nearly equal
// height, so fixed shares come out even; within a compute unit they would not (a
// SIMD serves its oldest wave first: workgroups of four waves with a ticket each,
// 2663 us for the 512 images below).  A queue for the whole device does not pay:
// a ticket drawn by atomics on one address takes ~14 ns, one after another, and each wave's
// last, empty one too (24 uint8 HWC images of 85 to 415 squared 82 -> 49 us
// in the same strips, 512 of 32 to 1024 squared 2540 -> 2424).
template <int COLS>
constexpr int batch_waves() { return COLS == 2 ? 12 : 16; }

// The table's parts come as arguments: an image count read from the table to
// find them would be one more load, from cold memory, ahead of the first strip.
template <int COLS, int BETA, int IO>
__global__ __launch_bounds__(kWave * batch_waves<COLS>()) void zoom2x_batched_kernel(
    const BatchRun* __restrict__ runs, const FwdJob* __restrict__ jobs, const int64_t* __restrict__ prefix,
    const FwdParams* __restrict__ params)
{
    __shared__ int next;
    const int lane = threadIdx.x & (kWave - 1);
    float* const stage = wave_stage<COLS, IO, batch_waves<COLS>()>();
    if (threadIdx.x == 0) next = batch_waves<COLS>();
    __syncthreads();
    auto draw = [&]() {
        int got = 0;
        if (lane == 0) got = atomicAdd(&next, 1);
        // broadcast lane 0's ticket as a provably uniform (scalar) value, so the
        // image table is read with scalar loads and the buffer resources stay
        // in SGPRs
        return __builtin_amdgcn_readfirstlane(got);
    };
    // the workgroup's place among the units of a run
    auto place = [&](int planes) {
        const int nb = gridDim.x, xcd = blockIdx.x % kXcds;
        return planes > 8 ? xcd * (nb / kXcds) + min(xcd, nb % kXcds) + (int)blockIdx.x / kXcds : (int)blockIdx.x;
    };
    // The run of units the wave is at, the workgroup's tickets before it, where
    // the run starts among the places (modulo the grid), and how far ahead of
    // that the workgroup's first unit is
    int passed = 0, start = 0;
    // A wave's first ticket is its number, which spreads the first strips over
    // the SIMDs: drawn, several may go to one (8 gray and RGB uint8 images of 32
    // to 128 squared 13.1 us, drawn 18.5; 8 float32 HWC ones of 128 to 512
    // squared in 32-row two-column strips 33, drawn 49).
    int ticket = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    BatchRun run = runs[IO];
    int ahead = place(run.planes);
    for (;; ticket = draw()) {
        int slot;
        int64_t unit;
        for (;;) {
            const int turn = (ticket - passed) / run.planes;
            slot = ticket - passed - turn * run.planes;
            unit = run.first + ahead + (int64_t)turn * gridDim.x;
            if (unit < run.end) break;
            if (run.next < 0) return;  // every wave reaches this exit; no barrier follows
            const int64_t units = run.end - run.first;
            if (ahead < units) passed += (int)((units - ahead + gridDim.x - 1) / gridDim.x) * run.planes;
            start = (int)((start + units) % gridDim.x);
            run = runs[run.next];
            ahead = place(run.planes) - start;
            if (ahead < 0) ahead += (int)gridDim.x;
        }
        // image k of the run with prefix[k] <= unit < prefix[k+1]
        int lo = run.image, hi = run.image_end - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (prefix[mid] <= unit) lo = mid; else hi = mid - 1;
        }
        const FwdJob jb = jobs[lo];
        const FwdParams P = params[lo];
        const int per_plane = jb.strips_x * jb.strips_y;
        int64_t strip = unit - prefix[lo];   // of the image's planes, or of its interleaved ones as a whole
        int group = 0;
        const int groups = wz_unit_groups(jb.C, jb.share);
        if (groups > 1) {
            const int64_t whole = strip / groups;
            group = (int)(strip - whole * groups);
            strip = whole;
        }
        const int outer = (int)(strip / per_plane);
        const int wv = (int)(strip - (int64_t)outer * per_plane);
        const int sy = wv / jb.strips_x;
        const int sx = wv - sy * jb.strips_x;
        int n = outer, c = group * run.planes + slot;
        if (!jb.share) {
            n = outer / jb.C;
            c = outer - n * jb.C;
        }
        if (c >= jb.C) continue;   // the last group holds fewer planes
        const StripCtx cx = make_ctx(jb, n, c, P.out_scale);
        const int R0 = sy * jb.rows;
        const int R1 = min(R0 + jb.rows, jb.H);
        zoom_strip<COLS, BETA, IO>(cx, P, sx * strip_own<COLS>(), R0, R1, stage);
    }
}

// Workgroups of a kernel that one compute unit holds at once.  Cached per
// kernel: it depends only on the kernel's registers and the architecture,
// and the library is built for one architecture.
template <int COLS, int BETA, int IO>
int resident_blocks()
{
    static std::atomic<int> cache{0};
    int v = cache.load();
    if (v == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &v, reinterpret_cast<const void*>(zoom2x_kernel<COLS, BETA, IO, kPacedThrough>), kBlock, 0) != hipSuccess ||
            v <= 0)
            v = 1;
        cache.store(v);
    }
    return v;
}

// A launch whose workgroups all fit on the device at once (one round) is
// paced (zoom_strip); one of several rounds is not.
template <int COLS, int BETA, int IO, bool TAIL>
hipError_t launch_paced(const FwdJob& jb, const FwdParams& P, int rows, dim3 grid, hipStream_t st)
{
    const int64_t blocks = (int64_t)grid.x * grid.y;
    if (blocks > (int64_t)resident_blocks<COLS, BETA, IO>() * wz_device_cus()) {
        hipLaunchKernelGGL((zoom2x_kernel<COLS, BETA, IO, kRounds, TAIL>), grid, dim3(kBlock), 0, st, jb, P, rows);
        return hipGetLastError();
    }
    if constexpr (!io_out_u8(IO) && !io_out_spread(IO)) {
        const int64_t px = (int64_t)jb.planes * jb.H * jb.W;
        if (px * (io_in_u8(IO) ? 1 : 4) + 4 * px * 4 > kInfinityCache) {
            hipLaunchKernelGGL((zoom2x_kernel<COLS, BETA, IO, kPacedBack, TAIL>), grid, dim3(kBlock), 0, st, jb, P,
                               rows);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((zoom2x_kernel<COLS, BETA, IO, kPacedThrough, TAIL>), grid, dim3(kBlock), 0, st, jb, P, rows);
    return hipGetLastError();
}

template <int COLS, int BETA, int IO>
hipError_t launch_single(const FwdJob& jb, const FwdParams& P, int rows, hipStream_t st)
{
    dim3 grid(wz_grid_x((int64_t)jb.strips_x * jb.strips_y, jb.share), jb.planes);
    if (jb.share) grid = dim3(grid.x * jb.C, jb.planes / jb.C);   // an image's planes interleaved (zoom2x_kernel)
    if constexpr (COLS == 2) {
        if (jb.tail_rows > 0) {  // one wave index across the planes
            const int64_t waves = (int64_t)jb.planes * ((int64_t)jb.strips_x * jb.strips_y + jb.tail_bands);
            grid = dim3((unsigned)((waves + kWavesPerBlock - 1) / kWavesPerBlock), 1);
            return launch_paced<COLS, BETA, IO, true>(jb, P, rows, grid, st);
        }
    }
    return launch_paced<COLS, BETA, IO, false>(jb, P, rows, grid, st);
}

// persistent launch: a workgroup per compute unit, no more than there are units
// for
template <int COLS, int BETA, int IO>
hipError_t launch_batched(const weno_batch_plan_t* plan, hipStream_t st)
{
    const int64_t blocks = std::min<int64_t>(wz_device_cus(), plan->total_items);
    const uint8_t* const tab = (const uint8_t*)plan->d_workspace;
    hipLaunchKernelGGL((zoom2x_batched_kernel<COLS, BETA, IO>), dim3((unsigned)blocks),
                       dim3(kWave * batch_waves<COLS>()), 0, st, (const BatchRun*)(tab + batch_runs_offset()),
                       (const FwdJob*)(tab + batch_jobs_offset(plan->count)),
                       (const int64_t*)(tab + batch_prefix_offset(plan->count)),
                       (const FwdParams*)(tab + batch_params_offset(plan->count)));
    return hipGetLastError();
}

template <int COLS, int IO>
hipError_t single_beta(const FwdJob& jb, const FwdParams& P, int beta_mode, int rows, hipStream_t st)
{
    if (beta_mode == 2) return launch_single<COLS, 2, IO>(jb, P, rows, st);
    if (beta_mode == 1) return launch_single<COLS, 1, IO>(jb, P, rows, st);
    return launch_single<COLS, kBetaGeneral, IO>(jb, P, rows, st);
}

template <int COLS, int IO>
hipError_t batched_beta(const weno_batch_plan_t* plan, hipStream_t st)
{
    if (plan->beta_mode == 2) return launch_batched<COLS, 2, IO>(plan, st);
    if (plan->beta_mode == 1) return launch_batched<COLS, 1, IO>(plan, st);
    return launch_batched<COLS, kBetaGeneral, IO>(plan, st);
}

hipError_t single(const FwdJob& jb, const FwdParams& P, int beta_mode, int cols, int rows, hipStream_t st)
{
    return cols == 1 ? single_beta<1, WENO_IO>(jb, P, beta_mode, rows, st)
                     : single_beta<2, WENO_IO>(jb, P, beta_mode, rows, st);
}

hipError_t batched(const weno_batch_plan_t* plan, hipStream_t st)
{
    return plan->cols_per_lane == 1 ? batched_beta<1, WENO_IO>(plan, st) : batched_beta<2, WENO_IO>(plan, st);
}

}  // namespace

template <>
ZoomLauncher zoom_launcher<WENO_IO>()
{
    return {single, batched};
}
