// C ABI of the WD-WENO 2x zoom library (declarations and contracts in
// include/weno_zoom.h).  Host-side validation, launch configuration and the
// batched and cascade entry points; the doubling's kernels live in
// weno_zoom.hip, the adjoint in weno_bwd.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "weno_zoom.h"
#include "weno_fwd.h"
#include "weno_internal.h"

using namespace wz;

// --------------------------------------------------------------------------
// status / configuration
// --------------------------------------------------------------------------
static thread_local std::string g_status_text;
// 0 / 0 = automatic (chosen per launch from the image size)
static std::atomic<int32_t> g_rows_per_strip{0};
static std::atomic<int32_t> g_cols_per_lane{0};

int wz_hip_error(hipError_t e, const char* what)
{
    g_status_text = std::string(what) + ": " + hipGetErrorString(e);
    return WENO_EHIP;
}

extern "C" const char* weno_status_string(int status)
{
    switch (status) {
    case WENO_OK: return "ok";
    case WENO_EINVAL: return "invalid argument (null pointer, size, shape or parameter)";
    case WENO_EDTYPE: return "unsupported dtype combination";
    case WENO_EOVERLAP: return "output overlaps an input";
    case WENO_ENOSPC: return "workspace too small (weno_zoom2x_batched_noalloc: more images than its fixed scratch holds)";
    case WENO_EHIP:
        if (g_status_text.empty()) return "HIP runtime error";
        return g_status_text.c_str();
    default: return "unknown status";
    }
}

extern "C" const char* weno_version(void) { return "1.0.0"; }

extern "C" weno_params_t weno_default_params(void)
{
    weno_params_t p;
    p.beta = 2.0f;
    p.k_eps = 1e-8f;
    p.h = 1.0f;
    p.nbw = -1.0f;
    p.boundary = WENO_BOUNDARY_CLAMP;
    return p;
}

extern "C" int weno_set_launch_config(int32_t rows_per_strip, int32_t cols_per_lane)
{
    if (rows_per_strip == 0 && cols_per_lane == 0) {  // back to automatic
        g_rows_per_strip.store(0);
        g_cols_per_lane.store(0);
        return WENO_OK;
    }
    if (rows_per_strip < 4 || rows_per_strip > 4096) return WENO_EINVAL;
    if (cols_per_lane != 1 && cols_per_lane != 2) return WENO_EINVAL;
    g_rows_per_strip.store(rows_per_strip);
    g_cols_per_lane.store(cols_per_lane);
    return WENO_OK;
}

extern "C" void weno_get_launch_config(int32_t* rows_per_strip, int32_t* cols_per_lane)
{
    if (rows_per_strip) *rows_per_strip = g_rows_per_strip.load();
    if (cols_per_lane) *cols_per_lane = g_cols_per_lane.load();
}

// --------------------------------------------------------------------------
// validation helpers (shared with the adjoint and the cascade)
// --------------------------------------------------------------------------
int wz_esize(int32_t dtype) { return dtype == WENO_U8 ? 1 : (dtype == WENO_F32 ? 4 : 0); }


int wz_check_tensor(const weno_tensor_t* t)
{
    if (!t || !t->data) return WENO_EINVAL;
    if (wz_esize(t->dtype) == 0) return WENO_EDTYPE;
    if (t->n < 1 || t->c < 1 || t->h < 1 || t->w < 1) return WENO_EINVAL;
    if (t->sn < 0 || t->sc < 0 || t->sh < 0 || t->sw < 0) return WENO_EINVAL;
    return WENO_OK;
}

void wz_byte_range(const weno_tensor_t* t, uintptr_t* lo, uintptr_t* hi)
{
    const int64_t es = wz_esize(t->dtype);
    const int64_t last = ((int64_t)(t->n - 1) * t->sn + (int64_t)(t->c - 1) * t->sc + (int64_t)(t->h - 1) * t->sh +
                          (int64_t)(t->w - 1) * t->sw) * es;
    *lo = (uintptr_t)t->data;
    *hi = (uintptr_t)t->data + (uintptr_t)last + (uintptr_t)es;
}

// bytes spanned by one (h, w) plane of t
int64_t wz_plane_extent(const weno_tensor_t* t)
{
    const int64_t es = wz_esize(t->dtype);
    return ((int64_t)(t->h - 1) * t->sh + (int64_t)(t->w - 1) * t->sw) * es + es;
}

bool wz_overlap(const weno_tensor_t* a, const weno_tensor_t* b)
{
    uintptr_t alo, ahi, blo, bhi;
    wz_byte_range(a, &alo, &ahi);
    wz_byte_range(b, &blo, &bhi);
    return alo < bhi && blo < ahi;
}

int wz_check_params(const weno_params_t* p)
{
    if (!p) return WENO_EINVAL;
    if (!(p->beta >= 0.0f) || !std::isfinite(p->beta) || p->beta > 64.0f) return WENO_EINVAL;
    if (!(p->k_eps >= 0.0f) || !std::isfinite(p->k_eps)) return WENO_EINVAL;
    if (!(p->h > 0.0f) || !std::isfinite(p->h)) return WENO_EINVAL;
    if (!std::isfinite(p->nbw)) return WENO_EINVAL;
    if (p->boundary != WENO_BOUNDARY_CLAMP && p->boundary != WENO_BOUNDARY_EXTERNAL) return WENO_EINVAL;
    const double eps = (double)p->k_eps * (double)p->h * (double)p->h;
    // The kernels weigh with alpha = t^-beta for a scaled t = c (eps + D) on the
    // [0,1] scale (c = 1/4 in the doubling, 3/13 in its adjoint, 1 in the
    // resampler), and sum four of them: keep 4 ((3/13) eps)^-beta below 2^126
    // so that the sum stays finite in FP32 where every indicator vanishes.
    if (p->beta > 0.0f && (eps <= 0.0 || std::log2(eps * (3.0 / 13.0)) * (double)p->beta < -124.0))
        return WENO_EINVAL;
    return WENO_OK;
}

double wz_nbw(const weno_params_t* p) { return p->nbw < 0.0f ? (double)p->h * (double)p->h / 8.0 : (double)p->nbw; }

FwdParams wz_fwd_params(const weno_params_t* p, int in_u8, int out_u8)
{
    const double w = wz_nbw(p);
    const double vs = in_u8 ? 255.0 : 1.0;  // kernel value scale relative to [0,1]
    const double eps = (double)p->k_eps * (double)p->h * (double)p->h * vs * vs;
    FwdParams P;
    // with beta = 0 the weights are t^0 = 1 whatever the indicator, and eps
    // (which may then be 0) only has to keep t away from 0 for log2
    P.eps_hat = p->beta == 0.0f ? 1.0f : (float)(eps * (3.0 / 13.0) / (1.0 + 4.0 * w));
    P.eps_q = p->beta == 0.0f ? 1.0f : (float)(eps / (4.0 * (1.0 + 4.0 * w)));
    P.w = (float)w;
    P.beta = p->beta;
    const double os = out_u8 ? 255.0 : 1.0;
    P.out_scale = (float)(os / vs);
    return P;
}

int wz_beta_mode(float beta)
{
    if (beta == 2.0f) return 2;
    if (beta == 1.0f) return 1;
    return kBetaGeneral;
}

// Fill a FwdJob for src -> dst (shapes already validated).
// The readable source region of src for a boundary mode: src itself, or
// (WENO_BOUNDARY_EXTERNAL) rows -4 .. h+4 and columns -4 .. w+4 around it.
// Returns WENO_EINVAL if that region's start address would wrap.
int wz_source_region(const weno_tensor_t* src, int boundary, weno_tensor_t* region)
{
    *region = *src;
    if (boundary != WENO_BOUNDARY_EXTERNAL) return WENO_OK;
    const int64_t back = (4 * src->sh + 4 * src->sw) * wz_esize(src->dtype);
    if ((uintptr_t)src->data < (uintptr_t)back) return WENO_EINVAL;
    region->data = (void*)((uintptr_t)src->data - (uintptr_t)back);
    region->h = src->h + 9;
    region->w = src->w + 9;
    return WENO_OK;
}

// I/O mode of a doubling.  A lane's outputs are stored together where the
// columns are contiguous.  Float rows are 4-byte aligned, which is all a vector
// store needs (a pointer that is not takes element stores); packed bytes go out
// as one word at any alignment, which this architecture allows buffer stores.
static int io_mode(const weno_tensor_t* src, const weno_tensor_t* dst)
{
    const bool in_u8 = src->dtype == WENO_U8, out_u8 = dst->dtype == WENO_U8;
    const bool rows_ok = dst->sw == 1 && (out_u8 || (uintptr_t)dst->data % 4 == 0);
    if (out_u8) return in_u8 ? (rows_ok ? kIoU8 : kIoU8S) : (rows_ok ? kIoF32U8 : kIoF32U8S);
    return in_u8 ? (rows_ok ? kIoU8F32 : kIoU8F32S) : (rows_ok ? kIoF32 : kIoF32S);
}

// tail_rows > 0 (two columns only): the last strip column is walked by
// one-column strips of tail_rows rows (zoom2x_kernel)
FwdJob wz_make_job(const weno_tensor_t* src, const weno_tensor_t* dst, int cols, int rows_per_strip, int boundary,
                   int tail_rows)
{
    FwdJob jb;
    const int64_t ei = wz_esize(src->dtype), eo = wz_esize(dst->dtype);
    jb.src = (const uint8_t*)src->data;
    jb.dst = (uint8_t*)dst->data;
    jb.H = src->h;
    jb.W = src->w;
    jb.C = src->c;
    jb.planes = src->n * src->c;
    jb.s_n = src->sn * ei;
    jb.s_c = src->sc * ei;
    jb.s_h = src->sh * ei;
    jb.s_w = src->sw * ei;
    jb.d_n = dst->sn * eo;
    jb.d_c = dst->sc * eo;
    jb.d_h = dst->sh * eo;
    jb.d_w = dst->sw * eo;
    jb.in_u8 = src->dtype == WENO_U8;
    jb.out_u8 = dst->dtype == WENO_U8;
    const int own = cols == 1 ? strip_own<1>() : strip_own<2>();
    jb.rows = rows_per_strip;
    jb.strips_x = (src->w + own - 1) / own;
    jb.strips_y = (src->h + rows_per_strip - 1) / rows_per_strip;
    jb.tail_rows = 0;
    jb.tail_bands = 0;
    if (cols == 2 && tail_rows > 0 && jb.strips_x >= 2 && src->w - (jb.strips_x - 1) * own <= strip_own<1>()) {
        jb.strips_x -= 1;
        jb.tail_rows = tail_rows;
        jb.tail_bands = (src->h + tail_rows - 1) / tail_rows;
    }
    jb.share = planes_share_lines(jb.C, jb.s_c, jb.s_h) || planes_share_lines(jb.C, jb.d_c, jb.d_h);
    jb.io = io_mode(src, dst);
    jb.dst_extent = (uint32_t)wz_plane_extent(dst);
    weno_tensor_t region;
    wz_source_region(src, boundary, &region);   // validated by the caller
    jb.src = (const uint8_t*)region.data;
    jb.src_extent = (uint32_t)wz_plane_extent(&region);
    jb.src_shift = boundary == WENO_BOUNDARY_EXTERNAL ? 4 : 0;
    jb.src_h = region.h;
    jb.src_w = region.w;
    return jb;
}

// Checks of a doubling's source region beyond wz_check_pair: with caller
// ghost samples, the extended region must span less than 2^31 bytes per
// plane and must not overlap dst.
int wz_check_region(const weno_tensor_t* src, const weno_tensor_t* dst, int boundary)
{
    if (boundary != WENO_BOUNDARY_EXTERNAL) return WENO_OK;
    weno_tensor_t region;
    if (wz_source_region(src, boundary, &region) != WENO_OK) return WENO_EINVAL;
    if (wz_plane_extent(&region) >= (1ll << 31)) return WENO_EINVAL;
    if (wz_overlap(&region, dst)) return WENO_EOVERLAP;
    return WENO_OK;
}

// shape rules of one doubling
int wz_check_pair(const weno_tensor_t* src, const weno_tensor_t* dst, int factor)
{
    int rc = wz_check_tensor(src);
    if (rc) return rc;
    rc = wz_check_tensor(dst);
    if (rc) return rc;
    if (dst->n != src->n || dst->c != src->c) return WENO_EINVAL;
    if ((int64_t)dst->h != (int64_t)src->h * factor || (int64_t)dst->w != (int64_t)src->w * factor) return WENO_EINVAL;
    if ((int64_t)src->n * src->c > 65535) return WENO_EINVAL;
    // buffer offsets are 32-bit: every plane must span less than 2^31 bytes
    if (wz_plane_extent(src) >= (1ll << 31) || wz_plane_extent(dst) >= (1ll << 31)) return WENO_EINVAL;
    if (wz_overlap(src, dst)) return WENO_EOVERLAP;
    return WENO_OK;
}

// compute units of the current device, cached per device
int wz_device_cus()
{
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int v = cache[dev].load();
    if (v == 0) {
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
        cache[dev].store(v);
    }
    return v;
}

// Automatic launch configuration from a cost model of the strip walk.  Four
// strips (waves) make a workgroup, which runs on one compute unit, one wave
// per SIMD.  A launch whose busiest compute unit runs m workgroups takes about
//   m x (rows + 4) x R(cols, m)  microseconds,
// where rows + 4 are the iterations of one wave plus the fixed cost of
// starting it (its launch and the pipeline fill) and R(cols, m) the time of
// one iteration of one of m waves sharing a SIMD (a compute unit holds three
// two-column or five one-column workgroups at once: up to that, one paced
// round; beyond it, several rounds).  m counts workgroups, not waves: one
// compute unit given one workgroup more than the rest holds up the launch.
// R is fitted (least squares on the log of the time) to 511 timed launches
// on MI355X: 20 shapes from 1x64x64 to 3x2160x3840 and 48x512x512, both
// column counts, the three shortest strips of each m = 1..8.  Candidates
// are, for each column count and m = 1..8, the shortest strips that put at
// most m workgroups on a compute unit; the cheapest wins.  On those shapes
// the pick is within 6.2 % of the best measured launch (1080p RGB: two
// columns, 27-row strips).
static double iteration_cost(int cols, int64_t m)
{
    static const double one[8] = {0.421, 0.348, 0.319, 0.309, 0.302, 0.313, 0.308, 0.306};
    static const double two[8] = {0.708, 0.589, 0.557, 0.581, 0.571, 0.563, 0.562, 0.578};
    return (cols == 1 ? one : two)[m < 8 ? m - 1 : 7];
}
constexpr int kStartCost = 4;

// Tail strips: when the columns left of the last two-column strip fit one
// one-column strip, that strip column can be walked in one-column strips
// (half the work per row) with bands kTailStretch / 4 times as tall, so that
// each walks about as long as a two-column strip (a one-column iteration
// costs ~0.59 of a two-column one in the fit); the launch then numbers its
// waves across the planes.  48x512x512: four two-column strips and 40
// columns per band, 80.1 -> 71.9 predicted.  They serve every I/O mode: planes
// with spread columns gain as much (48x512x512 uint8 98.5 -> 71.8 us, float32
// 217 -> 194; 3x512x512 uint8 15.2 -> 9.8).
constexpr int kTailStretch = 7;

// spread_bytes: a destination of bytes with spread columns, whose two-column
// kernels store eight elements a row: an iteration costs ~1.09 of the table's,
// with tail strips too.  On 18 shapes from 3x64x64 to 3x4320x7680 to uint8 HWC
// and to every second column, the pick with the factor is never slower than
// without and up to 18 % faster (4x700x1000 float32 to uint8 HWC 21.5 us against
// 26.0, 3x768x1024 18.5 and 20.8, 3x1500x954 30.1 and 32.8); on 43 shapes whose
// pick it changes from tail strips, 14 % faster to 5 % slower, 4 % faster on
// average (4x480x640 12.6 and 14.2, 48x600x591 107 and 102).  Rows of packed
// bytes cost what the table says; a batch's unpaced strips cost more
// (batched_config).
void wz_auto_config(int64_t planes, int H, int W, bool share, bool spread_bytes, int* rows, int* cols, int* tail_rows)
{
    const int64_t cus = wz_device_cus();
    double best = 0.0;
    int best_rows = 8, best_cols = 2, best_tail = 0;
    for (int c = 2; c >= 1; --c) {
        const int own = c == 1 ? strip_own<1>() : strip_own<2>();
        const int64_t strips_x = (W + own - 1) / own;
        for (int64_t m = 1; m <= 8; ++m) {
            // the most bands whose workgroups (planes x ceil(strips / 4), padded
            // as the launch pads them) fit m per compute unit
            int64_t per_plane = m * cus / planes;
            if (share) per_plane = per_plane / kXcds * kXcds;
            int64_t bands = kWavesPerBlock * per_plane / strips_x;
            if (bands < 1) bands = 1;
            int r = (int)((H + bands - 1) / bands);
            r = r < 4 ? 4 : (r > 4096 ? 4096 : r);
            const int64_t blocks = planes * wz_grid_x(strips_x * ((H + r - 1) / r), share);
            const int64_t mm = (blocks + cus - 1) / cus;
            const double cost =
                (double)mm * (r + kStartCost) * iteration_cost(c, mm) * (spread_bytes && c == 2 ? 1.09 : 1.0);
            if (best == 0.0 || cost < best) {
                best = cost;
                best_rows = r;
                best_cols = c;
                best_tail = 0;
            }
        }
    }
    // two-column strips with a one-column tail strip column (planar only)
    const int64_t sx = (W + strip_own<2>() - 1) / strip_own<2>();
    if (!share && sx >= 2 && W - (sx - 1) * strip_own<2>() <= strip_own<1>()) {
        const int64_t s2 = sx - 1;
        for (int64_t m = 1; m <= 8; ++m) {
            // waves per plane: s2 x bands + tail bands (~ bands x 4 / kTailStretch)
            const int64_t per_plane = kWavesPerBlock * m * cus / planes;
            int64_t bands = per_plane * kTailStretch / (s2 * kTailStretch + 4);
            if (bands < 1) bands = 1;
            int r = (int)((H + bands - 1) / bands);
            r = r < 4 ? 4 : (r > 4096 ? 4096 : r);
            int rt = r * kTailStretch / 4;
            rt = rt > H ? H : rt;
            const int64_t waves = planes * (s2 * ((H + r - 1) / r) + (H + rt - 1) / rt);
            const int64_t blocks = (waves + kWavesPerBlock - 1) / kWavesPerBlock;
            const int64_t mm = (blocks + cus - 1) / cus;
            const double cost = (double)mm * (r + kStartCost) * iteration_cost(2, mm) * (spread_bytes ? 1.09 : 1.0);
            if (cost < best) {
                best = cost;
                best_rows = r;
                best_cols = 2;
                best_tail = rt;
            }
        }
    }
    *rows = best_rows;
    *cols = best_cols;
    *tail_rows = best_tail;
}

// launch shape of one doubling: the caller's (weno_set_launch_config, never
// with tail strips) or the cost model's
void wz_config_for(const weno_tensor_t* src, const weno_tensor_t* dst, int* rows, int* cols, int* tail_rows)
{
    *rows = g_rows_per_strip.load();
    *cols = g_cols_per_lane.load();
    *tail_rows = 0;
    const bool share = planes_share_lines(src->c, src->sc, src->sh) || planes_share_lines(dst->c, dst->sc, dst->sh);
    if (*rows == 0 || *cols == 0)
        wz_auto_config((int64_t)src->n * src->c, src->h, src->w, share, dst->dtype == WENO_U8 && dst->sw != 1, rows,
                       cols, tail_rows);
    // taller strips where a set height would need more workgroups than a launch
    // may have (a column of 2^29 samples in 4-row strips: 2^25)
    if ((int64_t)src->h * src->w * src->c <= 4 * kMaxGridX || *tail_rows > 0) return;
    const int own = *cols == 1 ? strip_own<1>() : strip_own<2>();
    const int64_t strips_x = (src->w + own - 1) / own;
    while (*rows < 4096 &&
           wz_grid_blocks(strips_x * ((src->h + *rows - 1) / *rows), share) * (share ? src->c : 1) > kMaxGridX)
        *rows *= 2;
}

// the launchers of each I/O mode (weno_zoom.hip)
static const ZoomLauncher kZoomLaunchers[kIoModes] = {
    zoom_launcher<0>(), zoom_launcher<1>(), zoom_launcher<2>(), zoom_launcher<3>(),
    zoom_launcher<4>(), zoom_launcher<5>(), zoom_launcher<6>(), zoom_launcher<7>(),
};

int wz_launch_fwd(const weno_tensor_t* src, const weno_tensor_t* dst, const weno_params_t* p, hipStream_t st,
                  int rows, int cols, int tail_rows)
{
    const FwdJob jb = wz_make_job(src, dst, cols, rows, p->boundary, tail_rows);
    const FwdParams P = wz_fwd_params(p, jb.in_u8, jb.out_u8);
    const int bm = wz_beta_mode(p->beta);
    const hipError_t e = kZoomLaunchers[jb.io].single(jb, P, bm, cols, rows, st);
    if (e != hipSuccess) return wz_hip_error(e, "zoom2x_kernel launch");
    return WENO_OK;
}

extern "C" int weno_query_launch_config(const weno_tensor_t* src, const weno_tensor_t* dst, int32_t* rows_per_strip,
                                        int32_t* cols_per_lane, int32_t* tail_rows)
{
    int rc = wz_check_tensor(src);
    if (rc) return rc;
    if (dst) {
        rc = wz_check_tensor(dst);
        if (rc) return rc;
        if (dst->n != src->n || dst->c != src->c || (int64_t)dst->h != 2ll * src->h || (int64_t)dst->w != 2ll * src->w)
            return WENO_EINVAL;
    }
    int rows, cols, tail;
    wz_config_for(src, dst ? dst : src, &rows, &cols, &tail);
    if (rows_per_strip) *rows_per_strip = rows;
    if (cols_per_lane) *cols_per_lane = cols;
    if (tail_rows) *tail_rows = tail;
    return WENO_OK;
}

// --------------------------------------------------------------------------
// single doubling
// --------------------------------------------------------------------------
extern "C" int weno_zoom2x(const weno_tensor_t* src, const weno_tensor_t* dst, const weno_params_t* p,
                           void* hip_stream)
{
    int rc = wz_check_pair(src, dst, 2);
    if (rc) return rc;
    rc = wz_check_params(p);
    if (rc) return rc;
    rc = wz_check_region(src, dst, p->boundary);
    if (rc) return rc;
    int rows, cols, tail;
    wz_config_for(src, dst, &rows, &cols, &tail);
    return wz_launch_fwd(src, dst, p, (hipStream_t)hip_stream, rows, cols, tail);
}

// --------------------------------------------------------------------------
// batched
// --------------------------------------------------------------------------
extern "C" size_t weno_zoom2x_batched_workspace(int32_t count)
{
    if (count < 1) return 0;
    return batch_table_bytes(count);
}

// argument rules of a batched call (host only, nothing is touched on the device)
static int batched_check(const weno_tensor_t* srcs, const weno_tensor_t* dsts, int32_t count, const weno_params_t* p)
{
    if (!srcs || !dsts || count < 1) return WENO_EINVAL;
    int rc = wz_check_params(p);
    if (rc) return rc;
    for (int i = 0; i < count; ++i) {
        rc = wz_check_pair(&srcs[i], &dsts[i], 2);
        if (rc) return rc;
        rc = wz_check_region(&srcs[i], &dsts[i], p->boundary);
        if (rc) return rc;
    }
    // no output may overlap any input or another output: sweep all byte
    // ranges by start address, remembering the furthest end of each kind
    {
        struct Iv { uintptr_t lo, hi; bool out; };
        std::vector<Iv> iv(2 * (size_t)count);
        for (int i = 0; i < count; ++i) {
            weno_tensor_t region;   // what the kernel reads of image i
            wz_source_region(&srcs[i], p->boundary, &region);
            wz_byte_range(&region, &iv[2 * i].lo, &iv[2 * i].hi);
            iv[2 * i].out = false;
            wz_byte_range(&dsts[i], &iv[2 * i + 1].lo, &iv[2 * i + 1].hi);
            iv[2 * i + 1].out = true;
        }
        std::sort(iv.begin(), iv.end(), [](const Iv& a, const Iv& b) { return a.lo < b.lo; });
        uintptr_t end_in = 0, end_out = 0;
        for (const Iv& v : iv) {
            if (v.lo < end_out || (v.out && v.lo < end_in)) return WENO_EOVERLAP;
            if (v.out) end_out = std::max(end_out, v.hi); else end_in = std::max(end_in, v.hi);
        }
    }
    return WENO_OK;
}

// waves of 16-row one-column strips that six rounds of a batched launch hold
static int64_t batched_six_rounds() { return 6 * 16 * (int64_t)wz_device_cus(); }
static int64_t short_strips(const weno_tensor_t* t)
{
    return (int64_t)t->n * t->c * ((t->w + strip_own<1>() - 1) / strip_own<1>()) * ((t->h + 15) / 16);
}

// I/O modes of a batch's images.  Each mode is a launch, and the launches follow
// each other, each with its own start and its last waves running alone.  Where
// images of one pair of types go to contiguous and to spread columns, all take
// the spread mode, which stores any columns: half planar, half HWC, uint8, 8
// images of 128 to 512 squared 23.2 -> 17.2 us, 128 of 64 to 512 squared 160 ->
// 146, 64 of 256 to 1024 squared 381 -> 360; images of all eight modes, 8 57 ->
// 39, 64 135 -> 107.  Float rows lose more by it, and do so up to six rounds of
// waves only: 24 images of 85 to 415 squared 47 -> 39, 128 images (6.5 rounds)
// 190 -> 185, 64 of 256 to 1024 squared (17 rounds) 484 -> 503.
static std::vector<int> batched_modes(const weno_tensor_t* srcs, const weno_tensor_t* dsts, int32_t count)
{
    std::vector<int> io(count);
    bool present[kIoModes] = {};
    int64_t strips[kIoModes] = {};   // of both modes of a pair of types, at its contiguous one
    for (int i = 0; i < count; ++i) {
        io[i] = io_mode(&srcs[i], &dsts[i]);
        present[io[i]] = true;
        strips[io[i] & ~2] += short_strips(&srcs[i]);
    }
    for (int& m : io)
        if (present[m | 2] && (io_out_u8(m) || strips[m & ~2] <= batched_six_rounds())) m |= 2;
    return io;
}

// Strip shape of a batch from the cost model of a single launch
// (iteration_cost): a compute unit's waves share its strips out one by one, so
// it takes the rounds of its busiest wave, about 0.4 of a round more than the
// mean, at the rate of the waves that share a SIMD.  Two-column strips of bytes
// cost more per iteration than the model's float rows (x 1.17), as do those of
// floats from or to interleaved planes.  Interleaved float destinations take
// short one-column strips: the planes of a strip drift apart as they go down,
// and with them the parts of the lines that an L2 should put together (256
// float32 HWC images of 64 to 512 squared: 16 rows 566 us, 64 rows 720, two
// columns 633 and 796; 512 uint8 HWC to float32 HWC of 32 to 1024 squared 1145
// and, in 24 rows, 1264).  They decide where they hold an eighth of the pixels
// (a quarter among uint8 HWC images: 128 images 158 us, in 32 rows 166); one
// among 511 uint8 HWC images does not (16 rows 873 us, 96 rows 820).
// A batch with a float destination and an interleaved end takes such strips
// too while they are no more than six rounds of waves: its planes are walked
// side by side, and short strips leave fewer waves waiting at the end (uint8
// HWC to planar float32, 16 rows against the model's: 24 images 37 and 42 us,
// 64 images 69 and 72, 128 images, 6.5 rounds, 158 and 151, 256 images 267 and
// 257).  On batches of 8 to
// 512 images, all types, the pick is within 16 % of the best of 14 shapes, for
// most within 5 (24 uint8 HWC images of 85 to 415 squared 40-45 us, 512 of 32 to
// 1024 squared 2353; 32-row two-column strips, the choice before, 49 and 2424).
static void batched_config(const weno_tensor_t* srcs, const weno_tensor_t* dsts, const std::vector<int>& modes,
                           int32_t count, int* rows, int* cols)
{
    const int64_t cus = wz_device_cus();
    bool floats_shared = false;
    int64_t px = 0, px_spread = 0;     // pixels: all, and those of interleaved float destinations
    int64_t strips16 = 0;
    for (int i = 0; i < count; ++i) {
        const bool share = planes_share_lines(srcs[i].c, srcs[i].sc, srcs[i].sh) ||
                           planes_share_lines(dsts[i].c, dsts[i].sc, dsts[i].sh);
        floats_shared = floats_shared || (dsts[i].dtype == WENO_F32 && share);
        const int64_t planes = (int64_t)srcs[i].n * srcs[i].c, image = planes * srcs[i].h * srcs[i].w;
        px += image;
        if (dsts[i].dtype == WENO_F32 && planes_share_lines(dsts[i].c, dsts[i].sc, dsts[i].sh)) px_spread += image;
        strips16 += short_strips(&srcs[i]);
    }
    const bool spread = 8 * px_spread >= px || (floats_shared && strips16 <= batched_six_rounds());
    double best = 0.0;
    for (int c = 2; c >= 1; --c) {
        if (spread && c == 2) continue;
        const int own = c == 1 ? strip_own<1>() : strip_own<2>();
        const int64_t resident = c == 1 ? 4 : 3;   // waves per SIMD (zoom2x_batched_kernel)
        for (int r : {8, 16, 24, 32, 48, 64, 96}) {
            if (spread && r > 16) break;
            struct Launch {
                int64_t strips, iterations, units[17];   // units by their planes
                int longest;
            } launches[kIoModes] = {};
            for (int i = 0; i < count; ++i) {
                const bool share = planes_share_lines(srcs[i].c, srcs[i].sc, srcs[i].sh) ||
                                   planes_share_lines(dsts[i].c, dsts[i].sc, dsts[i].sh);
                Launch& l = launches[modes[i]];
                const int64_t places = (int64_t)srcs[i].n * ((srcs[i].w + own - 1) / own), walks = places * srcs[i].c;
                const int64_t bands = (srcs[i].h + r - 1) / r;
                l.strips += walks * bands;
                l.units[wz_unit_planes(srcs[i].c, share)] +=
                    places * bands * (share ? wz_unit_groups(srcs[i].c, true) : srcs[i].c);
                l.iterations += walks * (srcs[i].h + kStartCost * bands);
                l.longest = std::max(l.longest, (int)((srcs[i].h + bands - 1) / bands));
            }
            double cost = 0.0;   // the launches follow each other
            for (int io = 0; io < kIoModes; ++io) {
                const Launch& l = launches[io];
                if (l.strips == 0) continue;
                int64_t per_cu = 0;   // strips of the busiest compute unit
                for (int planes = 1; planes <= 16; ++planes) per_cu += (l.units[planes] + cus - 1) / cus * planes;
                const int64_t m = std::min(resident, (per_cu + 3) / 4);   // waves per SIMD
                const double rounds = (double)per_cu / (double)std::min(per_cu, 4 * resident);
                double each = l.longest + kStartCost;
                if (rounds > 1.0) each = std::max(each, (rounds + 0.4) * (double)l.iterations / (double)l.strips);
                cost += (double)m * each * iteration_cost(c, m) *
                        (c == 2 && (io_out_u8(io) || floats_shared) ? 1.17 : 1.0);
            }
            if (best == 0.0 || cost < best) {
                best = cost;
                *rows = r;
                *cols = c;
            }
        }
    }
}

// Host memory that runs out while a plan is made is an error of the call: no
// exception leaves a C entry.
template <typename F>
static int guarded(F&& call)
{
    try {
        return call();
    } catch (const std::bad_alloc&) {
        return wz_hip_error(hipErrorOutOfMemory, "host memory of a batch plan");
    }
}

static int make_plan(const weno_tensor_t* srcs, const weno_tensor_t* dsts, int32_t count, const weno_params_t* p,
                     void* d_workspace, size_t ws_bytes, void* hip_stream, weno_batch_plan_t* plan)
{
    if (!srcs || !dsts || !plan || count < 1 || !d_workspace) return WENO_EINVAL;
    int rc = wz_check_params(p);
    if (rc) return rc;
    if ((uintptr_t)d_workspace % 256 != 0) return WENO_EINVAL;
    if (ws_bytes < batch_table_bytes(count)) return WENO_ENOSPC;
    rc = batched_check(srcs, dsts, count, p);
    if (rc) return rc;
    int rows = g_rows_per_strip.load(), cols = g_cols_per_lane.load();
    const std::vector<int> modes_of = batched_modes(srcs, dsts, count);
    if (rows == 0 || cols == 0) batched_config(srcs, dsts, modes_of, count, &rows, &cols);
    // by I/O mode (each has a launch of its own), then most planes per unit (one
    // run of units after another, zoom2x_batched_kernel), then largest images first
    std::vector<FwdJob> made(count);
    std::vector<int> order(count);
    for (int i = 0; i < count; ++i) {
        // bands of nearly equal height, `rows` at most
        const int bands = (srcs[i].h + rows - 1) / rows;
        made[i] = wz_make_job(&srcs[i], &dsts[i], cols, (srcs[i].h + bands - 1) / bands, p->boundary, 0);
        made[i].io = modes_of[i];
        order[i] = i;
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        const FwdJob &A = made[a], &B = made[b];
        if (A.io != B.io) return A.io < B.io;
        const int ua = wz_unit_planes(A.C, A.share), ub = wz_unit_planes(B.C, B.share);
        if (ua != ub) return ua > ub;
        return (int64_t)A.H * A.W * A.planes > (int64_t)B.H * B.W * B.planes;
    });
    std::vector<uint8_t> host(batch_table_bytes(count), 0);
    FwdJob* jobs = (FwdJob*)(host.data() + batch_jobs_offset(count));
    int64_t* prefix = (int64_t*)(host.data() + batch_prefix_offset(count));
    FwdParams* prm = (FwdParams*)(host.data() + batch_params_offset(count));
    BatchRun* runs = (BatchRun*)(host.data() + batch_runs_offset());
    int64_t total = 0, modes = 0, items = 0;
    for (int io = 0; io < kIoModes; ++io) runs[io] = {0, 0, 0, 0, 1, -1};   // modes without images: empty runs
    BatchRun* run = nullptr;   // the run of image k - 1
    int more = kIoModes;       // entries of runs
    for (int k = 0; k < count; ++k) {
        const FwdJob& jb = jobs[k] = made[order[k]];
        prm[k] = wz_fwd_params(p, jb.in_u8, jb.out_u8);
        const int together = wz_unit_planes(jb.C, jb.share);
        const bool new_mode = !((modes >> jb.io) & 1);
        if (new_mode || run->planes != together) {
            BatchRun* const begun = &runs[new_mode ? jb.io : more];
            if (!new_mode) run->next = more++;
            run = begun;
            run->first = total;
            run->image = k;
            run->planes = together;
            run->next = -1;
        }
        modes |= 1ll << jb.io;
        prefix[k] = total;
        const int64_t strips = (int64_t)jb.strips_x * jb.strips_y;
        total += strips * (jb.share ? jb.planes / jb.C * wz_unit_groups(jb.C, true) : jb.planes);
        items += strips * jb.planes;
        run->image_end = k + 1;
        run->end = total;
    }
    prefix[count] = total;
    hipStream_t st = (hipStream_t)hip_stream;
    hipError_t e = hipMemcpyAsync(d_workspace, host.data(), host.size(), hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return wz_hip_error(e, "batch table copy");
    e = hipStreamSynchronize(st);  // the host table is freed on return
    if (e != hipSuccess) return wz_hip_error(e, "batch table copy");
    plan->d_workspace = d_workspace;
    plan->ws_bytes = ws_bytes;
    plan->total_items = items;
    plan->count = count;
    plan->rows_per_strip = rows;
    plan->cols_per_lane = cols;
    plan->beta_mode = wz_beta_mode(p->beta);
    plan->reserved = modes;
    return WENO_OK;
}

extern "C" int weno_zoom2x_batched_plan(const weno_tensor_t* srcs, const weno_tensor_t* dsts, int32_t count,
                                        const weno_params_t* p, void* d_workspace, size_t ws_bytes,
                                        void* hip_stream, weno_batch_plan_t* plan)
{
    return guarded([&] { return make_plan(srcs, dsts, count, p, d_workspace, ws_bytes, hip_stream, plan); });
}

extern "C" int weno_zoom2x_batched_run(const weno_batch_plan_t* plan, void* hip_stream)
{
    if (!plan || !plan->d_workspace || plan->count < 1 || plan->total_items < 1) return WENO_EINVAL;
    if (plan->cols_per_lane != 1 && plan->cols_per_lane != 2) return WENO_EINVAL;
    if (plan->reserved < 1 || plan->reserved >= (1ll << kIoModes)) return WENO_EINVAL;   // the set of modes to launch
    hipStream_t st = (hipStream_t)hip_stream;
    // one launch per I/O mode of the plan, nearly always one in all
    for (int io = 0; io < kIoModes; ++io) {
        if (!((plan->reserved >> io) & 1)) continue;
        const hipError_t e = kZoomLaunchers[io].batched(plan, st);
        if (e != hipSuccess) return wz_hip_error(e, "zoom2x_batched_kernel launch");
    }
    return WENO_OK;
}

extern "C" int weno_zoom2x_batched(const weno_tensor_t* srcs, const weno_tensor_t* dsts, int32_t count,
                                   const weno_params_t* p, void* d_workspace, size_t ws_bytes, void* hip_stream)
{
    weno_batch_plan_t plan;
    int rc = weno_zoom2x_batched_plan(srcs, dsts, count, p, d_workspace, ws_bytes, hip_stream, &plan);
    if (rc) return rc;
    return weno_zoom2x_batched_run(&plan, hip_stream);
}

// --------------------------------------------------------------------------
// batched, without a caller workspace
// --------------------------------------------------------------------------
// The image table of weno_zoom2x_batched_noalloc lives in this
// file-scope device array (one copy per GPU, alive until the process ends).
// In host code its name is only a stand-in for the symbol: the device
// address comes from hipGetSymbolAddress, once per device, and only that
// address is ever handed to a copy or a kernel.
constexpr size_t kNoAllocScratchBytes = batch_table_bytes(WENO_NOALLOC_MAX_IMAGES);
static __device__ __align__(256) uint8_t scratch[kNoAllocScratchBytes];

static std::mutex g_scratch_mu;
static void* g_scratch_ptr[64];  // device address of `scratch` per device, set on first use

static int noalloc_scratch(void** out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return wz_hip_error(e, "hipGetDevice");
    if (dev < 0 || dev >= 64) return WENO_EINVAL;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));  // the current device's copy
        if (e != hipSuccess) return wz_hip_error(e, "hipGetSymbolAddress(scratch)");
        if (!ptr || (uintptr_t)ptr % 256 != 0) return wz_hip_error(hipErrorInvalidSymbol, "scratch address");
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return WENO_OK;
}

extern "C" int weno_zoom2x_batched_noalloc(const weno_tensor_t* srcs, const weno_tensor_t* dsts, int32_t count,
                                           const weno_params_t* p, void* hip_stream)
{
    if (!srcs || !dsts || count < 1) return WENO_EINVAL;
    if (count > WENO_NOALLOC_MAX_IMAGES) return WENO_ENOSPC;
    int rc = guarded([&] { return batched_check(srcs, dsts, count, p); });
    if (rc) return rc;
    void* ws = nullptr;
    rc = noalloc_scratch(&ws);
    if (rc) return rc;
    // the plan validates everything before it writes the table into the
    // scratch (one host-to-device copy, then a wait on the stream)
    weno_batch_plan_t plan;
    rc = weno_zoom2x_batched_plan(srcs, dsts, count, p, ws, kNoAllocScratchBytes, hip_stream, &plan);
    if (rc) return rc;
    return weno_zoom2x_batched_run(&plan, hip_stream);
}

// --------------------------------------------------------------------------
// cascade of doublings
// --------------------------------------------------------------------------
// row pitch (floats) of the float intermediates: a multiple of 4, rows on 16
// bytes.  The stores need 4-byte alignment only, and any pitch measures the same
// (3x1079x1919 doubled twice: 175-178 us at pitches of 0..3 modulo 4).
static int64_t cascade_pitch(int64_t w) { return (w + 3) / 4 * 4; }

static void cascade_level_shape(const weno_tensor_t* src, int lvl, int64_t* h, int64_t* w)
{
    *h = (int64_t)src->h << lvl;
    *w = (int64_t)src->w << lvl;
}

extern "C" size_t weno_zoom2x_cascade_workspace(const weno_tensor_t* src, int32_t levels)
{
    if (wz_check_tensor(src) != WENO_OK || levels < 1 || levels > 8) return 0;
    size_t total = 0;
    for (int l = 1; l < levels; ++l) {
        int64_t h, w;
        cascade_level_shape(src, l, &h, &w);
        const size_t bytes = (size_t)src->n * src->c * h * cascade_pitch(w) * 4;
        total += (bytes + 255) / 256 * 256;
    }
    return total == 0 ? 256 : total;
}

extern "C" int weno_zoom2x_cascade(const weno_tensor_t* src, const weno_tensor_t* dst, int32_t levels,
                                   const weno_params_t* p, void* d_workspace, size_t ws_bytes, void* hip_stream)
{
    if (levels < 1 || levels > 8) return WENO_EINVAL;
    int rc = wz_check_tensor(src);
    if (rc) return rc;
    rc = wz_check_tensor(dst);
    if (rc) return rc;
    rc = wz_check_params(p);
    if (rc) return rc;
    // intermediate levels have no caller ghost samples
    if (p->boundary != WENO_BOUNDARY_CLAMP) return WENO_EINVAL;
    if (dst->n != src->n || dst->c != src->c || (int64_t)dst->h != ((int64_t)src->h << levels) ||
        (int64_t)dst->w != ((int64_t)src->w << levels))
        return WENO_EINVAL;
    if (wz_overlap(src, dst)) return WENO_EOVERLAP;
    if (levels > 1) {
        if (!d_workspace || (uintptr_t)d_workspace % 256 != 0) return WENO_EINVAL;
        if (ws_bytes < weno_zoom2x_cascade_workspace(src, levels)) return WENO_ENOSPC;
    }
    weno_tensor_t cur = *src;
    size_t off = 0;
    weno_params_t lp = *p;
    const double w0 = wz_nbw(p);
    for (int l = 0; l < levels; ++l) {
        weno_tensor_t out;
        if (l == levels - 1) {
            out = *dst;
        } else {
            int64_t h, w;
            cascade_level_shape(src, l + 1, &h, &w);
            out.data = (uint8_t*)d_workspace + off;
            out.dtype = WENO_F32;
            out.n = src->n;
            out.c = src->c;
            out.h = (int32_t)h;
            out.w = (int32_t)w;
            out.sw = 1;
            out.sh = cascade_pitch(w);
            out.sc = h * out.sh;
            out.sn = (int64_t)src->c * out.sc;
            const size_t bytes = (size_t)src->n * src->c * h * out.sh * 4;
            off += (bytes + 255) / 256 * 256;
            if (wz_overlap(&out, dst) || wz_overlap(&out, src)) return WENO_EOVERLAP;
        }
        rc = wz_check_pair(&cur, &out, 2);
        if (rc) return rc;
        // level l works on spacing h / 2^l; an explicit neighbour weight scales with h^2
        const double scale = std::ldexp(1.0, -l);
        lp.h = (float)(p->h * scale);
        lp.nbw = (float)(w0 * scale * scale);
        int rows, cols;
        int tail;
        wz_config_for(&cur, &out, &rows, &cols, &tail);
        rc = wz_launch_fwd(&cur, &out, &lp, (hipStream_t)hip_stream, rows, cols, tail);
        if (rc) return rc;
        cur = out;
    }
    return WENO_OK;
}
