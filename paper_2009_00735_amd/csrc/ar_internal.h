// Internal declarations shared by the HIP translation units of libaraullo.
#pragma once

#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>

#include <algorithm>
#include <map>
#include <memory>
#include <string>
#include <vector>

#include "araullo.h"

namespace ar {

// Record a thread-local error message and return `s`.
ar_status fail(ar_status s, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

#define AR_HIP(call)                                                                   \
    do {                                                                               \
        hipError_t e_ = (call);                                                        \
        if (e_ != hipSuccess)                                                          \
            return ::ar::fail(AR_EDEVICE, "%s failed: %s", #call, hipGetErrorString(e_)); \
    } while (0)

#define AR_TRY(expr)                                                                   \
    do {                                                                               \
        ar_status s_ = (expr);                                                         \
        if (s_ != AR_OK) return s_;                                                    \
    } while (0)

#define AR_CHECK(cond, ...)                                                            \
    do {                                                                               \
        if (!(cond)) return ::ar::fail(AR_EINVAL, __VA_ARGS__);                        \
    } while (0)

// Grow-only device buffer.  Growing frees the old allocation (hipFree waits
// for outstanding work on the device).
struct DeviceBuffer {
    void *ptr = nullptr;
    size_t bytes = 0;
    ~DeviceBuffer();
    ar_status reserve(size_t n);
    template <class T> T *as() const { return static_cast<T *>(ptr); }
};

// Eq. (1) constants, computed once in FP64 and rounded to FP32.
struct BinConsts {
    float shift;   // (float)(R + dR)
    float scale;   // (float)(nbins / (2R + 2dR))
};
BinConsts bin_consts(float radius, int nbins);

constexpr int kMaxWindows = 16;
struct WindowSet {
    int n;
    int kmin, kmax;          // union of all windows
    int rows;                // 1: n <= 4, kmax - kmin < 64 and every window at most 16 bins wide;
                             // 2: the same within 32 bins (two lanes per bin in the last FFT stage)
    int lo[kMaxWindows];
    int hi[kMaxWindows];
};
ar_status make_windows(const int32_t *windows, int32_t n_win, int32_t nbins, WindowSet *ws);

bool valid_nbins(int32_t nbins);
int log2i(int32_t x);

}  // namespace ar

struct ar_context {
    int device = 0;
    int cu_count = 0;
    int lds_per_block = 0;
    // gather workspace
    ar::DeviceBuffer g_keys, g_slot, g_vals, g_counts32, g_cell_start, g_sorted, g_counts, g_rows, g_temp, g_offsets;
    // host memory that kernels write sizes the host waits for into (kHostBytes), and its device address
    void *host = nullptr, *host_dev = nullptr;
    // gathered CSR used by the position-taking signature entry points
    ar::DeviceBuffer s_rel;
    // one channel's images in the typed-signature entry point
    ar::DeviceBuffer s_typed;
    // correlation tile: per-wave 32x32 MFMA tiles (wtm x wtn) and K step; used
    // when set by ar_index_set_tile, else chosen per candidate count
    int corr_waves = 8, corr_wtm = 4, corr_wtn = 2, corr_bk = 32;
    bool corr_tile_set = false;
    // indexing workspace
    ar::DeviceBuffer i_bf16, i_inv, i_cand_idx, i_cand_score, i_merge_idx;
    // sparse indexing workspace
    ar::DeviceBuffer sp_half, sp_inv, sp_cand_s, sp_cand_i, sp_merge;
    // refinement workspace
    ar::DeviceBuffer r_partials, r_state, r_dirs;
    // nearest-node candidate lists of the last mesh (count [6 G^2], lists [6 G^2][cap])
    ar::DeviceBuffer m_cells;
    // twiddle tables exp(-2 pi i j / nbins), j < nbins, per nbins
    std::map<int, std::unique_ptr<ar::DeviceBuffer>> twiddles;
    ar_status twiddle_table(int nbins, const float2 **out);
    ~ar_context();
};

struct ar_library {
    ar_context *ctx = nullptr;
    int device = 0;               // the context may be destroyed before the library
    const float *ref = nullptr;   // caller-owned FP32 raw images [n_lib][K]
    int64_t n_lib = 0;
    int32_t n_win = 0, n_dir = 0;
    int64_t K = 0;                // n_win * n_dir
    int64_t Kp = 0;               // padded to a multiple of the GEMM K tile
    int64_t n_pad = 0;            // n_lib padded to a multiple of the GEMM N tile
    ar::DeviceBuffer bf16;        // [n_pad][Kp] bf16, normalised
    ar::DeviceBuffer norm2;       // [n_pad] float, |bf16 row|^2 (pad rows: +inf)
    ar::DeviceBuffer inv_max;     // [n_lib][n_win] float, 1/max (0 for a zero image)
    ar::DeviceBuffer quats;       // [n_lib][4] double (w, x, y, z), if prepared with orientations
    ar::DeviceBuffer phase;       // [n_lib] int32, if prepared with orientations
    bool has_orientations = false;
};

namespace ar {
// internal entry points used across translation units
ar_status gather_csr(ar_context *ctx, const float *positions, const int32_t *types, int64_t n_atoms,
                     const float *centres, int64_t n_roi, float radius, uint64_t type_mask, int64_t *offsets,
                     float *rel, int64_t cap, int64_t *total, hipStream_t stream);
// The rows of one gather: ROI r at rel[offsets[stride r] .. offsets[stride r +
// 1]), and the largest ROI (or a bound of it).
struct GatheredRois {
    const float *rel;
    const int64_t *offsets;
    int stride;
    int64_t big;
};
// A reference to a callable (const GatheredRois &, int mask) -> ar_status.
struct RoiUse {
    void *self;
    ar_status (*call)(void *, const GatheredRois &, int);
    template <class F>
    RoiUse(F &f) : self(&f), call([](void *p, const GatheredRois &g, int c) { return (*static_cast<F *>(p))(g, c); })
    {
    }
    ar_status operator()(const GatheredRois &g, int c) const { return call(self, g, c); }
};
// Gather once per type mask into the context's buffers, the atoms sorted once
// for all of them, and hand each gather to `use`, which queues the work that
// reads it.  counts: device int32 [n_roi][n_masks] or NULL, out.  want_big:
// `big` must be the largest ROI, not a bound (may wait for it).  The rows'
// order within a ROI is unspecified.
ar_status gather_rois(ar_context *ctx, const float *positions, const int32_t *types, int64_t n_atoms,
                      const float *centres, int64_t n_roi, float radius, const uint64_t *type_masks, int n_masks,
                      int32_t *counts, bool want_big, hipStream_t stream,
                      RoiUse use);
constexpr size_t kHostBytes = 256;
// A grid holds fewer than 2^32 work items along x; a larger one is not refused
// but wraps around and leaves rows unwritten.  launch(r0, count) for the n rows
// in as many parts as that needs, `threads` work items per row.
template <class F> ar_status by_rows(int64_t n, int64_t threads, F &&launch)
{
    const int64_t most = std::max<int64_t>((int64_t)UINT32_MAX / threads, 1);
    for (int64_t r0 = 0; r0 < n; r0 += most) {
        launch(r0, (unsigned)std::min(most, n - r0));
        AR_HIP(hipGetLastError());
    }
    return AR_OK;
}
struct MeshCells;
// cube-map nearest-node candidate lists of `dirs` in ctx->m_cells (mesh.hip)
ar_status build_mesh_cells(ar_context *ctx, const float *dirs, int n_dir, hipStream_t stream, MeshCells &mc);
// looks up, once per device, the device address of the fixed workspace of
// ar_sf_score_grad_noalloc (refine.hip); `device` must be current
ar_status scratch_setup(int device);
}
