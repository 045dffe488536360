// ROI query: atoms within radius R of each ROI centre, as a CSR of relative
// coordinates (Sec. 2.1: spherical ROIs scan the dataset; supplement, cost
// model: one neighbour query per ROI before the projections).
//
// GPU design: a uniform cell grid (cell edge R/2) over the box spanned by the
// ROI centres +- R; atoms are bucketed by cell with a counting sort (per-cell
// counts by atomics whose return value is the atom's slot in its cell, an
// exclusive scan for the cell starts, a scatter, then each cell's atoms ranked
// by their index, so the result is the stable sort by cell id; many atoms are
// counted and placed in LDS by runs of cells instead).  Rows of cells
// are contiguous in the sorted array, so each row is one coalesced range.  A
// ROI is served by one workgroup: its wavefronts take the rows its ball
// reaches in turn, each row cut to the ball's chord (with slack against FP32
// rounding of the cell index), once to count and once to write; the row counts
// of the first pass give every row its place in the second.
// Membership is decided exactly as the paper's single-precision test:
// fmaf(dz,dz,fmaf(dy,dy,dx*dx)) <= (float)(R*R).
//
// Measured on a tip of 2.8e6 atoms and 8000 ROIs (R = 2 nm): 0.34-0.37 ms per
// call, 0.48 with the sort by global atomics, and 0.97 where one wavefront per ROI
// walked its bounding cube, a second atomic pass scattered and one thread per
// cell sorted; 300 ROIs in 1.2e5 atoms 0.09 ms, 0.37.  Bound: the two passes
// over the ROIs' rows (0.17 ms), then the sort's passes over its records.
#include <math.h>

#include <algorithm>

#include "ar_internal.h"
#include "scan_device.h"

namespace ar {
namespace {

struct Grid {
    float ox, oy, oz, inv_h;
    int nx, ny, nz;
    float reach;   // R in cell edges
};

__global__ __launch_bounds__(1024) void k_centre_bbox(const float *__restrict__ c, int64_t n,
                                                      float *__restrict__ out)
{
    __shared__ float red[6][1024];
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x)
        for (int a = 0; a < 3; ++a) {
            float v = c[3 * i + a];
            lo[a] = fminf(lo[a], v);
            hi[a] = fmaxf(hi[a], v);
        }
    for (int a = 0; a < 3; ++a) {
        red[a][threadIdx.x] = lo[a];
        red[3 + a][threadIdx.x] = hi[a];
    }
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int a = 0; a < 3; ++a) {
                red[a][threadIdx.x] = fminf(red[a][threadIdx.x], red[a][threadIdx.x + s]);
                red[3 + a][threadIdx.x] = fmaxf(red[3 + a][threadIdx.x], red[3 + a][threadIdx.x + s]);
            }
        __syncthreads();
    }
    if (threadIdx.x < 6) out[threadIdx.x] = red[threadIdx.x][0];
}

__device__ __forceinline__ int cell_coord(float p, float o, float inv_h) { return (int)floorf((p - o) * inv_h); }

// Cell id of an atom, ncells outside the grid.
__device__ __forceinline__ uint32_t cell_key(float x, float y, float z, const Grid &g)
{
    const int cx = cell_coord(x, g.ox, g.inv_h), cy = cell_coord(y, g.oy, g.inv_h), cz = cell_coord(z, g.oz, g.inv_h);
    const bool in = cx >= 0 && cx < g.nx && cy >= 0 && cy < g.ny && cz >= 0 && cz < g.nz;
    return in ? (uint32_t)(cx + g.nx * (cy + g.ny * cz)) : (uint32_t)g.nx * g.ny * g.nz;
}

__global__ __launch_bounds__(256) void k_fill_i32(int32_t *__restrict__ a, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = 0;
}

// Cell id of every atom (ncells for atoms outside the grid), its slot in the
// cell (in arrival order) and the count of every cell.
__global__ __launch_bounds__(256) void k_cell_keys(const float *__restrict__ pos, int64_t n, Grid g,
                                                   uint32_t *__restrict__ keys, int32_t *__restrict__ slot,
                                                   int32_t *__restrict__ counts)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t ncells = (uint32_t)g.nx * g.ny * g.nz;
    const uint32_t key = cell_key(pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], g);
    keys[i] = key;
    if (key < ncells) slot[i] = atomicAdd(&counts[key], 1);
}

// Each atom inside the grid, with its cell, to its slot.
__global__ __launch_bounds__(256) void k_cell_scatter(const uint32_t *__restrict__ keys, const int32_t *__restrict__ slot,
                                                      int64_t n, uint32_t ncells,
                                                      const int32_t *__restrict__ cell_start, int2 *__restrict__ idx)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t key = keys[i];
    if (key >= ncells) return;
    idx[cell_start[key] + slot[i]] = make_int2((int32_t)i, (int32_t)key);
}

// Sorted positions: one thread per slot finds its atom's rank in the cell by
// the atom index (cells hold tens of atoms at the R/2 cell edge of a specimen,
// and the threads of a cell read the same entries together).  That is c reads
// for every one of a crowded cell's c atoms, spread over the chip: putting such
// a cell in order by one thread's insertion takes c^2 / 4 moves in a row when
// the arrivals are mixed, minutes at 1.3e5 atoms.  The 4th component carries
// the atom type's bits (0 when the call has no types).
__global__ __launch_bounds__(256) void k_sorted_pos(const float *__restrict__ pos, const int32_t *__restrict__ types,
                                                    const int2 *__restrict__ idx,
                                                    const int32_t *__restrict__ cell_start, uint32_t ncells,
                                                    float4 *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= cell_start[ncells]) return;
    const int2 v = idx[i];
    const int64_t a = v.x;
    const float4 p = make_float4(pos[3 * a], pos[3 * a + 1], pos[3 * a + 2], __int_as_float(types ? types[a] : 0));
    const int s0 = cell_start[v.y], s1 = cell_start[v.y + 1];
    int rank = 0;
#pragma unroll 8
    for (int j = s0; j < s1; ++j) rank += idx[j].x < v.x ? 1 : 0;
    out[s0 + rank] = p;
}

// ---------------------------------------------- the sort by parts
// The same sorted positions for many atoms: the cells fall into at most kParts
// runs of 2^shift, the atoms go to their run (counts per workgroup, one scan,
// a scatter of position and index), and a workgroup per run counts and
// places its atoms by cell in LDS.  Bound: the passes over the 16-byte
// records; the form above is bound by its global atomics, 7e9 a second
// (k_cell_keys), and the random reads of k_sorted_pos.
constexpr int kParts = 512;
constexpr int kPartAtoms = 4096;                 // atoms per workgroup of the first two passes
constexpr int kPartCells = 8192;                 // cells of a run, in LDS
constexpr int64_t kPartMin = 262144;             // atoms

// SCATTER == false: counts[part][workgroup]; true: the records to their places.
template <bool SCATTER>
__global__ __launch_bounds__(kParts) void k_part(const float *__restrict__ pos, int64_t n, Grid g, int shift,
                                                 int n_parts, int32_t *__restrict__ counts,
                                                 const int32_t *__restrict__ start, float4 *__restrict__ rec)
{
    __shared__ int h[kParts];
    const int tid = threadIdx.x;
    const int64_t at = (int64_t)tid * gridDim.x + blockIdx.x;
    h[tid] = SCATTER && tid < n_parts ? start[at] : 0;
    __syncthreads();
    const uint32_t ncells = (uint32_t)g.nx * g.ny * g.nz;
#pragma unroll
    for (int k = 0; k < kPartAtoms / kParts; ++k) {
        const int64_t i = (int64_t)blockIdx.x * kPartAtoms + k * kParts + tid;
        if (i >= n) break;
        const float x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2];
        const uint32_t key = cell_key(x, y, z, g);
        if (key >= ncells) continue;
        const int slot = atomicAdd(&h[key >> shift], 1);
        if (SCATTER) rec[slot] = make_float4(x, y, z, __int_as_float((int)i));
    }
    if (SCATTER) return;
    __syncthreads();
    if (tid < n_parts) counts[at] = h[tid];
}

// One run of cells: cell starts, and its records by cell (in any order).
__global__ __launch_bounds__(1024) void k_part_cells(const float4 *__restrict__ rec, const int32_t *__restrict__ start,
                                                     int n_wg, int n_parts, Grid g, int shift,
                                                     int32_t *__restrict__ cell_start, float4 *__restrict__ out)
{
    __shared__ int cnt[kPartCells];
    __shared__ int wave_sum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t ncells = (uint32_t)g.nx * g.ny * g.nz, k0 = blockIdx.x << shift;
    const int nc = (int)min(1u << shift, ncells - k0);
    const int base = start[(int64_t)blockIdx.x * n_wg], end = start[((int64_t)blockIdx.x + 1) * n_wg];
    for (int c = tid; c < kPartCells; c += 1024) cnt[c] = 0;
    __syncthreads();
    for (int i = base + tid; i < end; i += 1024) {
        const float4 a = rec[i];
        atomicAdd(&cnt[min(cell_key(a.x, a.y, a.z, g) - k0, (uint32_t)nc - 1)], 1);
    }
    __syncthreads();
    constexpr int PER = kPartCells / 1024;
    int v[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) sum += v[k] = cnt[tid * PER + k];
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int run = base + incl - sum;
    for (int w = 0; w < wave; ++w) run += wave_sum[w];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int c = tid * PER + k;
        cnt[c] = run;
        if (c < nc) cell_start[k0 + c] = run;
        run += v[k];
    }
    if (tid == 0 && (int)blockIdx.x == n_parts - 1) cell_start[ncells] = end;
    __syncthreads();
    for (int i = base + tid; i < end; i += 1024) {
        const float4 a = rec[i];
        out[atomicAdd(&cnt[min(cell_key(a.x, a.y, a.z, g) - k0, (uint32_t)nc - 1)], 1)] = a;
    }
}

// Records to their rank in the cell by atom index, as k_sorted_pos.
__global__ __launch_bounds__(256) void k_part_rank(const float4 *__restrict__ rec, const int32_t *__restrict__ types,
                                                   const int32_t *__restrict__ cell_start, Grid g,
                                                   float4 *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t ncells = (uint32_t)g.nx * g.ny * g.nz;
    if (i >= cell_start[ncells]) return;
    const float4 p = rec[i];
    const uint32_t key = min(cell_key(p.x, p.y, p.z, g), ncells - 1);
    const int a = __float_as_int(p.w), s0 = cell_start[key], s1 = cell_start[key + 1];
    int rank = 0;
#pragma unroll 8
    for (int j = s0; j < s1; ++j) rank += __float_as_int(rec[j].w) < a ? 1 : 0;
    out[s0 + rank] = make_float4(p.x, p.y, p.z, __int_as_float(types ? types[a] : 0));
}

// Atom type t is accepted iff 0 <= t < 64 and bit t of the mask is set.
__device__ __forceinline__ bool type_accepted(float w, uint64_t mask)
{
    const uint32_t t = (uint32_t)__float_as_int(w);
    return t < 64u && ((mask >> t) & 1ull);
}

// One workgroup per ROI.  FILL == false: counts per row (rows[r][kRows]) and
// per ROI; FILL == true: the rows of rel.  Rows are taken in turn by the
// wavefronts; a ROI with more rows than kRows (only grids so long that FP32
// rounding needs several cells of slack), and every ROI of a call of more than
// kRowRois (whose ROIs alone fill the chip, and whose row counts would be
// large), is walked by one wavefront in order.
constexpr int kRows = 64;
constexpr int64_t kRowRois = 262144;
template <bool FILL>
__global__ __launch_bounds__(1024) void k_roi_query(const float4 *__restrict__ spos,
                                                    const int32_t *__restrict__ cell_start, Grid g, float reach,
                                                    const float *__restrict__ centres, float R2, uint64_t type_mask,
                                                    int32_t *__restrict__ rows, int32_t *__restrict__ counts,
                                                    int32_t *__restrict__ count_out, int64_t count_stride,
                                                    const int64_t *__restrict__ offsets, float4 *__restrict__ rel)
{
    __shared__ int64_t wave_count[16];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int64_t r = blockIdx.x;
    const float cx = centres[3 * r], cy = centres[3 * r + 1], cz = centres[3 * r + 2];
    // the ball in cell units; a computed cell index is off by at most 2.4e-7
    // of its size from the exact one, the slack is four times that and 1/20
    const float tx = (cx - g.ox) * g.inv_h, ty = (cy - g.oy) * g.inv_h, tz = (cz - g.oz) * g.inv_h;
    const bool finite = fabsf(tx) < INFINITY && fabsf(ty) < INFINITY && fabsf(tz) < INFINITY;
    const int y0 = (int)fmaxf(floorf(ty - reach), 0.f), y1 = (int)fminf(floorf(ty + reach), (float)(g.ny - 1));
    const int z0 = (int)fmaxf(floorf(tz - reach), 0.f), z1 = (int)fminf(floorf(tz + reach), (float)(g.nz - 1));
    const int nyr = y1 - y0 + 1;
    const int64_t nrow = finite && nyr > 0 && z1 >= z0 ? (int64_t)nyr * (z1 - z0 + 1) : 0;
    const bool in_turn = rows != nullptr && nrow <= kRows;
    int64_t before = 0;   // FILL: rows of this lane's row index start here
    if (FILL) {
        int c = in_turn && lane < nrow ? rows[r * kRows + lane] : 0;
        int incl = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(incl, o);
            if (lane >= o) incl += v;
        }
        before = offsets[r] + incl - c;
    }
    const uint64_t lt_mask = (1ull << lane) - 1;
    int64_t count = 0;
    if (in_turn || wave == 0)
        for (int64_t i = in_turn ? wave : 0; i < nrow; i += in_turn ? waves : 1) {
            const int z = z0 + (int)(i / nyr), y = y0 + (int)(i % nyr);
            // distance of the row from the centre, and the chord left of the ball
            const float dy = fmaxf(0.f, fmaxf((float)y - ty, ty - (float)(y + 1)));
            const float dz = fmaxf(0.f, fmaxf((float)z - tz, tz - (float)(z + 1)));
            const float c2 = reach * reach - dy * dy - dz * dz;
            int row_count = 0;
            if (c2 >= 0.f) {
                const float c = sqrtf(c2);
                const int x0 = (int)fmaxf(floorf(tx - c - (reach - g.reach)), 0.f);
                const int x1 = (int)fminf(floorf(tx + c + (reach - g.reach)), (float)(g.nx - 1));
                if (x1 >= x0) {
                    const int row = g.nx * (y + g.ny * z);
                    const int a0 = cell_start[row + x0], a1 = cell_start[row + x1 + 1];
                    int64_t base = 0;
                    if (FILL) base = in_turn ? __shfl(before, (int)i) : offsets[r] + count;
                    for (int i0 = a0; i0 < a1; i0 += 64) {
                        const int k = i0 + lane;
                        bool in = false;
                        float dx = 0.f, ddy = 0.f, ddz = 0.f;
                        if (k < a1) {
                            const float4 p = spos[k];
                            dx = p.x - cx;
                            ddy = p.y - cy;
                            ddz = p.z - cz;
                            in = fmaf(ddz, ddz, fmaf(ddy, ddy, dx * dx)) <= R2 && type_accepted(p.w, type_mask);
                        }
                        const uint64_t m = __ballot(in);
                        if (FILL && in)
                            rel[base + row_count + __popcll(m & lt_mask)] = make_float4(dx, ddy, ddz, 0.f);
                        row_count += __popcll(m);
                    }
                }
            }
            if (!FILL && in_turn && lane == 0) rows[r * kRows + i] = row_count;
            count += row_count;
        }
    if (!FILL) {
        if (lane == 0) wave_count[wave] = count;
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t total = 0;
            for (int w = 0; w < waves; ++w) total += wave_count[w];
            counts[r] = (int32_t)total;
            if (count_out) count_out[r * count_stride] = (int32_t)total;
        }
    }
}

// Offsets (exclusive scan of the counts), their total and the largest count,
// by one workgroup: a call of up to kOffsetsMax ROIs needs one launch for all
// three, and the host reads the last two from its own memory.
constexpr int64_t kOffsetsMax = 65536;
struct Summary {
    int64_t total, big;
};
__global__ __launch_bounds__(1024) void k_roi_offsets(const int32_t *__restrict__ counts, int64_t n, bool scan,
                                                      int64_t *__restrict__ offsets, Summary *__restrict__ out)
{
    __shared__ int64_t wsum[16];
    __shared__ int wbig[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t carry = 0;
    int big = 0;
    for (int64_t c0 = 0; c0 < n; c0 += 1024) {
        const int64_t i = c0 + threadIdx.x;
        const int v = i < n ? counts[i] : 0;
        big = max(big, v);
        if (!scan) continue;
        int64_t incl = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        __syncthreads();   // the previous chunk's sums have been read
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        int64_t base = carry;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) base += wsum[w];
            carry += wsum[w];
        }
        if (i < n) offsets[i] = base + incl - v;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) big = max(big, __shfl_xor(big, o));
    if (lane == 0) wbig[wave] = big;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) big = max(big, wbig[w]);
        if (scan) offsets[n] = carry;
        out->total = offsets[n];
        out->big = big;
    }
}

// The same rows for a small specimen, without sorting it: one workgroup per
// ROI tests every atom (input order).  Row r starts at r * n; pairs[2 r] and
// pairs[2 r + 1] are its first and last + 1.
__global__ __launch_bounds__(1024) void k_roi_scan(const float *__restrict__ pos, const int32_t *__restrict__ types,
                                                   int n, const float *__restrict__ centres, float R2,
                                                   uint64_t type_mask, int64_t *__restrict__ pairs,
                                                   int32_t *__restrict__ counts, int32_t *__restrict__ count_out,
                                                   int64_t count_stride, float4 *__restrict__ rel)
{
    __shared__ int wsum[2][16];   // two sets so that one barrier per 1024 atoms is enough
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t r = blockIdx.x;
    const float cx = centres[3 * r], cy = centres[3 * r + 1], cz = centres[3 * r + 2];
    float4 *out = rel + r * n;
    int base = 0;
    for (int c0 = 0, set = 0; c0 < n; c0 += 1024, set ^= 1) {
        const int i = c0 + threadIdx.x;
        bool in = false;
        float dx = 0.f, dy = 0.f, dz = 0.f;
        if (i < n) {
            dx = pos[3 * i] - cx;
            dy = pos[3 * i + 1] - cy;
            dz = pos[3 * i + 2] - cz;
            in = fmaf(dz, dz, fmaf(dy, dy, dx * dx)) <= R2 &&
                 type_accepted(__int_as_float(types ? types[i] : 0), type_mask);
        }
        const uint64_t m = __ballot(in);
        if (lane == 0) wsum[set][wave] = __popcll(m);
        __syncthreads();
        int at = base;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) at += wsum[set][w];
            base += wsum[set][w];
        }
        if (in) out[at + __popcll(m & ((1ull << lane) - 1))] = make_float4(dx, dy, dz, 0.f);
    }
    if (threadIdx.x == 0) {
        pairs[2 * r] = r * n;
        pairs[2 * r + 1] = r * n + base;
        counts[r] = base;
        if (count_out) count_out[r * count_stride] = base;
    }
}

}  // namespace

static ar_status check_gather(ar_context *ctx, const float *positions, int64_t n_atoms, const float *centres,
                              int64_t n_roi, float radius)
{
    AR_CHECK(ctx != nullptr, "context is NULL");
    AR_CHECK(n_atoms >= 0 && n_atoms < (int64_t)INT32_MAX, "n_atoms must be in [0, 2^31-1)");
    AR_CHECK(n_roi >= 1, "n_roi must be >= 1");
    AR_CHECK(radius > 0.f && isfinite(radius), "radius must be finite and > 0");
    AR_CHECK(centres != nullptr, "centres must not be NULL");
    AR_CHECK(n_atoms == 0 || positions, "positions is NULL");
    AR_CHECK(n_roi < (int64_t)INT32_MAX, "too many ROIs");
    AR_HIP(hipSetDevice(ctx->device));
    return AR_OK;
}

static float ball2(float radius) { return (float)((double)radius * (double)radius); }

// Bounding box of the centres, written by the kernel into host memory (waits
// for it): min x y z, max x y z, all finite.
static ar_status centres_box(ar_context *ctx, const float *centres, int64_t n_roi, float (&bb)[6], hipStream_t stream)
{
    k_centre_bbox<<<1, 1024, 0, stream>>>(centres, n_roi, static_cast<float *>(ctx->host_dev));
    AR_HIP(hipGetLastError());
    AR_HIP(hipStreamSynchronize(stream));
    for (int a = 0; a < 6; ++a) {
        bb[a] = static_cast<const float *>(ctx->host)[a];
        AR_CHECK(isfinite(bb[a]), "ROI centres must be finite");
    }
    return AR_OK;
}

// Sort the atoms into the cell grid of centres with box bb (ctx->g_sorted,
// ctx->g_cell_start).
static ar_status gather_sort(ar_context *ctx, const float *positions, const int32_t *types, int64_t n_atoms,
                             const float (&bb)[6], int64_t n_roi, float radius, Grid *grid, hipStream_t stream)
{
    // grid: cell edge R/2, grown if the box would need too many cells
    double h = 0.5 * (double)radius;
    const double pad = (double)radius + h;
    double ext[3];
    for (int a = 0; a < 3; ++a) ext[a] = (double)bb[3 + a] - (double)bb[a] + 2.0 * pad;
    for (;;) {
        double cells = 1.0;
        for (int a = 0; a < 3; ++a) cells *= floor(ext[a] / h) + 1.0;
        if (cells <= 6.4e7) break;
        h *= 1.5;
    }
    Grid g;
    g.ox = (float)((double)bb[0] - pad);
    g.oy = (float)((double)bb[1] - pad);
    g.oz = (float)((double)bb[2] - pad);
    g.inv_h = (float)(1.0 / h);
    g.nx = (int)(floor(ext[0] / h) + 1.0);
    g.ny = (int)(floor(ext[1] / h) + 1.0);
    g.nz = (int)(floor(ext[2] / h) + 1.0);
    g.reach = (float)((double)radius / h);
    *grid = g;
    const uint32_t ncells = (uint32_t)g.nx * g.ny * g.nz;

    // counting sort of the atoms by cell: counts and slots, cell starts
    // (exclusive scan), scatter, per-cell input order
    const int64_t n = n_atoms;
    AR_TRY(ctx->g_cell_start.reserve(sizeof(int32_t) * ((size_t)ncells + 1)));
    AR_TRY(ctx->g_sorted.reserve(sizeof(float4) * (n + 1)));
    // by parts from 262144 atoms on (2.8e6 atoms 0.16 ms, the form below 0.28; at 1.2e5
    // both 0.04), where a run of cells fits LDS
    if (n >= kPartMin && ncells <= (uint32_t)kParts * kPartCells) {
        int shift = 0;
        while ((ncells - 1) >> shift >= (uint32_t)kParts) ++shift;
        const int n_parts = (int)((ncells - 1) >> shift) + 1;
        const int n_wg = (int)((n + kPartAtoms - 1) / kPartAtoms);
        const int64_t n_counts = (int64_t)n_parts * n_wg;
        AR_TRY(ctx->g_slot.reserve(sizeof(int32_t) * n_counts));
        AR_TRY(ctx->g_counts32.reserve(sizeof(int32_t) * (n_counts + 1)));
        AR_TRY(ctx->g_vals.reserve(sizeof(float4) * n));
        AR_TRY(ctx->g_temp.reserve(std::max(sizeof(int32_t) * scan::tiles(n_counts), sizeof(int64_t) * scan::tiles(n_roi)) +
                                   16));
        int32_t *counts = ctx->g_slot.as<int32_t>(), *start = ctx->g_counts32.as<int32_t>();
        // the records by run lie where the sorted atoms go in the end: 32 bytes per atom in all
        float4 *rec = ctx->g_sorted.as<float4>(), *by_cell = ctx->g_vals.as<float4>();
        k_part<false><<<n_wg, kParts, 0, stream>>>(positions, n, g, shift, n_parts, counts, nullptr, nullptr);
        AR_HIP(hipGetLastError());
        AR_TRY((scan::exclusive_scan<int32_t, int32_t>(counts, n_counts, start, ctx->g_temp.as<int32_t>(), stream)));
        k_part<true><<<n_wg, kParts, 0, stream>>>(positions, n, g, shift, n_parts, nullptr, start, rec);
        AR_HIP(hipGetLastError());
        k_part_cells<<<n_parts, 1024, 0, stream>>>(rec, start, n_wg, n_parts, g, shift,
                                                   ctx->g_cell_start.as<int32_t>(), by_cell);
        AR_HIP(hipGetLastError());
        k_part_rank<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(by_cell, types, ctx->g_cell_start.as<int32_t>(), g,
                                                                     ctx->g_sorted.as<float4>());
        AR_HIP(hipGetLastError());
        return AR_OK;
    }
    AR_TRY(ctx->g_keys.reserve(sizeof(uint32_t) * (n + 1)));
    AR_TRY(ctx->g_slot.reserve(sizeof(int32_t) * (n + 1)));
    AR_TRY(ctx->g_vals.reserve(sizeof(int2) * (n + 1)));
    AR_TRY(ctx->g_counts32.reserve(sizeof(int32_t) * ((size_t)ncells + 1)));
    AR_TRY(ctx->g_temp.reserve(std::max(sizeof(int32_t) * scan::tiles(ncells), sizeof(int64_t) * scan::tiles(n_roi)) +
                               16));
    int32_t *counts = ctx->g_counts32.as<int32_t>();
    int32_t *cell_start = ctx->g_cell_start.as<int32_t>();
    const unsigned fill_blocks = (unsigned)std::min<int64_t>(((int64_t)ncells + 255) / 256, 4096);
    k_fill_i32<<<fill_blocks, 256, 0, stream>>>(counts, ncells);
    AR_HIP(hipGetLastError());
    const unsigned blocks = (unsigned)((n + 255) / 256);
    if (n > 0) {
        k_cell_keys<<<blocks, 256, 0, stream>>>(positions, n, g, ctx->g_keys.as<uint32_t>(), ctx->g_slot.as<int32_t>(),
                                                counts);
        AR_HIP(hipGetLastError());
    }
    AR_TRY((scan::exclusive_scan<int32_t, int32_t>(counts, ncells, cell_start, ctx->g_temp.as<int32_t>(), stream)));
    if (n > 0) {
        k_cell_scatter<<<blocks, 256, 0, stream>>>(ctx->g_keys.as<uint32_t>(), ctx->g_slot.as<int32_t>(), n, ncells,
                                                   cell_start, ctx->g_vals.as<int2>());
        AR_HIP(hipGetLastError());
        k_sorted_pos<<<blocks, 256, 0, stream>>>(positions, types, ctx->g_vals.as<int2>(), cell_start, ncells,
                                                 ctx->g_sorted.as<float4>());
        AR_HIP(hipGetLastError());
    }
    return AR_OK;
}

template <bool FILL>
static ar_status query(ar_context *ctx, const Grid &g, const float *centres, int64_t n_roi, float radius,
                       uint64_t type_mask, int32_t *count_out, int64_t count_stride, const int64_t *offsets, float *rel,
                       hipStream_t stream)
{
    const float reach = g.reach * (1.0f + 1e-6f) + 0.05f + 1e-6f * (float)std::max(g.nx, std::max(g.ny, g.nz));
    // 16 wavefronts per ROI where the ROIs alone would not fill the chip
    const unsigned threads = n_roi < 512 ? 1024 : n_roi <= kRowRois ? 256 : 64;
    int32_t *rows = n_roi <= kRowRois ? ctx->g_rows.as<int32_t>() : nullptr;
    return by_rows(n_roi, threads, [&](int64_t r0, unsigned n) {
        k_roi_query<FILL><<<n, threads, 0, stream>>>(
            ctx->g_sorted.as<float4>(), ctx->g_cell_start.as<int32_t>(), g, reach, centres + 3 * r0, ball2(radius),
            type_mask, rows ? rows + r0 * kRows : rows, ctx->g_counts.as<int32_t>() + r0,
            count_out ? count_out + r0 * count_stride : count_out, count_stride, offsets ? offsets + r0 : offsets,
            (float4 *)rel);
    });
}

// Offsets of every ROI's rows, their total and the largest ROI (waits for them).
static ar_status gather_count(ar_context *ctx, const Grid &g, const float *centres, int64_t n_roi, float radius,
                              uint64_t type_mask, int32_t *count_out, int64_t count_stride, int64_t *offsets,
                              int64_t *total, int64_t *big, hipStream_t stream)
{
    if (n_roi <= kRowRois) AR_TRY(ctx->g_rows.reserve(sizeof(int32_t) * kRows * n_roi));
    AR_TRY(ctx->g_counts.reserve(sizeof(int32_t) * n_roi));
    AR_TRY(query<false>(ctx, g, centres, n_roi, radius, type_mask, count_out, count_stride, nullptr, nullptr, stream));
    const bool one = n_roi <= kOffsetsMax;
    if (!one)
        AR_TRY((scan::exclusive_scan<int32_t, int64_t>(ctx->g_counts.as<int32_t>(), n_roi, offsets,
                                                       ctx->g_temp.as<int64_t>(), stream)));
    k_roi_offsets<<<1, 1024, 0, stream>>>(ctx->g_counts.as<int32_t>(), n_roi, one, offsets,
                                          static_cast<Summary *>(ctx->host_dev));
    AR_HIP(hipGetLastError());
    AR_HIP(hipStreamSynchronize(stream));
    const Summary *sum = static_cast<const Summary *>(ctx->host);
    *total = sum->total;
    *big = sum->big;
    return AR_OK;
}

ar_status gather_csr(ar_context *ctx, const float *positions, const int32_t *types, int64_t n_atoms,
                     const float *centres, int64_t n_roi, float radius, uint64_t type_mask, int64_t *offsets, float *rel,
                     int64_t cap, int64_t *total, hipStream_t stream)
{
    AR_CHECK(ctx != nullptr, "context is NULL");
    AR_CHECK(centres && offsets && total, "centres/offsets/total must not be NULL");
    AR_TRY(check_gather(ctx, positions, n_atoms, centres, n_roi, radius));
    Grid g;
    int64_t big = 0;
    float bb[6];
    AR_TRY(centres_box(ctx, centres, n_roi, bb, stream));
    AR_TRY(gather_sort(ctx, positions, types, n_atoms, bb, n_roi, radius, &g, stream));
    AR_TRY(gather_count(ctx, g, centres, n_roi, radius, type_mask, nullptr, 0, offsets, total, &big, stream));
    if (!rel) return AR_OK;
    AR_CHECK(cap >= *total, "rel capacity %lld is smaller than the %lld gathered rows", (long long)cap,
             (long long)*total);
    return query<true>(ctx, g, centres, n_roi, radius, type_mask, nullptr, 0, offsets, rel, stream);
}

// A call small enough to test every atom against every ROI: up to 4e6 tests
// and rows of storage (64 MiB), and no workgroup walks more than 32 blocks of
// 1024 atoms.  Sorting costs a dozen launches and a second wait whatever its
// size (75 us for one ROI of 1 nm); the tests take 5 to 20 us at these bounds.
// Hardly any atoms leave the ROIs: 1024 threads each have to fit one grid.
static bool small_gather(int64_t n_atoms, int64_t n_roi)
{
    return n_atoms <= 32768 && n_atoms * n_roi <= (1 << 22) && n_roi <= (int64_t)UINT32_MAX / 1024;
}

ar_status gather_rois(ar_context *ctx, const float *positions, const int32_t *types, int64_t n_atoms,
                      const float *centres, int64_t n_roi, float radius, const uint64_t *type_masks, int n_masks,
                      int32_t *counts, bool want_big, hipStream_t stream,
                      RoiUse use)
{
    AR_TRY(check_gather(ctx, positions, n_atoms, centres, n_roi, radius));
    float bb[6];
    AR_TRY(centres_box(ctx, centres, n_roi, bb, stream));
    if (small_gather(n_atoms, n_roi)) {
        AR_TRY(ctx->g_offsets.reserve(sizeof(int64_t) * 2 * n_roi));
        AR_TRY(ctx->g_counts.reserve(sizeof(int32_t) * n_roi));
        AR_TRY(ctx->s_rel.reserve(sizeof(float4) * (n_roi * n_atoms + 1)));
        for (int c = 0; c < n_masks; ++c) {
            k_roi_scan<<<(unsigned)n_roi, 1024, 0, stream>>>(positions, types, (int)n_atoms, centres, ball2(radius),
                                                             type_masks[c], ctx->g_offsets.as<int64_t>(),
                                                             ctx->g_counts.as<int32_t>(), counts ? counts + c : nullptr,
                                                             n_masks, ctx->s_rel.as<float4>());
            AR_HIP(hipGetLastError());
            int64_t big = n_atoms;
            if (want_big) {
                // offsets [n_roi] is only read for the total here, which is not used
                k_roi_offsets<<<1, 1024, 0, stream>>>(ctx->g_counts.as<int32_t>(), n_roi, false,
                                                      ctx->g_offsets.as<int64_t>(), static_cast<Summary *>(ctx->host_dev));
                AR_HIP(hipGetLastError());
                AR_HIP(hipStreamSynchronize(stream));
                big = static_cast<const Summary *>(ctx->host)->big;
            }
            AR_TRY(use(GatheredRois{ctx->s_rel.as<float>(), ctx->g_offsets.as<int64_t>(), 2, big}, c));
        }
        return AR_OK;
    }
    Grid g;
    AR_TRY(gather_sort(ctx, positions, types, n_atoms, bb, n_roi, radius, &g, stream));
    AR_TRY(ctx->g_offsets.reserve(sizeof(int64_t) * (n_roi + 1)));
    for (int c = 0; c < n_masks; ++c) {
        int64_t total = 0, big = 0;
        AR_TRY(gather_count(ctx, g, centres, n_roi, radius, type_masks[c], counts ? counts + c : nullptr, n_masks,
                            ctx->g_offsets.as<int64_t>(), &total, &big, stream));
        AR_TRY(ctx->s_rel.reserve(sizeof(float4) * (total + 1)));
        AR_TRY(query<true>(ctx, g, centres, n_roi, radius, type_masks[c], nullptr, 0, ctx->g_offsets.as<int64_t>(),
                           ctx->s_rel.as<float>(), stream));
        AR_TRY(use(GatheredRois{ctx->s_rel.as<float>(), ctx->g_offsets.as<int64_t>(), 1, big}, c));
    }
    return AR_OK;
}

}  // namespace ar

extern "C" ar_status ar_roi_gather(ar_context *ctx, const float *positions, int64_t n_atoms, const float *centres,
                                   int64_t n_roi, float radius, int64_t *offsets, float *rel, int64_t cap,
                                   int64_t *total, void *stream)
{
    return ar::gather_csr(ctx, positions, nullptr, n_atoms, centres, n_roi, radius, ~0ull, offsets, rel, cap, total,
                          (hipStream_t)stream);
}

extern "C" ar_status ar_roi_gather_typed(ar_context *ctx, const float *positions, const int32_t *types,
                                         int64_t n_atoms, const float *centres, int64_t n_roi, float radius,
                                         uint64_t type_mask, int64_t *offsets, float *rel, int64_t cap,
                                         int64_t *total, void *stream)
{
    AR_CHECK(n_atoms == 0 || types != nullptr, "types is NULL");
    return ar::gather_csr(ctx, positions, types, n_atoms, centres, n_roi, radius, type_mask, offsets, rel, cap, total,
                          (hipStream_t)stream);
}
