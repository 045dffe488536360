// Reciprocal-space signatures on a cubic grid (Sec. 2.2, FSP paragraph,
// Eq. (2); supplement, reciprocal-space cost O(N_roi N_w L_D^3)):
//   amp[r][a][b][c] = |F(k)|,  F(k) = sum_w exp(-2 pi i k . d_w),
//   k = ((a - L/2), (b - L/2), (c - L/2)) dk,  dk = 2 k_max / L.
//
// One octant of real sums.  With the cosine and sine of every axis' phase at
// k_a, k_b, k_c >= 0, the four rows cx cy, cx sy, sx cy, sx sy of a pair
// (a, b) times the two columns cz, sz of c are eight sums over the atoms,
//   S[r][z] = sum_w P_r[w] Z_z[w],
// and they give F at all eight points (+-a, +-b, +-c) (combine() below; |F|
// is even in k, so four moduli).  A quarter of the products of the complex
// GEMM over the whole grid: L^3 N_w real multiply-adds instead of 4 L^3 N_w.
// The points with an index 0 (k = -k_max, off the mirrored octant: 3 L^2 of
// L^3) are faces_item's and lines_item's.
//
// Matrix cores: each FP32 factor is split into two FP16 parts, x = hi + lo
// (22 bits), and a product of two factors is hi hi + hi lo + lo hi on
// v_mfma_f32_32x32x16_f16, exact products accumulated in FP32.  Both parts
// are rounded to nearest, so |lo| <= 2^-11 |x| and the dropped lo lo is at most
// 2^-22 of the product, of either sign.  (With hi cut toward zero it reaches
// 2^-20 and always has the product's sign, which does not average out over the
// atoms: amplitudes on average 0.77 2^-22 too small, now 0.39, with FP32
// factors 0.27; the conversions cost the same.)  Three FP16 MFMAs replace one
// FP32 product at sixteen times its rate.  The phases are formed and reduced to
// [-1/2, 1/2] turns in FP64, where an FP32 phase of up to 20 turns was most of
// the error.  Measured against 64 bits (relative 2-norm, 256 ROIs of 2016 and
// 2836 atoms, L = 64): 4.3e-7, where the FP32 matrix form with FP32 phases had
// 1.4e-6.
//
// octant_item: a workgroup of 8 wavefronts takes 16 a, 16 b and 32 c; a wavefront
// one tile of 32 pairs (2 a by 16 b).  Per 32 atoms it forms the factors once
// in LDS (X and Y in FP32, Z as FP16 fragments); each wavefront multiplies
// its rows in registers (8 atoms of one pair per lane, the A operand's
// layout), splits them (96 vector instructions) and feeds 24 MFMAs of 32
// cycles per 16 atoms.  The factors are double buffered and the two
// wavefronts of a SIMD take the two halves of a step in opposite order: one
// forms the next step's factors while the other feeds the matrix cores.
// Measured, those 256 ROIs: 1.11 ms per call against 10.5 ms for the whole
// grid as one complex GEMM on FP32 MFMA (which ran at 97 % of that unit's
// rate), and 1.9-2.1 ms for half the grid with complex products on FP16
// parts; the faces and lines as launches of their own 1.23 ms.  One ROI at
// L = 64: 0.16 ms (0.57 before), at L = 32 with 130 atoms 26 us (27).  ROIs of
// a handful of atoms are slower than they were, since a step always forms 32
// atoms' factors (64 ROIs of 1 atom at L = 64: 29 us, 16 before).  Bound: matrix cores
// 41 % of the kernel's cycles and the factor and split instructions, 39 %, which
// overlap only in part.
#include <math.h>

#include "ar_internal.h"

namespace ar {
namespace fsp {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kSlice = 16;             // atoms of one MFMA
constexpr int kAtoms = 2 * kSlice;     // atoms per step
constexpr int kChunk = kThreads;       // atoms staged in LDS at a time (a multiple of kAtoms)

// cos and sin of `turns`, reduced in FP64.
__device__ __forceinline__ float2 unit(double turns)
{
    const float f = (float)(turns - rint(turns));
    return make_float2(__builtin_amdgcn_cosf(f), __builtin_amdgcn_sinf(f));
}

// Two values split in FP16, x = hi + lo: the high parts rounded to nearest in
// one instruction, each remainder x - hi formed and rounded in one more
// (v_fma_mixlo_f16, v_fma_mixhi_f16).  `minus` is -1, kept from the compiler:
// a plain subtraction is not fused with the two conversions.
__device__ __forceinline__ void split2(float x0, float x1, float minus, uint32_t &hi, uint32_t &lo)
{
    const f16x2 h = __builtin_convertvector((f32x2{x0, x1}), f16x2);
    f16x2 l;
    l.x = (_Float16)fmaf((float)h.x, minus, x0);
    l.y = (_Float16)fmaf((float)h.y, minus, x1);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, l);
}

template <int N> struct Words {
    uint32_t w[N];
};

// N values to FP16 parts in element order.
template <int N> __device__ __forceinline__ void split(const float (&x)[2 * N], Words<N> &hi, Words<N> &lo)
{
    float minus = -1.0f;
    asm("" : "+s"(minus));
#pragma unroll
    for (int e = 0; e < N; ++e) split2(x[2 * e], x[2 * e + 1], minus, hi.w[e], lo.w[e]);
}

__device__ __forceinline__ f16x8 frag(const Words<4> &x) { return __builtin_bit_cast(f16x8, x); }

// The rows P_r of one pair tile, FP16 parts: 0 cos cos, 1 cos sin, 2 sin cos,
// 3 sin sin of the first and second axis.
struct Rows {
    f16x8 hi[4], lo[4];
};

__device__ __forceinline__ void set_row(const float (&x)[8], f16x8 &hi, f16x8 &lo)
{
    Words<4> h, l;
    split<4>(x, h, l);
    hi = frag(h);
    lo = frag(l);
}

// S[r][z] += P_r Z_z over one slice, the small products first; z: cos hi,
// cos lo, sin hi, sin lo of the columns.
__device__ __forceinline__ void multiply_tile(const Rows &p, const f16x8 (&z)[4], f32x16 (&S)[4][2])
{
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                S[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(q == 0 ? p.lo[r] : p.hi[r], z[2 * c + (q == 1)],
                                                                 S[r][c], 0, 0, 0);
}

__device__ __forceinline__ void clear(f32x16 (&S)[4][2])
{
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) S[r][c][i] = 0.f;
}

// |F| at (a, sb b, sc c) from the eight sums of (a, b, c): with P = (cx + i sx)
// (cy + i sb sy) and Z = cz + i sc sz, F = sum P Z.
__device__ __forceinline__ float combine(const f32x16 (&S)[4][2], int i, float sb, float sc)
{
    const float re = (S[0][0][i] - sb * S[3][0][i]) - sc * (S[2][1][i] + sb * S[1][1][i]);
    const float im = (S[2][0][i] + sb * S[1][0][i]) + sc * (S[0][1][i] - sb * S[3][1][i]);
    return sqrtf(fmaf(re, re, im * im));
}

// C layout of a 32 x 32 MFMA: lane l, value i -> row 8 (i / 4) + 4 (l / 32) + i % 4, column l % 32
__device__ __forceinline__ int tile_row(int lane, int i) { return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3); }

// Factors of one step in LDS.  Fragment order: element e of lane l belongs to
// row (or column) l % 32 and atom 8 (l / 32) + e of the slice, for A and B
// alike.
struct Stage {
    f16x8 z[2][4][64];         // per slice: cos hi, cos lo, sin hi, sin lo of the columns
    float4 x[2][4][2][16];     // per slice: (cos, sin) of atoms 2 q, 2 q + 1 of half h, value a
    float4 y[2][4][2][16];     // the same of b
};

// One workgroup of the octant: item = (ROI, 16 a, 16 b, 32 c).
__device__ __forceinline__ void octant_item(const float4 *__restrict__ rel, const int64_t *__restrict__ offsets,
                                            int64_t item, int L, double dk, int per_roi, float *__restrict__ amp,
                                            Stage (&st)[2], float4 (&xs)[2 * kChunk])
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r = item / per_roi;
    int t = (int)(item - r * per_roi);
    const int half = L >> 1, nt = half / 16, ct = (half + 31) / 32;
    const int c0 = (t % ct) * 32;
    t /= ct;
    const int a0 = (t / nt) * 16, b0 = (t % nt) * 16;

    f32x16 S[4][2];
    clear(S);
    const int64_t o0 = offsets[r];
    const int nw = (int)(offsets[r + 1] - o0);

    // atoms [w0, w0 + kChunk) to LDS; the fourth component marks the atoms
    // past the end, whose column factors are zero
    auto stage = [&](int w0) {
        const int w = w0 + tid;
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
        if (w < nw) {
            a = rel[o0 + w];
            a.w = 1.f;
        }
        xs[w % (2 * kChunk)] = a;
    };
    // factors of step `step` into buffer b: per thread two atoms of one
    // column, one atom of one a and of one b
    auto form = [&](int step, int b) {
        const float4 *x = xs + (step * kAtoms) % (2 * kChunk);
        {
            const int l = tid & 63, pair = (tid >> 6) & 3, sl = tid >> 8;
            const double k = (double)(c0 + (l & 31)) * dk;
            float c[2], s[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float4 p = x[kSlice * sl + 8 * (l >> 5) + 2 * pair + e];
                const float2 f = unit(k * (double)p.z);
                c[e] = p.w != 0.f ? f.x : 0.f;
                s[e] = p.w != 0.f ? f.y : 0.f;
            }
            Words<1> hi, lo;
            split<1>(c, hi, lo);
            reinterpret_cast<uint32_t *>(&st[b].z[sl][0][l])[pair] = hi.w[0];
            reinterpret_cast<uint32_t *>(&st[b].z[sl][1][l])[pair] = lo.w[0];
            split<1>(s, hi, lo);
            reinterpret_cast<uint32_t *>(&st[b].z[sl][2][l])[pair] = hi.w[0];
            reinterpret_cast<uint32_t *>(&st[b].z[sl][3][l])[pair] = lo.w[0];
        }
        const int e = tid & 1, i = (tid >> 1) & 15, h = (tid >> 5) & 1, q = (tid >> 6) & 3, sl = tid >> 8;
        const float4 p = x[kSlice * sl + 8 * h + 2 * q + e];
        reinterpret_cast<float2 *>(&st[b].x[sl][q][h][i])[e] = unit((double)(a0 + i) * dk * (double)p.x);
        reinterpret_cast<float2 *>(&st[b].y[sl][q][h][i])[e] = unit((double)(b0 + i) * dk * (double)p.y);
    };
    const int h = lane >> 5, la = 2 * wave + ((lane >> 4) & 1), lb = lane & 15;
    auto multiply = [&](int b) {
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) {
            f16x8 z[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) z[p] = st[b].z[sl][p][lane];
            float P[4][8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 u = st[b].x[sl][q][h][la], v = st[b].y[sl][q][h][lb];
                P[0][2 * q] = u.x * v.x;
                P[1][2 * q] = u.x * v.y;
                P[2][2 * q] = u.y * v.x;
                P[3][2 * q] = u.y * v.y;
                P[0][2 * q + 1] = u.z * v.z;
                P[1][2 * q + 1] = u.z * v.w;
                P[2][2 * q + 1] = u.w * v.z;
                P[3][2 * q + 1] = u.w * v.w;
            }
            Rows p;
#pragma unroll
            for (int i = 0; i < 4; ++i) set_row(P[i], p.hi[i], p.lo[i]);
            multiply_tile(p, z, S);
        }
    };

    const int steps = (nw + kAtoms - 1) / kAtoms;
    if (steps > 0) {
        stage(0);
        __syncthreads();
        form(0, 0);
        __syncthreads();
    }
    const bool late = wave >= kWaves / 2;
    for (int s = 0; s < steps; ++s) {
        // a chunk is staged two steps before its first atom, one before its factors are formed
        if ((s + 2) * kAtoms % kChunk == 0 && s + 2 < steps) stage((s + 2) * kAtoms);
        if (!late && s + 1 < steps) form(s + 1, (s + 1) & 1);
        multiply(s & 1);
        if (late && s + 1 < steps) form(s + 1, (s + 1) & 1);
        __syncthreads();
    }

    float *out = amp + r * L * L * (int64_t)L;
    const int c = c0 + (lane & 31);
    if (c >= half) return;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = tile_row(lane, i);
        const int a = a0 + 2 * wave + (row >> 4), b = b0 + (row & 15);
#pragma unroll
        for (int sg = 0; sg < 4; ++sg) {
            const int sb = sg & 1 ? -1 : 1, sc = sg & 2 ? -1 : 1;
            // k = 0 has one sign
            if ((sb < 0 && b == 0) || (sc < 0 && c == 0)) continue;
            const float v = combine(S, i, (float)sb, (float)sc);
            out[((int64_t)(half + a) * L + half + sb * b) * L + half + sc * c] = v;
            if (a > 0) out[((int64_t)(half - a) * L + half - sb * b) * L + half - sc * c] = v;
        }
    }
}

// The points with two or three indices 0 (k = -k_max on those axes), 3 L - 2
// of them: (0, 0, c), (0, b, 0), (a, 0, 0), the corner once.  A wavefront
// takes kLine points, its lanes over the atoms.
constexpr int kLine = 4;
__device__ __forceinline__ void lines_item(const float4 *__restrict__ rel, const int64_t *__restrict__ offsets,
                                           int64_t item, int L, double dk, int items, int lane, float *__restrict__ amp)
{
    const int64_t r = item / items;
    const int p0 = (int)(item - r * items) * kLine, half = L >> 1;
    const int64_t o0 = offsets[r];
    const int nw = (int)(offsets[r + 1] - o0);
    int idx[kLine][3];
    float re[kLine], im[kLine];
#pragma unroll
    for (int u = 0; u < kLine; ++u) {
        const int p = p0 + u;   // points past the end are formed and not stored
        const int line = p < L ? 0 : p < 2 * L - 1 ? 1 : 2;
        const int j = line == 0 ? p : line == 1 ? p - L + 1 : p - 2 * L + 2;
        idx[u][0] = line == 2 ? j : 0;
        idx[u][1] = line == 1 ? j : 0;
        idx[u][2] = line == 0 ? j : 0;
        re[u] = im[u] = 0.f;
    }
    for (int w = lane; w < nw; w += 64) {
        const float4 x = rel[o0 + w];
#pragma unroll
        for (int u = 0; u < kLine; ++u) {
            const double ka = (double)(idx[u][0] - half) * dk, kb = (double)(idx[u][1] - half) * dk,
                         kc = (double)(idx[u][2] - half) * dk;
            const float2 f = unit(fma(kc, (double)x.z, fma(kb, (double)x.y, ka * (double)x.x)));
            re[u] += f.x;
            im[u] += f.y;
        }
    }
#pragma unroll
    for (int u = 0; u < kLine; ++u) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            re[u] += __shfl_xor(re[u], o);
            im[u] += __shfl_xor(im[u], o);
        }
        if (lane == 0 && p0 + u < 3 * L - 2)
            amp[((r * L + idx[u][0]) * L + idx[u][1]) * L + idx[u][2]] = sqrtf(fmaf(re[u], re[u], im[u] * im[u]));
    }
}

// The points with one index 0, in tiles: that axis fixed at -k_max, 32 rows
// of a second axis by 32 columns of a third (both >= 0, the four signs
// combined), the factors formed in registers: fixed x (rows y, columns z),
// y (x, z) and z (x, y).  One wavefront per tile.
// tiles = 3 ceil(L / 64)^2 per ROI.
__device__ __forceinline__ void faces_item(const float4 *__restrict__ rel, const int64_t *__restrict__ offsets,
                                           int64_t item, int L, double dk, int tiles, int lane, float *__restrict__ amp)
{
    const int64_t r = item / tiles;
    int t = (int)(item - r * tiles);
    const int half = L >> 1, ht = (half + 31) / 32;
    float *out = amp + r * L * L * (int64_t)L;
    const int64_t o0 = offsets[r];
    const int nw = (int)(offsets[r + 1] - o0);
    const int fixed = t / (ht * ht);          // axis at -k_max: 0 x, 1 y, 2 z
    t -= fixed * ht * ht;
    const int row0 = (t / ht) * 32, col0 = (t % ht) * 32;
    const double kf = -(double)half * dk, kr = (double)(row0 + (lane & 31)) * dk, kc = (double)(col0 + (lane & 31)) * dk;
    f32x16 S[4][2];
    clear(S);
    const int we = 8 * (lane >> 5);
    float4 next[8];   // the next slice's atoms, loaded a slice ahead
#pragma unroll
    for (int e = 0; e < 8; ++e) next[e] = nw > 0 ? rel[o0 + min(we + e, nw - 1)] : make_float4(0.f, 0.f, 0.f, 0.f);
    for (int w0 = 0; w0 < nw; w0 += kSlice) {
        float P[4][8], cz[8], sz[8];
        float4 x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            x[e] = next[e];
            next[e] = rel[o0 + min(w0 + kSlice + we + e, nw - 1)];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int w = w0 + we + e;
            const float4 p = x[e];
            const float2 f = unit(kf * (double)(fixed == 0 ? p.x : fixed == 1 ? p.y : p.z));
            const float2 g = unit(kr * (double)(fixed == 0 ? p.y : p.x));
            const float2 z = unit(kc * (double)(fixed == 2 ? p.y : p.z));
            P[0][e] = f.x * g.x;
            P[1][e] = f.x * g.y;
            P[2][e] = f.y * g.x;
            P[3][e] = f.y * g.y;
            cz[e] = w < nw ? z.x : 0.f;
            sz[e] = w < nw ? z.y : 0.f;
        }
        Rows p;
#pragma unroll
        for (int i = 0; i < 4; ++i) set_row(P[i], p.hi[i], p.lo[i]);
        f16x8 z[4];
        set_row(cz, z[0], z[1]);
        set_row(sz, z[2], z[3]);
        multiply_tile(p, z, S);
    }
    const int64_t L2 = (int64_t)L * L;
    const int64_t sr = fixed == 0 ? L : L2, sc = fixed == 2 ? L : 1;   // strides of rows and columns
    const int c = col0 + (lane & 31);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int b = row0 + tile_row(lane, i);
        if (b >= half || c >= half) continue;
#pragma unroll
        for (int sg = 0; sg < 4; ++sg) {
            const int mb = sg & 1 ? -1 : 1, mc = sg & 2 ? -1 : 1;
            if ((mb < 0 && b == 0) || (mc < 0 && c == 0)) continue;
            out[(half + mb * b) * sr + (half + mc * c) * sc] = combine(S, i, (float)mb, (float)mc);
        }
    }
}

// Work of a call: per ROI `tiles` face tiles (one per wavefront), `per`
// octant workgroups and `items` line items (one per wavefront).  One launch:
// the face tiles first, whose single wavefronts run longest, so that they
// end behind the octant's workgroups instead of after them; a small call
// pays one launch.
struct Plan {
    int64_t n_roi;
    int L, tiles, per, items;
    int64_t face_blocks, octant_blocks;
};
__global__ __launch_bounds__(kThreads) void k_fsp(const float4 *__restrict__ rel, const int64_t *__restrict__ offsets,
                                                  Plan pl, double dk, float *__restrict__ amp)
{
    __shared__ Stage st[2];
    __shared__ float4 xs[2 * kChunk];                 // chunk c in half c % 2
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t b = blockIdx.x;
    if (b < pl.face_blocks) {
        const int64_t item = b * kWaves + wave;
        if (item < pl.n_roi * pl.tiles) faces_item(rel, offsets, item, pl.L, dk, pl.tiles, lane, amp);
        return;
    }
    b -= pl.face_blocks;
    if (b < pl.octant_blocks) {
        octant_item(rel, offsets, b, pl.L, dk, pl.per, amp, st, xs);
        return;
    }
    b -= pl.octant_blocks;
    const int64_t item = b * kWaves + wave;
    if (item < pl.n_roi * pl.items) lines_item(rel, offsets, item, pl.L, dk, pl.items, lane, amp);
}

}  // namespace fsp
}  // namespace ar

extern "C" {

ar_status ar_fsp_amplitudes(ar_context *ctx, const float *rel, const int64_t *offsets, int64_t n_roi, int32_t L,
                            float k_max, float *amp, void *stream)
{
    AR_CHECK(ctx != nullptr, "context is NULL");
    AR_CHECK(rel && offsets && amp, "rel/offsets/amp must not be NULL");
    AR_CHECK(n_roi >= 1, "n_roi must be >= 1");
    AR_CHECK(L >= 32 && L <= 512 && L % 32 == 0, "L must be a multiple of 32 in [32, 512], got %d", L);
    AR_CHECK(k_max > 0.0f && isfinite(k_max), "k_max must be finite and > 0");
    AR_HIP(hipSetDevice(ctx->device));
    hipStream_t s = (hipStream_t)stream;
    const double dk = 2.0 * (double)k_max / (double)L;
    const int nt = L / 32, ht = (L / 2 + 31) / 32, kw = ar::fsp::kWaves;
    ar::fsp::Plan pl{n_roi, L, 3 * ht * ht, nt * nt * ht, (3 * L - 2 + ar::fsp::kLine - 1) / ar::fsp::kLine, 0, 0};
    AR_CHECK(n_roi < (int64_t)INT32_MAX, "too many ROIs per call (%lld)", (long long)n_roi);
    auto blocks = [&](int64_t n) {
        pl.n_roi = n;
        pl.face_blocks = (n * pl.tiles + kw - 1) / kw;
        pl.octant_blocks = n * pl.per;
        return pl.face_blocks + pl.octant_blocks + (n * pl.items + kw - 1) / kw;
    };
    AR_CHECK(blocks(n_roi) < (int64_t)INT32_MAX, "too many workgroups (%lld): index fewer ROIs per call",
             (long long)blocks(n_roi));
    return ar::by_rows(n_roi, ar::fsp::kThreads * (blocks(kw) / kw + 1), [&](int64_t r0, unsigned n) {
        const unsigned grid = (unsigned)blocks(n);
        ar::fsp::k_fsp<<<grid, ar::fsp::kThreads, 0, s>>>((const float4 *)rel, offsets + r0, pl, dk,
                                                          amp + (size_t)r0 * L * L * L);
    });
}

}  // extern "C"
