// Device building blocks of the real-space signature kernels (Sec. 2.2,
// Eq. (1); supplement "Controlled windowing of the SDMs" and "Sequential
// implementation tricks": FFT of each histogram in single precision using
// conjugate-even symmetry).  Included by signatures.hip only.
//
// This translation unit is compiled with -ffp-contract=off: the Eq. (1)
// projection must round exactly as mul, fma, fma, add, mul; every fused
// multiply-add in the FFT is written out with fmaf.
#pragma once

#include "ar_internal.h"

namespace ar {
namespace sig {

constexpr int kWave = 64;

__device__ __forceinline__ void wave_lds_sync()
{
    // LDS operations of one wavefront complete in issue order; this keeps the
    // compiler from moving LDS accesses across the point.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b)
{
    return make_float2(fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.x, b.y, a.y * b.x));
}
// acc + a * b and acc + a * conj(b)
__device__ __forceinline__ float2 cmac(float2 acc, float2 a, float2 b)
{
    return make_float2(fmaf(-a.y, b.y, fmaf(a.x, b.x, acc.x)), fmaf(a.y, b.x, fmaf(a.x, b.y, acc.y)));
}
__device__ __forceinline__ float2 cmac_conj(float2 acc, float2 a, float2 b)
{
    return make_float2(fmaf(a.y, b.y, fmaf(a.x, b.x, acc.x)), fmaf(-a.x, b.y, fmaf(a.y, b.x, acc.y)));
}
// multiply by -i
__device__ __forceinline__ float2 cmul_mi(float2 a) { return make_float2(a.y, -a.x); }

// In-register forward DFTs (exp(-2 pi i s t / R)).
__device__ __forceinline__ void dft2(float2 *v)
{
    float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}

__device__ __forceinline__ void dft4(float2 &a0, float2 &a1, float2 &a2, float2 &a3)
{
    const float2 s02 = cadd(a0, a2), d02 = csub(a0, a2);
    const float2 s13 = cadd(a1, a3), d13 = cmul_mi(csub(a1, a3));
    a0 = cadd(s02, s13);
    a2 = csub(s02, s13);
    a1 = cadd(d02, d13);
    a3 = csub(d02, d13);
}

__device__ __forceinline__ void dft4(float2 *v) { dft4(v[0], v[1], v[2], v[3]); }

__device__ __forceinline__ void dft8(float2 *v)
{
    const float h = 0.70710678118654752440f;
    float2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
    float2 o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
    dft4(e0, e1, e2, e3);
    dft4(o0, o1, o2, o3);
    // o_t *= exp(-2 pi i t / 8)
    o1 = make_float2((o1.x + o1.y) * h, (o1.y - o1.x) * h);
    o2 = cmul_mi(o2);
    o3 = make_float2((o3.y - o3.x) * h, -(o3.x + o3.y) * h);
    v[0] = cadd(e0, o0); v[4] = csub(e0, o0);
    v[1] = cadd(e1, o1); v[5] = csub(e1, o1);
    v[2] = cadd(e2, o2); v[6] = csub(e2, o2);
    v[3] = cadd(e3, o3); v[7] = csub(e3, o3);
}

template <int R> __device__ __forceinline__ void dftR(float2 *v)
{
    if constexpr (R == 8) dft8(v);
    else if constexpr (R == 4) dft4(v);
    else dft2(v);
}

// Swizzled float2 layout of the FFT buffer: element i lives at
// i ^ h(i >> 5), h(x) = (x & 7) | (((x >> 1) & 3) << 3).  Within each aligned
// block of 32 elements this is a bijection.  Reads of a pass touch 32
// consecutive elements per half-wavefront (XOR by a constant: still one
// element per bank pair); the strided writes of the first two passes land on
// 32 distinct bank pairs (low bits taken by the stride XORed with the block
// index), so no pass has LDS bank conflicts.
__device__ __forceinline__ int swz(int i)
{
    const int x = i >> 5;
    return i ^ ((x & 7) | (((x >> 1) & 3) << 3));
}

// Radix plan of the NC-point complex transform: radix-8 passes on
// sub-transform lengths NS = 1, 8, 64, ... while more than a factor 8 is
// left, then one last stage of radix NC / NS_LAST (2, 4 or 8).  Every pass
// before the last has NS <= 64, so the twiddle factor of butterfly j,
// exp(-2 pi i t (j mod NS) / (8 NS)), depends on the lane only
// (j mod NS = lane mod NS): each lane keeps those factors in registers.
template <int NC> struct FftPlan {
    static constexpr int last_ns()
    {
        int ns = 1;
        while (NC / ns > 8) ns *= 8;
        return ns;
    }
    static constexpr int NS_LAST = last_ns();
    static constexpr int R_LAST = NC / NS_LAST;
    static_assert(NS_LAST <= 512, "transform length out of range");
};

// Per-lane twiddle factors of one radix-8 pass with sub-transform length NS
// (NS = 8 or 64), taken from the NB-point table Wg[m] = exp(-2 pi i m / NB).
template <int NB, int NS> struct PassTwiddles {
    float2 w[7];
    __device__ __forceinline__ void load(const float2 *__restrict__ Wg, int lane)
    {
        constexpr int STRIDE = NB / (NS * 8);
        const int k = lane & (NS - 1);
#pragma unroll
        for (int t = 1; t < 8; ++t) w[t - 1] = Wg[(t * k * STRIDE) & (NB - 1)];
    }
};

// One in-place Stockham autosort pass of radix R on NC complex points in
// LDS, sub-transform length NS before the pass.  Butterfly j reads element
// j + t NC/R, applies twiddles exp(-2 pi i t (j mod NS)/(NS R)) (tw[t-1],
// the same for every butterfly of a lane) and writes element
// (j - j mod NS) R + j mod NS + t NS.  Every lane loads the inputs of all its
// butterflies before any write; LDS operations of a wavefront execute in
// order, so the pass can overwrite its own input.  FROM_HIST: the input is
// the int32 histogram read unswizzled as pairs (h_2n, h_2n+1) = z_n.
template <int NC, int R, int NS, bool FROM_HIST>
__device__ __forceinline__ void stockham_pass(float2 *buf, const float2 *tw, int lane)
{
    constexpr int NBF = NC / R;
    constexpr int PER = (NBF + kWave - 1) / kWave;   // butterflies per lane
    float2 v[PER][R];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int j = p * kWave + lane;
        if (NBF % kWave == 0 || j < NBF) {
#pragma unroll
            for (int t = 0; t < R; ++t) {
                if constexpr (FROM_HIST) {
                    const int2 q = reinterpret_cast<const int2 *>(buf)[j + t * NBF];
                    v[p][t] = make_float2((float)q.x, (float)q.y);
                } else {
                    v[p][t] = buf[swz(j + t * NBF)];
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int j = p * kWave + lane;
        if (NBF % kWave == 0 || j < NBF) {
            const int k = j & (NS - 1);
            if constexpr (NS > 1) {
#pragma unroll
                for (int t = 1; t < R; ++t) v[p][t] = cmul(v[p][t], tw[t - 1]);
            }
            dftR<R>(v[p]);
            const int base = (j - k) * R + k;
#pragma unroll
            for (int t = 0; t < R; ++t) buf[swz(base + t * NS)] = v[p][t];
        }
    }
}

// The last stage in full (every output), twiddles read from the global
// table; used only where the whole spectrum is written out.
template <int NB, int NC, int R, int NS>
__device__ __forceinline__ void stockham_last_full(float2 *buf, const float2 *__restrict__ Wg, int lane)
{
    constexpr int NBF = NC / R;
    constexpr int PER = (NBF + kWave - 1) / kWave;
    constexpr int STRIDE = NB / (NS * R);
    float2 v[PER][R];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int j = p * kWave + lane;
        if (NBF % kWave == 0 || j < NBF) {
#pragma unroll
            for (int t = 0; t < R; ++t) v[p][t] = buf[swz(j + t * NBF)];
        }
    }
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int j = p * kWave + lane;
        if (NBF % kWave == 0 || j < NBF) {
            const int k = j & (NS - 1);
#pragma unroll
            for (int t = 1; t < R; ++t) v[p][t] = cmul(v[p][t], Wg[(t * k * STRIDE) & (NB - 1)]);
            dftR<R>(v[p]);
            const int base = (j - k) * R + k;
#pragma unroll
            for (int t = 0; t < R; ++t) buf[swz(base + t * NS)] = v[p][t];
        }
    }
}

// All passes before the last stage.
template <int NB, int NC, int NS, bool FROM_HIST>
__device__ __forceinline__ void fft_head(float2 *buf, const PassTwiddles<NB, 8> &tw8,
                                         const PassTwiddles<NB, 64> &tw64, int lane)
{
    if constexpr (NS < FftPlan<NC>::NS_LAST) {
        const float2 *tw = NS == 8 ? tw8.w : tw64.w;
        stockham_pass<NC, 8, NS, FROM_HIST>(buf, tw, lane);
        wave_lds_sync();
        fft_head<NB, NC, NS * 8, false>(buf, tw8, tw64, lane);
    }
}

// Element index of Y_t[m] (element t NS + m) in the swizzled layout.  For
// NS = 64: t NS + m has block index 2t + (m >> 5), so the swizzle XORs m with
// (m >> 5) ^ 10 (t mod 4): one XOR per t mod 4 and the rest an immediate
// offset (mm = m ^ (m >> 5) is per lane).  For NS >= 256 the block index of
// t NS + m agrees with that of m in the swizzled bits, so the element is
// swz(m) + t NS.
template <int NS> __device__ __forceinline__ int last_index(int mm, int t)
{
    if constexpr (NS == 64) return (mm ^ (10 * (t & 3))) + 64 * t;
    else if constexpr (NS >= 256) return mm + NS * t;
    else return swz(t * NS + mm);
}
template <int NS> __device__ __forceinline__ int last_base(int m)
{
    if constexpr (NS == 64) return m ^ (m >> 5);
    else if constexpr (NS >= 256) return swz(m);
    else return m;
}

// Last stage restricted to the outputs one real-spectrum bin needs.  After
// the earlier passes the buffer holds R sub-transforms Y_t of length NS
// (element t NS + m), and the packed transform is
//   Z_k = sum_t Y_t[k mod NS] w^(t k),  w = exp(-2 pi i / NC),
// so Z_k and Z_(NC-k) (twiddles conj(w^(t k))) come from 2R reads and
// R - 1 complex multiply-adds each.  Then, with E = (Z_k + conj Z_(NC-k))/2
// and O = -i (Z_k - conj Z_(NC-k))/2, X_k = E + exp(-2 pi i k / NB) O and the
// result is |X_k|.  mm1, mm2: last_base of k mod NS and (NC - k) mod NS;
// ftw[t-1] = w^(t k), wk = exp(-2 pi i k / NB).
template <int NC>
__device__ __forceinline__ float bin_amplitude(const float2 *buf, int mm1, int mm2, const float2 *ftw, float2 wk)
{
    constexpr int NS = FftPlan<NC>::NS_LAST;
    constexpr int R = FftPlan<NC>::R_LAST;
    float2 a = buf[last_index<NS>(mm1, 0)];
    float2 b = buf[last_index<NS>(mm2, 0)];
#pragma unroll
    for (int t = 1; t < R; ++t) {
        a = cmac(a, buf[last_index<NS>(mm1, t)], ftw[t - 1]);
        b = cmac_conj(b, buf[last_index<NS>(mm2, t)], ftw[t - 1]);
    }
    // 2E = Z_k + conj Z', 2O = -i (Z_k - conj Z')
    const float2 e2 = make_float2(a.x + b.x, a.y - b.y);
    const float2 o2 = make_float2(a.y + b.y, b.x - a.x);
    const float2 x2 = cmac(e2, o2, wk);
    return 0.5f * sqrtf(fmaf(x2.x, x2.x, x2.y * x2.y));
}

// The same |X_k| with the two R-term sums on two lanes: lane l < 32 sums
// Z_k, lane l + 32 sums Z_(NC-k) (its twiddles conjugated, base mmx = that
// lane's last_base), and the partial results are exchanged across the
// half-wavefronts.  Valid in lanes 0..31, for windows spanning at most 32
// bins: half the multiply-adds and LDS reads of bin_amplitude.
template <int NC>
__device__ __forceinline__ float bin_amplitude_split(const float2 *buf, int mmx, const float2 *ftw, float2 wk)
{
    constexpr int NS = FftPlan<NC>::NS_LAST;
    constexpr int R = FftPlan<NC>::R_LAST;
    float2 a = buf[last_index<NS>(mmx, 0)];
#pragma unroll
    for (int t = 1; t < R; ++t) a = cmac(a, buf[last_index<NS>(mmx, t)], ftw[t - 1]);
    const float2 b = make_float2(__shfl_xor(a.x, 32), __shfl_xor(a.y, 32));
    const float2 e2 = make_float2(a.x + b.x, a.y - b.y);
    const float2 o2 = make_float2(a.y + b.y, b.x - a.x);
    const float2 x2 = cmac(e2, o2, wk);
    return 0.5f * sqrtf(fmaf(x2.x, x2.x, x2.y * x2.y));
}

// |X_k| of the real input from the full packed transform Z (length NC,
// swizzled): X_k = E_k + exp(-2 pi i k / NB) O_k, 0 <= k <= NC.
template <int NC>
__device__ __forceinline__ float real_amplitude(const float2 *__restrict__ Z, const float2 *__restrict__ Wg, int k)
{
    const float2 zk = Z[swz(k & (NC - 1))];
    const float2 zm = Z[swz((NC - k) & (NC - 1))];
    const float2 e = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
    const float2 o = make_float2(0.5f * (zk.y + zm.y), -0.5f * (zk.x - zm.x));
    const float2 x = cadd(e, cmul(Wg[k], o));
    return sqrtf(fmaf(x.x, x.x, x.y * x.y));
}

// Maximum over the 16 lanes of each row of the wavefront (every lane of the
// row receives it): xor-1 and xor-2 quad permutations, then the half-row and
// row mirrors.
__device__ __forceinline__ float row_max16(float x)
{
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false)));
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, false)));
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xF, 0xF, false)));
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xF, 0xF, false)));
    return x;
}

// Eq. (1) for one atom: bin index, FP32, fixed operation order.  The
// conversion truncates, takes everything below 0 (and what is not a number) to
// 0 and everything past 2^32 to its largest, so with the minimum it is
// clamp(floor(t), 0, last) for every t; a clamp of t before a signed
// conversion is a half-rate instruction (200 ROIs of 1006 atoms and 10242
// directions: 1000 us with it, 985 without).
__device__ __forceinline__ int eq1_bin(float vx, float vy, float vz, float dx, float dy, float dz, float shift,
                                       float scale, int last)
{
    const float s = fmaf(vz, dz, fmaf(vy, dy, vx * dx));
    const float t = (s + shift) * scale;
    uint32_t b;
    asm("v_cvt_u32_f32 %0, %1" : "=v"(b) : "v"(t));
    return (int)min(b, (uint32_t)last);
}

// ------------------------------------------------- windows on matrix cores
// When the windows span at most 32 bins, only those bins of the spectrum are
// evaluated, as a product on the matrix cores instead of an FFT.  With
// n = N2 n1 + n2 (n1 < 64, N2 = NB / 64) and m = n1 + 1/2,
//   X_k = sum_n2 e^(-2 pi i k (n2 - N2 / 2) / NB) S[n2][k],
//   S[n2][k] = sum_n1 h[N2 n1 + n2] e^(-2 pi i k m / 64).
// m and 64 - m (n1 and 63 - n1) have the same cosine and opposite sines, so
// the sums run over 32 pairs, cosines of h + h' and sines of h - h'.  The
// inner sums of H = 32 / N2 directions are one 32-row product with the 32 x
// 32 tables of cosines and sines (v_mfma_f32_32x32x16_f16; row d N2 + n2,
// column k - kmin), the outer sum of N2 terms is FP32 on the vector unit.
//
// A histogram word holds two directions, d in its low 16 bits and d + H in
// its high 16, counted by adding 1 or 65536: a wavefront passes D = 2 H
// directions through H histograms, so that clearing and reading them, and
// reading the atoms, cost half as much per direction.  The low halves are one
// row tile of the product, the high halves another.  ROIs past kSpan atoms go
// through the histograms in spans, their spectra added.
//
// Exactness: a count c < 2048 is the FP16 number of bit pattern c, c 2^-24, so
// a pair of histogram words becomes a pair of A operands by packing, an
// integer addition of the partners' pair, and one v_pk_mul_f16 by 2^10
// (h + h') or v_pk_fma_f16 (h - h' = 2 h - (h + h')).  (The product makes it a
// normal number: the matrix cores keep subnormals but align them as if they
// were 2^-14, which cost the accumulator up to 10 of its bits, 3e-5 of |X_k|
// for one atom.)  The table entries are split into two FP16 parts (22 bits);
// products are exact and accumulate in FP32; 2^14 goes into the outer factors.
// Where a pair holds more than 2047 counts, they go in as their low 10 and
// high 6 bits.
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int NB> struct BinPlan {
    static constexpr int N2 = NB / 64;          // rows per direction
    static constexpr int H = 32 / N2;           // histograms per wavefront, two directions each
    static constexpr int D = 2 * H;             // directions per wavefront pass
    static constexpr int X = (H + 1) / 2;       // spectra per lane and row tile
    static constexpr int STRIDE = NB + N2;      // words from one histogram to the next: the rows read
                                                // together (d, n2) then lie in 32 different banks
    static constexpr int WORDS = H * STRIDE;    // histograms of one wavefront
    static constexpr int TW = N2 == 4 ? 4 : N2 / 2;   // outer factors per lane
    static_assert(NB >= 256 && NB <= 2048, "16, 8, 4 or 2 directions per pass");
};
// Most atoms in the histograms at once.  Spans start at its multiples, so what
// they add up, and in which order, does not depend on the stage.
constexpr int kSpan = 61440;
static_assert(kSpan < 65536, "a 16-bit half counts them");

// Per-lane tables, loaded once per kernel; k = the lane's bin (lane % 32).
template <int NB> struct BinTables {
    using P = BinPlan<NB>;
    f16x8 c_hi[2], c_lo[2], s_hi[2], s_lo[2];   // B operands of the two slices of 16 pairs: cos, -sin of 2 pi k m / 64
    float2 tw[P::TW];                            // 2^14 e^(-2 pi i k (n2 - N2 / 2) / NB), n2 of the lane's rows
    int rd;                                      // row reduction: bin read by this lane

    __device__ __forceinline__ void load(const float2 *__restrict__ Wg, const WindowSet &ws, int lane)
    {
        const int k = min(ws.kmin + (lane & 31), ws.kmax), h = lane >> 5;
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float2 w = Wg[(k * (2 * (16 * s + 8 * h + e) + 1) * (P::N2 / 2)) & (NB - 1)];
                c_hi[s][e] = (_Float16)w.x;
                c_lo[s][e] = (_Float16)(w.x - (float)c_hi[s][e]);
                s_hi[s][e] = (_Float16)w.y;
                s_lo[s][e] = (_Float16)(w.y - (float)s_hi[s][e]);
            }
        // D layout: value i of lane l is row 8 (i / 4) + 4 (l / 32) + i % 4
#pragma unroll
        for (int i = 0; i < P::TW; ++i) {
            const int n2 = P::N2 == 4 ? i : 8 * (i >> 2) + 4 * h + (i & 3);
            const float2 w = Wg[(k * (n2 - P::N2 / 2)) & (NB - 1)];
            tw[i] = make_float2(w.x * 16384.0f, w.y * 16384.0f);
        }
        rd = 0;
        const int w = lane >> 4, i = lane & 15;
        for (int u = 0; u < ws.n && u < 4; ++u)
            if (w == u) rd = ws.lo[u] - ws.kmin + min(i, ws.hi[u] - ws.lo[u]);
    }
};

// A operands of 8 pairs (c[e], p[e]) of at most 2047 counts together, in
// units of 2^-14: their sums and differences.  x, y: the counts packed in
// pairs.
__device__ __forceinline__ void pair_operands(const uint32_t (&x)[4], const uint32_t (&y)[4], f16x8 &sum, f16x8 &diff)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const f16x2 s = __builtin_bit_cast(f16x2, x[e] + y[e]) * (_Float16)1024.0f;
        const f16x2 d =
            __builtin_elementwise_fma(__builtin_bit_cast(f16x2, x[e]), f16x2{(_Float16)2048.0f, (_Float16)2048.0f}, -s);
        sum[2 * e] = s.x;
        sum[2 * e + 1] = s.y;
        diff[2 * e] = d.x;
        diff[2 * e + 1] = d.y;
    }
}

// Low (TILE 0) or high (TILE 1) halves of two words, packed.
template <int TILE> __device__ __forceinline__ uint32_t pack_half(uint32_t a, uint32_t b)
{
    return __builtin_amdgcn_perm(b, a, TILE == 0 ? 0x05040100u : 0x07060302u);
}

// Sums over the rows held by this lane for the directions of one row tile
// (the low or the high halves of the histogram words).  H = 1: y[0] is the
// tile's one direction; else y[2 j], y[2 j + 1] are directions 2 j and 2 j + 1
// (N2 = 4: y[j] alone, direction 2 j + lane / 32).  WIDE: some pair holds more
// than 2047 counts, so the counts go in as their low 10 and high 6 bits.
template <int NB, int TILE, bool WIDE>
__device__ __forceinline__ void tile_rows(const int *up, const int *down, const BinTables<NB> &t,
                                          float2 (&y)[BinPlan<NB>::H])
{
    using P = BinPlan<NB>;
    f32x16 C, S;
#pragma unroll
    for (int i = 0; i < 16; ++i) C[i] = S[i] = 0.f;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        uint32_t a[4], b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] = pack_half<TILE>((uint32_t)up[(16 * s + 2 * e) * P::N2], (uint32_t)up[(16 * s + 2 * e + 1) * P::N2]);
            b[e] = pack_half<TILE>((uint32_t)down[-(16 * s + 2 * e) * P::N2],
                                   (uint32_t)down[-(16 * s + 2 * e + 1) * P::N2]);
        }
#pragma unroll
        for (int hi = 0; hi < (WIDE ? 2 : 1); ++hi) {
            f16x8 sum, diff;
            if constexpr (WIDE) {
                const uint32_t mask = hi ? 0x003f003fu : 0x03ff03ffu;
                uint32_t c[4], d[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    c[e] = (a[e] >> (hi ? 10 : 0)) & mask;
                    d[e] = (b[e] >> (hi ? 10 : 0)) & mask;
                }
                pair_operands(c, d, sum, diff);
                sum = sum * (_Float16)(hi ? 1024.0f : 1.0f);
                diff = diff * (_Float16)(hi ? 1024.0f : 1.0f);
            } else {
                pair_operands(a, b, sum, diff);
            }
            C = __builtin_amdgcn_mfma_f32_32x32x16_f16(sum, t.c_lo[s], C, 0, 0, 0);
            S = __builtin_amdgcn_mfma_f32_32x32x16_f16(diff, t.s_lo[s], S, 0, 0, 0);
            C = __builtin_amdgcn_mfma_f32_32x32x16_f16(sum, t.c_hi[s], C, 0, 0, 0);
            S = __builtin_amdgcn_mfma_f32_32x32x16_f16(diff, t.s_hi[s], S, 0, 0, 0);
        }
    }
#pragma unroll
    for (int d = 0; d < 16 / P::TW && d < P::H; ++d) {
        const int i0 = d * P::TW;
        float2 z[4];   // four partial sums, as short as the terms allow
#pragma unroll
        for (int i = 0; i < 4; ++i) z[i] = cmul(make_float2(C[i0 + i], S[i0 + i]), t.tw[i]);
#pragma unroll
        for (int i = 4; i < P::TW; ++i) z[i & 3] = cmac(z[i & 3], make_float2(C[i0 + i], S[i0 + i]), t.tw[i]);
        y[d] = cadd(cadd(z[0], z[1]), cadd(z[2], z[3]));
    }
}

// Adds the spectra of the wavefront's histograms: x[t][j] is bin lane % 32 of
// direction t H + 2 j + lane / 32 (H = 1: x[0][0] of direction lane / 32).
// `hist` is the lane's row of its histogram, h its half (lane / 32).  large:
// pairs past 2047 counts are possible and looked for.
template <int NB>
__device__ __forceinline__ void bin_spectra(const int *hist, int h, const BinTables<NB> &t, bool large,
                                            float2 (&x)[2][BinPlan<NB>::X])
{
    using P = BinPlan<NB>;
    const int *up = hist + 8 * h * P::N2, *down = hist + (63 - 8 * h) * P::N2;   // n1 and 63 - n1
    uint32_t any = 0;
    if (large) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t c = (uint32_t)up[(16 * s + e) * P::N2], p = (uint32_t)down[-(16 * s + e) * P::N2];
                any |= ((c & 0xffffu) + (p & 0xffffu)) | ((c >> 16) + (p >> 16));
            }
    }
    float2 lo[P::H], hi[P::H];
    // both halves hold half the rows of two directions a and b: swap so that
    // the lower half sums a and the upper b
    auto join = [](float2 a, float2 b) {
        const auto re = __builtin_amdgcn_permlane32_swap(__float_as_uint(a.x), __float_as_uint(b.x), false, false);
        const auto im = __builtin_amdgcn_permlane32_swap(__float_as_uint(a.y), __float_as_uint(b.y), false, false);
        return make_float2(__uint_as_float(re[0]) + __uint_as_float(re[1]),
                           __uint_as_float(im[0]) + __uint_as_float(im[1]));
    };
    auto add = [&](int tile, const float2 (&y)[P::H]) {
#pragma unroll
        for (int j = 0; j < P::X; ++j) {
            if constexpr (P::N2 == 4) x[tile][j] = cadd(x[tile][j], y[j]);
            else if constexpr (P::H > 1) x[tile][j] = cadd(x[tile][j], join(y[2 * j], y[2 * j + 1]));
        }
    };
    if (!__any(any > 2047u)) {
        tile_rows<NB, 0, false>(up, down, t, lo);
        add(0, lo);
        tile_rows<NB, 1, false>(up, down, t, hi);
        add(1, hi);
    } else {
        tile_rows<NB, 0, true>(up, down, t, lo);
        add(0, lo);
        tile_rows<NB, 1, true>(up, down, t, hi);
        add(1, hi);
    }
    if constexpr (P::H == 1) x[0][0] = cadd(x[0][0], join(lo[0], hi[0]));
}

}  // namespace sig
}  // namespace ar
