// Power spectrum on the matrix cores (gfx950 MFMA), bfloat16 operands with
// float accumulation, and the same kernel with FP32 operands
// (v_mfma_f32_16x16x4_f32, four of the 2l+1 values per step) for the FP32
// path of many centres.
//
// For a centre and a degree l the power spectrum is the Gram matrix
//   P_l = C_l C_l^T,   C_l = [c_{k, l^2 .. l^2+2l}]  (K x (2l+1)),
// of which the packed upper triangle k1 <= k2 is kept (Sec. 2 Eq.
// nu2-basis-coupled with real coefficients).  bfloat16 keeps 8 significant
// bits, too few for a 2e-3 relative error on p, so C is split into
// H = bf16(C) and L = bf16(C - H) and
//   P_l ~= H H^T + H L^T + L H^T,
// three products of inner dimension 2l+1 (one 32-wide MFMA step each for
// lmax <= 12); the dropped L L^T term and the rounding of L leave a
// relative error of order 2^-16.
//
// W waves own one centre (W = 1, four centres per work-group, when C is
// small and K <= 48; otherwise one centre per work-group of W = 4 or 8 waves,
// see waves_per_centre): the centre's waves split C into their LDS region as {H, L} pairs, then for
// each l run the 16 x 16 output tiles (I <= J) as three
// v_mfma_f32_16x16x32_bf16 each (a lane reads 8 consecutive {H, L} words
// of each of its two rows; one wave per centre reads every row block's
// words into registers once per l, four waves take contiguous runs of
// tiles in row-major order and read a row block once per row they touch),
// put the packed upper triangle in LDS and store it as contiguous float4
// rows (the accumulators alone give 64-byte pieces).
// One wave per centre needs no work-group barrier; four take two per l.
#include "soap_internal.hpp"

namespace soap {

hipError_t launch_power_spectrum_valu(const FeatureArgs& a, bool f64, hipStream_t stream);

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kLoadBatch = 16;   // coefficient loads a lane keeps in flight
constexpr int kRows1 = 3;        // row blocks of 16 (K <= 48) a one-wave centre holds in registers
constexpr int kStepsF32 = 7;     // 4-wide MFMA steps of a row of 2l+1 <= 25 values (lmax <= 12)
constexpr int64_t kF32MfmaAtoms = 8192;   // FP32 spectra of at least this many centres use the matrix cores

// round to nearest even (finite inputs)
__device__ __forceinline__ unsigned short to_bf16(float f)
{
    unsigned int u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

__device__ __forceinline__ float from_bf16(unsigned short h) { return __uint_as_float((unsigned int)h << 16); }

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A lane's operand values of row k of C_l (hl_l points at m = 8 kg of row
// 0): {H, L} words m = 8 kg + j, zero for j >= nj (past 2l+1) or k >= K.
// Rows past K read row 0, and every read stays inside the {H, L} region
// (padded by 32 words past C).
__device__ __forceinline__ void row_operands(const unsigned int* hl_l, int k, int K, int L2, int nj, u16x8& h,
                                             u16x8& lo)
{
    const unsigned int* r = hl_l + (k < K ? k : 0) * L2;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const unsigned int x = j < nj && k < K ? r[j] : 0u;
        h[j] = (unsigned short)(x & 0xFFFFu);
        lo[j] = (unsigned short)(x >> 16);
    }
}

// The 16 x 16 tile (I, J) of P_l ~= H H^T + H L^T + L H^T into the packed
// upper triangle ob, given the operand values of rows I (ha, la) and J
// (hb, lb).
__device__ __forceinline__ void tile(float* ob, int I, int J, int row, int kg, int K, const u16x8& ha,
                                     const u16x8& la, const u16x8& hb, const u16x8& lb)
{
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ha), __builtin_bit_cast(bf16x8, hb), acc,
                                                  0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ha), __builtin_bit_cast(bf16x8, lb), acc,
                                                  0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, la), __builtin_bit_cast(bf16x8, hb), acc,
                                                  0, 0, 0);
    // lane holds D[4 kg + v][row] = P[k1][k2] with k1 = 16 I + 4 kg + v,
    // k2 = 16 J + row; the packed index k1 K - k1 (k1 - 1) / 2 + k2 - k1
    // grows by K - k1 - 1 from k1 to k1 + 1
    const int k2 = J * 16 + row;
    int k1 = I * 16 + 4 * kg;
    int idx = k1 * K - k1 * (k1 - 1) / 2 + (k2 - k1);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (k1 <= k2 && k2 < K) ob[idx] = acc[v];
        idx += K - k1 - 1;
        ++k1;
    }
}

// FP32 operands (v_mfma_f32_16x16x4_f32, NS = ceil((2l+1) / 4) steps of 4 of
// the 2l+1 values; a template parameter, so that a tile's reads are issued
// together and its steps follow without a branch each): lane (row, kg)
// supplies the values m = kg NS + s, s < NS, of row k of C_l (c_l points at
// m = 0 of row 0), so that its NS reads are consecutive; A and B take the
// same order of m, which leaves the product unchanged.  Zero past 2l+1; rows
// past K read row 0 (their outputs are not stored), and every read stays
// inside the region (padded by 32 words past C).
template <int NS>
__device__ __forceinline__ void row_operands_f32(const float* c_l, int k, int K, int L2, int w, int kg, float (&x)[NS])
{
    const float* r = c_l + (k < K ? k : 0) * L2 + kg * NS;
#pragma unroll
    for (int s = 0; s < NS; ++s) x[s] = r[s];
#pragma unroll
    for (int s = 0; s < NS; ++s) x[s] = kg * NS + s < w ? x[s] : 0.f;
}

// The tile (I, J) of P_l = C_l C_l^T from FP32 operands, into the packed
// upper triangle ob (the same output layout as the bfloat16 tile)
template <int NS>
__device__ __forceinline__ void tile_f32(float* ob, int I, int J, int row, int kg, int K, const float (&xa)[NS],
                                         const float (&xb)[NS])
{
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[s], xb[s], acc, 0, 0, 0);
    const int k2 = J * 16 + row;
    int k1 = I * 16 + 4 * kg;
    int idx = k1 * K - k1 * (k1 - 1) / 2 + (k2 - k1);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (k1 <= k2 && k2 < K) ob[idx] = acc[v];
        idx += K - k1 - 1;
        ++k1;
    }
}

// All tiles of degree l that this wave owns, FP32 operands (as the bfloat16
// form in the body below)
template <int W, int NS>
__device__ __forceinline__ void degree_f32(const float* c_l, float* ob, int K, int L2, int w, int T, int wc, int row,
                                           int kg)
{
    if constexpr (W == 1) {
        float rx[kRows1][NS];
#pragma unroll
        for (int I = 0; I < kRows1; ++I)
            if (I < T) row_operands_f32<NS>(c_l, I * 16 + row, K, L2, w, kg, rx[I]);
#pragma unroll
        for (int I = 0; I < kRows1; ++I)
#pragma unroll
            for (int J = I; J < kRows1; ++J)
                if (J < T) tile_f32<NS>(ob, I, J, row, kg, K, rx[I], rx[J]);
    } else {
        const int n_tiles = T * (T + 1) / 2;
        const int per = (n_tiles + W - 1) / W;
        const int t0 = wc * per, t1 = t0 + per < n_tiles ? t0 + per : n_tiles;
        if (t0 >= t1) return;
        int I = 0, rem = t0;
        while (I < T && rem >= T - I) { rem -= T - I; ++I; }
        int J = I + rem;
        float xa[NS], xb[NS];
        row_operands_f32<NS>(c_l, I * 16 + row, K, L2, w, kg, xa);
        row_operands_f32<NS>(c_l, J * 16 + row, K, L2, w, kg, xb);
        for (int t = t0;;) {
            // the next tile's column operands are read during this tile
            int I1 = I, J1 = J + 1;
            if (J1 == T) {
                ++I1;
                J1 = I1;
            }
            const bool more = ++t < t1;
            float xn[NS];
            if (more) row_operands_f32<NS>(c_l, J1 * 16 + row, K, L2, w, kg, xn);
            tile_f32<NS>(ob, I, J, row, kg, K, xa, xb);
            if (!more) break;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                xb[s] = xn[s];
                if (I1 != I) xa[s] = xn[s];   // a row starts on the diagonal
            }
            I = I1;
            J = J1;
        }
    }
}

// One body for both operand forms: F32 keeps C in FP32 (the FP32 path),
// otherwise the {H, L} bfloat16 split.
template <int W, bool F32>
__device__ __forceinline__ void spectrum_body(const FeatureArgs& a)
{
    constexpr int CPG = W > 4 ? 1 : 4 / W;   // centres per work-group
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int S = a.S, nmax = a.nmax, lmax = a.lmax;
    const int K = S * nmax, L2 = (lmax + 1) * (lmax + 1);
    const int KK = K * (K + 1) / 2;
    const int KL2 = K * L2;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int slot = wave / W, wc = wave - slot * W;   // centre slot in the work-group, wave within the centre
    const int64_t i = int64_t(blockIdx.x) * CPG + slot;
    if (i >= a.n_atoms) return;
    // {H, L} of every element of C: H in the low half, L in the high half;
    // then the packed P_l of the current l
    const int HLS = (KL2 + 32 + 3) & ~3, OBS = (KK + 3) & ~3;   // 16-byte aligned regions
    unsigned int* hl = reinterpret_cast<unsigned int*>(smem_raw) + size_t(slot) * (HLS + OBS);
    float* ob = reinterpret_cast<float*>(hl + HLS);
    const float* c_in = static_cast<const float*>(a.coeffs) + i * KL2;
    // kLoadBatch loads in flight per lane before any is used
    for (int e0 = wc * 64 + lane; e0 < KL2; e0 += kLoadBatch * W * 64) {
        float v[kLoadBatch];
#pragma unroll
        for (int u = 0; u < kLoadBatch; ++u) {
            const int e = e0 + u * W * 64;
            v[u] = e < KL2 ? c_in[e] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kLoadBatch; ++u) {
            const int e = e0 + u * W * 64;
            if (e < KL2) {
                if constexpr (F32) {
                    hl[e] = __float_as_uint(v[u]);
                } else {
                    const unsigned short h = to_bf16(v[u]);
                    hl[e] = (unsigned int)h | ((unsigned int)to_bf16(v[u] - from_bf16(h)) << 16);
                }
            }
        }
    }
    if (W == 1) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();   // one centre per work-group
    }
    const int T = (K + 15) / 16;
    const int row = lane & 15, kg = lane >> 4;
    float* p_out = static_cast<float*>(a.p) + i * int64_t(lmax + 1) * KK;
    for (int l = 0; l <= lmax; ++l) {
        const int w = 2 * l + 1;   // <= 25 for lmax <= 12: one 32-wide step per product
        const int nj = w - 8 * kg;  // this lane's operand values m = 8 kg + j with j < nj are inside the row
        const unsigned int* hl_l = hl + l * l + kg * 8;
        float* dst = p_out + int64_t(l) * KK;
        // tiles (I, J), I <= J, row-major over the upper triangle
        const float* c_l = reinterpret_cast<const float*>(hl) + l * l;
        if constexpr (F32) {
            switch ((w + 3) / 4) {
            case 1: degree_f32<W, 1>(c_l, ob, K, L2, w, T, wc, row, kg); break;
            case 2: degree_f32<W, 2>(c_l, ob, K, L2, w, T, wc, row, kg); break;
            case 3: degree_f32<W, 3>(c_l, ob, K, L2, w, T, wc, row, kg); break;
            case 4: degree_f32<W, 4>(c_l, ob, K, L2, w, T, wc, row, kg); break;
            case 5: degree_f32<W, 5>(c_l, ob, K, L2, w, T, wc, row, kg); break;
            case 6: degree_f32<W, 6>(c_l, ob, K, L2, w, T, wc, row, kg); break;
            default: degree_f32<W, kStepsF32>(c_l, ob, K, L2, w, T, wc, row, kg); break;
            }
        } else
        if constexpr (W == 1) {
            // one wave: the operand values of every row block read once
            // (T <= kRows1), all reads issued before the first product
            {
                u16x8 rh[kRows1], rl[kRows1];
#pragma unroll
                for (int I = 0; I < kRows1; ++I)
                    if (I < T) row_operands(hl_l, I * 16 + row, K, L2, nj, rh[I], rl[I]);
#pragma unroll
                for (int I = 0; I < kRows1; ++I)
#pragma unroll
                    for (int J = I; J < kRows1; ++J)
                        if (J < T) tile(ob, I, J, row, kg, K, rh[I], rl[I], rh[J], rl[J]);
            }
        } else {
            // each wave a contiguous run of tiles in row-major order, so
            // that row I's operand values are read once per row it touches
            const int n_tiles = T * (T + 1) / 2;
            const int per = (n_tiles + W - 1) / W;
            const int t0 = wc * per, t1 = t0 + per < n_tiles ? t0 + per : n_tiles;
            int I = 0, rem = t0;
            while (I < T && rem >= T - I) { rem -= T - I; ++I; }
            int J = I + rem;
            {
                u16x8 ha, la;
                if (t0 < t1) row_operands(hl_l, I * 16 + row, K, L2, nj, ha, la);
                for (int t = t0; t < t1; ++t) {
                    u16x8 hb, lb;
                    row_operands(hl_l, J * 16 + row, K, L2, nj, hb, lb);
                    tile(ob, I, J, row, kg, K, ha, la, hb, lb);
                    if (++J == T && t + 1 < t1) {
                        ++I;
                        J = I;
                        row_operands(hl_l, I * 16 + row, K, L2, nj, ha, la);
                    }
                }
            }
        }
        {
            // the packed P_l leaves as contiguous rows: float4 stores when
            // aligned, else one float per lane
            if (W == 1) wave_sync(); else __syncthreads();
            if ((KK & 3) == 0 && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
                for (int e = wc * 64 + lane; e < KK / 4; e += W * 64)
                    reinterpret_cast<float4*>(dst)[e] = reinterpret_cast<const float4*>(ob)[e];
            } else {
                for (int e = wc * 64 + lane; e < KK; e += W * 64) dst[e] = ob[e];
            }
            if (W == 1) wave_sync(); else __syncthreads();
        }
    }
}

template <int W>
__global__ void __launch_bounds__(W > 4 ? 64 * W : kThreads) k_power_spectrum_bf16(FeatureArgs a)
{
    spectrum_body<W, false>(a);
}

template <int W>
__global__ void __launch_bounds__(W > 4 ? 64 * W : kThreads) k_power_spectrum_f32mfma(FeatureArgs a)
{
    spectrum_body<W, true>(a);
}

// LDS words of one centre's slot: {H, L} of C (or C), then the packed P_l
size_t slot_words(int S, int nmax, int lmax)
{
    const size_t K = size_t(S) * nmax, KL2 = K * (lmax + 1) * (lmax + 1), KK = K * (K + 1) / 2;
    return ((KL2 + 32 + 3) & ~size_t(3)) + ((KK + 3) & ~size_t(3));
}

// Waves per centre: one when four centres' slots fit 40 KB of LDS (and
// K <= 16 kRows1), four otherwise up to K = 64.  Above, eight where four would
// leave a CU under 20 waves (a slot over 32 KB: 16,384 centres at K = 96, lmax
// 8 in bfloat16 851 us with four and 806 with eight; 4096 at K = 80, lmax 9
// 186 and 174), or where the centres are few (100 at K = 66, lmax 4: 14.9 and
// 11.4); four where their work-groups fill it (16,384 at K = 66, lmax 4: 244
// and 288, in float 214 and 241).
int waves_per_centre(int S, int nmax, int lmax, int64_t n_atoms)
{
    const int K = S * nmax;
    const size_t slot = 4 * slot_words(S, nmax, lmax);
    if (K <= 16 * kRows1 && 4 * slot <= 40 * 1024) return 1;
    return K > 64 && (n_atoms <= 512 || slot > 32 * 1024) ? 8 : 4;
}

// FP32 spectra (without gradient rows) of fewer than kF32MfmaAtoms centres:
// matrix cores or the VALU kernel.  At K = 96 (lmax 8) 100 centres take 22
// against 74 us, 4096 217 against 374; K = 64 (lmax 6) 1000 centres 21 against
// 31; K = 24 (lmax 6) 4096 centres 16 against 19; at K = 20 (lmax 8) 22.2
// against 21.4, so fewer than 24 channels stay with the VALU.  So do
// channels that leave much of their 16-wide blocks empty: with four waves per
// centre and where the rows of c are odd, which the VALU kernel's LDS reads
// like (lmax even; 4096 centres at K = 33, lmax 8 49 against 40 us, K = 27
// lmax 8 35 against 29, K = 50 lmax 4 38 against 33; K = 36 lmax 9 60 against
// 79; K = 24 also in between, lmax 9 37 against 34), but not few centres; with
// one wave per centre and three blocks few centres (100 at K = 36, lmax 6
// 12.9 against 10.8 us, 4096 26 against 33).
bool f32_on_matrix_cores(int K, int lmax, int W, int64_t n_atoms)
{
    if (n_atoms >= kF32MfmaAtoms) return true;
    if (K < 24) return false;
    const bool third = K > 32 && K <= 38;   // a few channels in a third block
    if (W == 1) return !(third && lmax >= 5 && n_atoms <= 1000);
    if (n_atoms < 1000 || (lmax % 2 != 0 && K > 24)) return true;
    return !(K <= 30 || third || ((K == 49 || K == 50) && lmax >= 2 && lmax <= 6));
}

}  // namespace

template <int W, bool F32>
hipError_t launch_mfma(const FeatureArgs& a, size_t lds, hipStream_t stream)
{
    const void* fn = F32 ? reinterpret_cast<const void*>(k_power_spectrum_f32mfma<W>)
                         : reinterpret_cast<const void*>(k_power_spectrum_bf16<W>);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
        if (e != hipSuccess) return e;
    }
    constexpr int cpg = W > 4 ? 1 : 4 / W, threads = W > 4 ? 64 * W : kThreads;
    const unsigned groups = unsigned((a.n_atoms + cpg - 1) / cpg);
    if constexpr (F32)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_power_spectrum_f32mfma<W>), dim3(groups), dim3(threads), lds, stream, a);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_power_spectrum_bf16<W>), dim3(groups), dim3(threads), lds, stream, a);
    return hipGetLastError();
}

template <bool F32>
hipError_t launch_mfma_waves(const FeatureArgs& a, hipStream_t stream)
{
    const int W = waves_per_centre(a.S, a.nmax, a.lmax, a.n_atoms);
    const size_t lds = size_t(W == 1 ? 4 : 1) * 4 * slot_words(a.S, a.nmax, a.lmax);
    if (lds > 160 * 1024 || (F32 && a.lmax > 12)) return hipErrorNotSupported;
    if (a.n_atoms == 0) return hipSuccess;
    return W == 1   ? launch_mfma<1, F32>(a, lds, stream)
           : W == 4 ? launch_mfma<4, F32>(a, lds, stream)
                    : launch_mfma<8, F32>(a, lds, stream);
}

hipError_t launch_power_spectrum(const FeatureArgs& a, soap_precision prec, hipStream_t stream)
{
    if (prec == SOAP_F32 && a.dp == nullptr &&
        f32_on_matrix_cores(a.S * a.nmax, a.lmax, waves_per_centre(a.S, a.nmax, a.lmax, a.n_atoms), a.n_atoms)) {
        const hipError_t e = launch_mfma_waves<true>(a, stream);
        if (e != hipErrorNotSupported) return e;
    }
    if (prec != SOAP_BF16_F32ACC) return launch_power_spectrum_valu(a, prec == SOAP_F64, stream);
    return launch_mfma_waves<false>(a, stream);
}

}  // namespace soap
