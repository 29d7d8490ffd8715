// A 64 x 64 tile of C = A B in float on the matrix cores, for the kernel
// matrices of spectra and the gradient of their loss.  (The sparse model has a
// tile of its own, gpr.hip: on this one its two products of 1024 centres, 715
// features and 2000 active points took 53 and 52 us against 51 and 48.)
//
// One work-group of four waves per tile; each wave owns a 32 x 32 quarter as
// 2 x 2 accumulators of v_mfma_f32_16x16x4_f32 (lane (r, g) = (lane & 15,
// lane >> 4) supplies A[r][g] and B[g][r] and holds D[4g + v][r]).  The
// contraction runs in slabs of 32 staged in LDS as [row][32 + 4] for both
// operands, so a lane's four consecutive values of one row are one 16-byte
// read that feeds four steps: step s of a 16-wide half takes the inner index
// 4g + s on both sides, a permutation that leaves the sum's terms unchanged.
// Per half, 4 LDS reads (16 bytes a lane) feed 16 MFMAs of 32 cycles; the
// row stride of 36 words puts 16 rows on distinct banks.  Two slab buffers
// and one barrier per slab: the next slab's global loads are in flight
// during the current slab's products.
//
// Bound by the FP32 matrix rate (a plain 8192-cubed library product reaches
// 150 TFLOP/s here); the tile needs 64 x 64 x 2 flops for 512 bytes read per
// inner index, 16 flop/B from L2.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace soap {
namespace tf {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;   // output rows and columns of a work-group
constexpr int kSlab = 32;   // inner indices per LDS slab
constexpr int kRow = kSlab + 4;

struct Smem {
    float a[2][kTile][kRow];
    float b[2][kTile][kRow];
};

// Output v < 4 of accumulator (bi, bj) of this lane sits at row
// out_row(bi) + v and column out_col(bj) of the tile.
__device__ __forceinline__ int out_row(int bi)
{
    const int w = threadIdx.x >> 6, g = (threadIdx.x >> 4) & 3;
    return 32 * (w >> 1) + 16 * bi + 4 * g;
}
__device__ __forceinline__ int out_col(int bj)
{
    const int w = threadIdx.x >> 6, r = threadIdx.x & 15;
    return 32 * (w & 1) + 16 * bj + r;
}

// Weight of inner index k in the full symmetric spectrum (k runs over
// repeated packed triangles q1 <= q2 of Q channels: 1 on the diagonal, 2 off
// it), walked in steps of one slab.
struct TriWeight {
    int Q, QQ, t, q, dq;   // t: position in the triangle, in row q that starts at dq
    __device__ __forceinline__ void init(int Q_, int64_t k)
    {
        Q = Q_;
        QQ = Q * (Q + 1) / 2;
        t = int(k % QQ);
        // row of t from the triangle's closed form, then to the exact row
        const float b = 2.0f * Q + 1.0f;
        q = int(0.5f * (b - sqrtf(fmaxf(b * b - 8.0f * t, 0.0f)))) - 1;
        q = q < 0 ? 0 : (q > Q - 1 ? Q - 1 : q);
        while (q > 0 && q * Q - q * (q - 1) / 2 > t) --q;
        dq = q * Q - q * (q - 1) / 2;
        settle();
    }
    __device__ __forceinline__ void settle()
    {
        while (t >= dq + Q - q) {
            dq += Q - q;
            ++q;
        }
    }
    __device__ __forceinline__ float value() const { return t == dq ? 1.0f : 2.0f; }
    __device__ __forceinline__ void advance()
    {
        t += kSlab;
        if (t >= QQ) {
            t %= QQ;
            q = 0;
            dq = 0;
        }
        settle();
    }
};
struct NoWeight {};

// acc = sum over k_begin <= k < k_end of A(i, k) B(k, j) for the tile's rows
// i (a points at its row 0, rows_a of them exist) and columns j (cols_b).
//   A(i, k) = a[i * lda + k], times w's value when W is TriWeight (w starts
//             at the lane's first index, k_begin + (threadIdx.x & 31))
//   B(k, j) = B_ROWS ? b[j * ldb + k] : b[k * ldb + j]
// Rows, columns and inner indices past the end read as zero.
template <bool B_ROWS, class W>
__device__ __forceinline__ void product(Smem& sm, const float* __restrict__ a, int64_t lda, int rows_a,
                                        const float* __restrict__ b, int64_t ldb, int cols_b, int64_t k_begin,
                                        int64_t k_end, W w, f32x4 (&acc)[2][2])
{
    constexpr bool WEIGHT = std::is_same<W, TriWeight>::value;
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
    // staging: rows of consecutive k (lane kl of a half-wave, rows rl + 8 u),
    // or for B_ROWS = false columns of consecutive j with four k each
    const int kl = tid & 31, rl = tid >> 5, jl = tid & 63, kq = tid >> 6;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (k_begin >= k_end) return;
    float ra[8], rb[8];
    const bool full = rows_a >= kTile && cols_b >= kTile;
    auto fetch = [&](int64_t k0) __attribute__((always_inline)) {
        const bool whole = full && k0 + kSlab <= k_end;
        const float* pa = a + int64_t(rl) * lda + k0 + kl;
        if (whole) {
#pragma unroll
            for (int u = 0; u < 8; ++u) ra[u] = pa[8 * u * lda];
            if (B_ROWS) {
                const float* pb = b + int64_t(rl) * ldb + k0 + kl;
#pragma unroll
                for (int u = 0; u < 8; ++u) rb[u] = pb[8 * u * ldb];
            } else {
                const float* pb = b + (k0 + 4 * kq) * ldb + jl;
#pragma unroll
                for (int u = 0; u < 8; ++u) rb[u] = pb[(16 * (u >> 2) + (u & 3)) * ldb];
            }
        } else {
            const bool kin = k0 + kl < k_end;
#pragma unroll
            for (int u = 0; u < 8; ++u) ra[u] = kin && rl + 8 * u < rows_a ? pa[8 * u * lda] : 0.0f;
            if (B_ROWS) {
                const float* pb = b + int64_t(rl) * ldb + k0 + kl;
#pragma unroll
                for (int u = 0; u < 8; ++u) rb[u] = kin && rl + 8 * u < cols_b ? pb[8 * u * ldb] : 0.0f;
            } else {
                const int64_t k1 = k0 + 4 * kq;
                const float* pb = b + k1 * ldb + jl;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int dk = 16 * (u >> 2) + (u & 3);
                    rb[u] = jl < cols_b && k1 + dk < k_end ? pb[dk * ldb] : 0.0f;
                }
            }
        }
    };
    auto put = [&](int buf) __attribute__((always_inline)) {
        if constexpr (WEIGHT) {
            const float wf = w.value();
            w.advance();
#pragma unroll
            for (int u = 0; u < 8; ++u) ra[u] *= wf;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) sm.a[buf][rl + 8 * u][kl] = ra[u];
        if (B_ROWS) {
#pragma unroll
            for (int u = 0; u < 8; ++u) sm.b[buf][rl + 8 * u][kl] = rb[u];
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
                *reinterpret_cast<float4*>(&sm.b[buf][jl][16 * h + 4 * kq]) =
                    make_float4(rb[4 * h], rb[4 * h + 1], rb[4 * h + 2], rb[4 * h + 3]);
        }
    };
    const int ar = 32 * (wave >> 1) + r, bc = 32 * (wave & 1) + r;
    fetch(k_begin);
    put(0);
    __syncthreads();
    int buf = 0;
    for (int64_t k0 = k_begin; k0 < k_end; k0 += kSlab, buf ^= 1) {
        const bool more = k0 + kSlab < k_end;
        if (more) fetch(k0 + kSlab);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            f32x4 av[2], bv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                av[i] = *reinterpret_cast<const f32x4*>(&sm.a[buf][ar + 16 * i][16 * h + 4 * g]);
                bv[i] = *reinterpret_cast<const f32x4*>(&sm.b[buf][bc + 16 * i][16 * h + 4 * g]);
            }
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][s], bv[j][s], acc[i][j], 0, 0, 0);
        }
        if (more) {
            put(buf ^ 1);
            __syncthreads();
        }
    }
}

}  // namespace tf
}  // namespace soap
