// Pieces of the bfloat16 compression network shared by its one-wave-per-
// centre kernels (compress.hip: weights staged in LDS per work-group;
// compress_infer.hip: weights from a laid-out image).  Lane (r, g) =
// (lane & 15, lane >> 4) throughout.
#pragma once

#include <hip/hip_runtime.h>

namespace soap {
namespace cmp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// two floats to packed bfloat16 (round to nearest even), low half first
__device__ __forceinline__ unsigned int pack_bf16(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(unsigned int, __builtin_convertvector(v, bf16x2));
}

// exchanges between halves of a wave: lanes 32..63 of a with lanes 0..31 of
// b, or odd rows of 16 lanes of a with the even rows of b; the sum leaves a's
// total of lane pairs (32 or 16 apart) in the lower member and b's in the
// upper one
__device__ __forceinline__ float swap32_sum(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_sum(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// out[k] = x of the lane's row k of 16 lanes, in every row
__device__ __forceinline__ void gather_rows(float x, float (&out)[4])
{
    const unsigned u = __float_as_uint(x);
    const auto e = __builtin_amdgcn_permlane16_swap(u, u, false, false);        // rows 0 0 2 2, rows 1 1 3 3
    const auto p = __builtin_amdgcn_permlane32_swap(e[0], e[0], false, false);   // row 0, row 2
    const auto q = __builtin_amdgcn_permlane32_swap(e[1], e[1], false, false);   // row 1, row 3
    out[0] = __uint_as_float(p[0]);
    out[1] = __uint_as_float(q[0]);
    out[2] = __uint_as_float(p[1]);
    out[3] = __uint_as_float(q[1]);
}

__device__ __forceinline__ f32x4 mfma_bf16(u16x8 a, u16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                   0);
}
__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c)
{
    return mfma_bf16(__builtin_bit_cast(u16x8, a), __builtin_bit_cast(u16x8, b), c);
}

constexpr int kCB = 36;   // row stride of the c~ staging (floats, 16-byte rows)

// hidden unit in column `col` of layer-1 tile t: two tiles side by side hold
// the two units of each bfloat16 pair
__device__ __forceinline__ int hidden_unit(int t, int col) { return 32 * (t >> 1) + 2 * col + (t & 1); }

// The gate 2 sigma(alpha |h| + beta) of every hidden unit of one centre and
// degree, from h of MT column tiles: lane (r, g) holds unit hidden_unit(t, r)
// at column 16 ct + 4 g + v in h[ct][t][v].  gate[t] is that of the lane's
// unit of tile t.
//
// |h|^2 over m is added as a tree: m and m + 8 (lanes 32 apart), m + 4 (16
// apart), m + 2 and m + 1 (in the lane).  Each exchange halves the tiles a
// lane answers for, so that of 128 units lane (r, g) ends with 32 g + 2 r and
// 32 g + 2 r + 1 (of 64: 32 (g / 2) + 2 r and the next, every two rows of
// lanes alike) and every gate is formed once in the wave.  With the units in
// the rows every one of the 16 column lanes formed all 32 of its row's: 650
// of the 1,190 VALU instructions per degree, 4.40 against 3.48 ms for 131,072
// centres of 96 -> 128 -> 16 channels.
// al, be: alpha and beta of the lane's two units, q0 the first (past H: gate 0).
template <int MT, int HT>
__device__ __forceinline__ void gates(const f32x4 (&h)[MT][HT], const float2 al, const float2 be, bool in, float (&gate)[HT])
{
    auto square = [&](int t, int v) __attribute__((always_inline)) {
        if constexpr (MT == 2) return h[0][t][v] * h[0][t][v] + h[MT - 1][t][v] * h[MT - 1][t][v];
        else return h[0][t][v] * h[0][t][v];
    };
    float s4[2][4];
    if constexpr (HT == 8) {
        float s8[4][4];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) s8[t][v] = swap32_sum(square(t, v), square(t + 4, v));
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) s4[t][v] = swap16_sum(s8[t][v], s8[t + 2][v]);
    } else {
        float s8[2][4];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) s8[t][v] = swap32_sum(square(t, v), square(t + 2, v));
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) s4[t][v] = swap16_sum(s8[t][v], s8[t][v]);
    }
    const float alv[2] = {al.x, al.y}, bev[2] = {be.x, be.y};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const float s = (s4[t][0] + s4[t][2]) + (s4[t][1] + s4[t][3]);
        const float x = alv[t] * __builtin_amdgcn_sqrtf(s) + bev[t];
        const float G = in ? 2.0f * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x)) : 0.0f;
        float rows[4];
        gather_rows(G, rows);
#pragma unroll
        for (int k = 0; k < HT / 2; ++k) gate[2 * k + t] = rows[HT == 8 ? k : 2 * k];
    }
}

// first of the lane's two gated units
template <int HT>
__device__ __forceinline__ int gate_unit(int r, int g)
{
    return HT == 8 ? 32 * g + 2 * r : 32 * (g >> 1) + 2 * r;
}

// p~ of one degree from c~ staged as [output][kCB] over MT column tiles: the
// Gram matrix over m on the matrix cores, c~ split into bfloat16 high and low
// parts (H H^T + H L^T + L H^T, as for the full spectrum)
template <int MT, int QT>
__device__ __forceinline__ void spectrum_out(const float* cb, int Q, int r, int g, float* dst)
{
    // rows 16 P + r of c~ as the lane's operand: m = 8 g + j, zero past the
    // columns written for this degree
    u32x4 hi[QT], lo[QT];
#pragma unroll
    for (int P = 0; P < QT; ++P) {
        float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (8 * g < 16 * MT) {
            const float4 x0 = *reinterpret_cast<const float4*>(cb + (16 * P + r) * kCB + 8 * g);
            const float4 x1 = *reinterpret_cast<const float4*>(cb + (16 * P + r) * kCB + 8 * g + 4);
            x[0] = x0.x; x[1] = x0.y; x[2] = x0.z; x[3] = x0.w;
            x[4] = x1.x; x[5] = x1.y; x[6] = x1.z; x[7] = x1.w;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const unsigned int hp = pack_bf16(x[2 * j], x[2 * j + 1]);
            hi[P][j] = hp;
            lo[P][j] = pack_bf16(x[2 * j] - __uint_as_float(hp << 16), x[2 * j + 1] - __uint_as_float(hp & 0xFFFF0000u));
        }
    }
#pragma unroll
    for (int P1 = 0; P1 < QT; ++P1)
#pragma unroll
        for (int P2 = P1; P2 < QT; ++P2) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            acc = mfma_bf16(hi[P1], hi[P2], acc);
            acc = mfma_bf16(hi[P1], lo[P2], acc);
            acc = mfma_bf16(lo[P1], hi[P2], acc);
            // lane holds p~[p1][p2], p1 = 16 P1 + 4 g + v, p2 = 16 P2 + r
            const int p2 = 16 * P2 + r;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int p1 = 16 * P1 + 4 * g + v;
                if (p1 <= p2 && p2 < Q) dst[p1 * Q - p1 * (p1 - 1) / 2 + (p2 - p1)] = acc[v];
            }
        }
}

}  // namespace cmp
}  // namespace soap
