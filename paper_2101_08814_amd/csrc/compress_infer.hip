// bfloat16 inference of the learned compression with the weights laid out in
// a workspace: c of a centre is read from HBM once, as one contiguous run.
//
// One wave per centre and per work-group; no work-group barriers.
//   c        the centre's K x L2 floats, loaded 64 consecutive columns of a
//            channel at a time, rounded to bfloat16 and put into the wave's LDS as rows
//            [lm][k], so that a layer-1 operand is one 16-byte read.
//   per l    the columns of every product are the m of the centre (one
//            16-wide tile, two when 2l + 1 > 16):
//            layer 1 transposed (rows m, columns hidden units), the gate,
//            layer 2 through LDS in halves of 64 units, p~ from c~
//            (compress_bf16.hpp).
//   weights  k_cmp_image lays every degree's weights out as the operands of
//            the waves, 1 KB a fragment, so that a wave takes a fragment with
//            one coalesced 16-byte load per lane from L2; layer 1's fragments
//            of l + 1 are loaded during the gate, layer 2 and p~ of l.
//
// The form before shared a degree's weights in LDS between eight waves and
// read c one degree at a time: rows of 2l+1 floats every L2, whose cache
// lines were evicted from L2 before the next degree came back to them
// (155 M L2 misses, 19.8 GB, for 4.1 GB of c at K = 96, lmax 8), so the
// kernel ran at the memory's rate for five times its input.
#include "soap_internal.hpp"

#include "compress_bf16.hpp"

#include <type_traits>

namespace soap {
namespace {

using namespace cmp;

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a value that is the same in every lane, kept in a scalar register
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

constexpr int kHalf = 36;   // row stride of the gated columns in pairs of units: 32 of one half, and 4

struct InferLayout {
    int KS, HT, QT;
    int xs;                  // row stride of X in bfloat16 pairs: 4 more than K needs, so that
                             // 16 consecutive rows meet distinct banks in 16-byte reads
    int da, dm;              // 64 = da L2 + dm
    int x, stage, total;     // LDS byte offsets
    int frags;               // 1 KB fragments of one degree: layer 1, layer 2, {alpha, beta}
};

__host__ __device__ inline InferLayout infer_layout(int K, int Q, int H, int lmax)
{
    InferLayout L;
    L.KS = (K + 31) / 32;
    L.HT = H <= 64 ? 4 : 8;
    L.QT = (Q + 15) / 16;
    L.xs = 16 * L.KS + 4;
    const int L2 = (lmax + 1) * (lmax + 1);
    const int gt = 16 * kHalf * 4, cb = L.QT * 16 * kCB * 4;
    L.da = 64 / L2;
    L.dm = 64 - L.da * L2;
    L.x = 0;
    L.stage = (L2 + 1) * L.xs * 4;   // one more row, of zeros
    L.total = L.stage + (gt > cb ? gt : cb);
    L.frags = L.HT * L.KS + L.QT * (L.HT / 2) + 1;
    return L;
}

// fragment f of degree l, lane (r, g): layer 1 (t, kk): W1[unit of column r
// of tile t][32 kk + 8 g + j]; layer 2 (pt, ks): W2[16 pt + r][32 ks + 8 g +
// j], j < 8, as bfloat16; then alpha and beta in float, each 16 HT long
__global__ void __launch_bounds__(256) k_cmp_image(CompressArgs a, InferLayout L)
{
    const int l = blockIdx.y, K = a.K, H = a.H, Q = a.Q;
    const int e = blockIdx.x * 256 + threadIdx.x;   // 16-byte piece of the degree's image
    if (e >= L.frags * 64) return;
    const int f = e >> 6, r = e & 15, g = (e >> 4) & 3, n1 = L.HT * L.KS, n2 = L.QT * (L.HT / 2);
    const float* W1 = a.w + size_t(l) * (H * K + Q * H + 2 * H);
    const float* W2 = W1 + H * K;
    const float* al = W2 + Q * H;
    u32x4 out;
    if (f < n1 + n2) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (f < n1) {
                const int q = hidden_unit(f / L.KS, r), k = 32 * (f % L.KS) + 8 * g + j;
                x[j] = q < H && k < K ? W1[q * K + k] : 0.0f;
            } else {
                const int p = 16 * ((f - n1) / (L.HT / 2)) + r, q = 32 * ((f - n1) % (L.HT / 2)) + 8 * g + j;
                x[j] = p < Q && q < H ? W2[p * H + q] : 0.0f;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] = pack_bf16(x[2 * j], x[2 * j + 1]);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int t = 4 * (e & 63) + j, q = t % (16 * L.HT);   // alpha, then beta
            out[j] = t < 32 * L.HT && q < H ? __float_as_uint(al[t < 16 * L.HT ? q : H + q]) : 0u;
        }
    }
    static_cast<u32x4*>(a.img)[size_t(l) * L.frags * 64 + e] = out;
}

template <int QT, int KS, int HT>
__global__ void __launch_bounds__(64, 2) k_cmp_infer(CompressArgs a, InferLayout L)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int XS = 16 * KS + 4, KS2 = HT / 2;
    constexpr int N1 = HT * KS, N2 = QT * KS2, kFrags = N1 + N2 + 1;
    const int K = a.K, Q = a.Q, H = a.H, lmax = a.lmax, L2 = (lmax + 1) * (lmax + 1);
    const int QQ = Q * (Q + 1) / 2;
    const int lane = threadIdx.x, r = lane & 15, g = lane >> 4;
    // units in the last pair of tiles: without, its columns are zeros also
    // where c is not finite
    const bool last = H > 32 * (KS2 - 1);
    const int64_t i = blockIdx.x;
    unsigned* X = reinterpret_cast<unsigned*>(smem_raw);
    unsigned* gt = reinterpret_cast<unsigned*>(smem_raw + L.stage);
    float* cb = reinterpret_cast<float*>(smem_raw + L.stage);

    // layer 1's fragments of a degree, kept one degree ahead
    const u32x4* img = static_cast<const u32x4*>(a.img);
    u32x4 w1[N1];
    auto fetch_w1 = [&](int l) __attribute__((always_inline)) {
        const u32x4* src = img + size_t(l) * (kFrags * 64);
#pragma unroll
        for (int f = 0; f < N1; ++f) w1[f] = src[f * 64 + lane];
    };

    // c -> X.  Element f = 64 it + lane is (kq, lm) = (f / L2, f % L2): the
    // four channels 4 kq + j of column lm (K is a multiple of 4), one 8-byte
    // store; loads past the centre's array (channels past K) return zero.
    {
        const uint64_t c0 = reinterpret_cast<uint64_t>(a.c + i * int64_t(K) * L2);
        const uint64_t base = (uint64_t(unsigned(uniform(int(c0 >> 32)))) << 32) | unsigned(uniform(int(c0)));
        const int next = uniform(L2 * 4);   // bytes from a channel to the next one
        const __amdgpu_buffer_rsrc_t src =
            __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(base), 0, uniform(K * L2 * 4), 0x00020000);
        constexpr int kBatch = 8;   // elements in flight per lane; the next batch is loaded before this one is stored
        const int n = (8 * KS) * L2;
        const int dm = L.dm, step_from = (4 * L.da * L2 + dm) * 4, step_at = dm * XS + 2 * L.da;
        const int wrap_from = 3 * next, wrap_at = 2 - L2 * XS;
        const int kq = int((float(lane) + 0.5f) / float(L2));
        int lm = lane - kq * L2, from = (4 * kq * L2 + lm) * 4, to = lm * XS + 2 * kq;
        unsigned v[2][kBatch][4];
        int at[2][kBatch];
        auto load = [&](int b) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[b][u][j] = __builtin_amdgcn_raw_buffer_load_b32(src, from, j * next, 0);
                at[b][u] = to;
                lm += dm;
                const bool wrap = lm >= L2;
                lm -= wrap ? L2 : 0;
                from += step_from + (wrap ? wrap_from : 0);
                to += step_at + (wrap ? wrap_at : 0);
            }
        };
        auto store = [&](int b, int f0) __attribute__((always_inline)) {
            const bool whole = f0 + 64 * kBatch <= n;
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                if (whole || f0 + 64 * u + lane < n)
                    *reinterpret_cast<uint2*>(X + at[b][u]) =
                        make_uint2(pack_bf16(__uint_as_float(v[b][u][0]), __uint_as_float(v[b][u][1])),
                                   pack_bf16(__uint_as_float(v[b][u][2]), __uint_as_float(v[b][u][3])));
        };
        load(0);
        for (int f0 = 0; f0 < n; f0 += 2 * 64 * kBatch) {
            load(1);
            store(0, f0);
            load(0);
            store(1, f0 + 64 * kBatch);
        }
        if (lane < XS) X[L2 * XS + lane] = 0u;
        if (XS > 64 && lane + 64 < XS) X[L2 * XS + lane + 64] = 0u;
    }
    fetch_w1(0);
    wave_sync();

    // one degree with MT tiles of 16 columns m
    auto degree = [&](auto mt, int l) __attribute__((always_inline)) {
        constexpr int MT = decltype(mt)::value;
        const int M = 2 * l + 1, b = l * l;
        const u32x4* wl = img + size_t(l) * (kFrags * 64);
        u32x4 w2[N2];
#pragma unroll
        for (int f = 0; f < N2; ++f) w2[f] = wl[(N1 + f) * 64 + lane];
        const float* ab = reinterpret_cast<const float*>(wl + (N1 + N2) * 64);
        const int q0 = gate_unit<HT>(r, g);
        const float2 al = *reinterpret_cast<const float2*>(ab + q0);
        const float2 be = *reinterpret_cast<const float2*>(ab + 16 * HT + q0);
        // layer 1: rows m (of X, or the row of zeros), columns hidden units
        f32x4 h[MT][HT];
#pragma unroll
        for (int ct = 0; ct < MT; ++ct)
#pragma unroll
            for (int t = 0; t < HT; ++t) h[ct][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            u32x4 x[MT];
#pragma unroll
            for (int ct = 0; ct < MT; ++ct) {
                const int row = 16 * ct + r < M ? b + 16 * ct + r : L2;
                x[ct] = *reinterpret_cast<const u32x4*>(X + row * XS + 16 * kk + 4 * g);
            }
#pragma unroll
            for (int t = 0; t < HT; ++t)
#pragma unroll
                for (int ct = 0; ct < MT; ++ct) h[ct][t] = mfma_bf16(x[ct], w1[t * KS + kk], h[ct][t]);
        }
        if (l < lmax) fetch_w1(l + 1);
        float gate[HT];
        gates<MT, HT>(h, al, be, q0 < H, gate);
        // layer 2, 64 units at a time: the gated columns as bfloat16 pairs of
        // units in rows m, read back as operands
        f32x4 acc2[MT][QT];
#pragma unroll
        for (int ct = 0; ct < MT; ++ct)
#pragma unroll
            for (int pt = 0; pt < QT; ++pt) acc2[ct][pt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int hf = 0; hf < KS2 / 2; ++hf)
#pragma unroll
            for (int ct = 0; ct < MT; ++ct) {
                wave_sync();
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int t = 4 * hf + 2 * u;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        gt[(4 * g + v) * kHalf + 16 * u + r] =
                            2 * hf + u < KS2 - 1 || last ? pack_bf16(h[ct][t][v] * gate[t], h[ct][t + 1][v] * gate[t + 1]) : 0u;
                }
                wave_sync();
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const u32x4 B = *reinterpret_cast<const u32x4*>(gt + r * kHalf + 16 * u + 4 * g);
#pragma unroll
                    for (int pt = 0; pt < QT; ++pt) acc2[ct][pt] = mfma_bf16(w2[pt * KS2 + 2 * hf + u], B, acc2[ct][pt]);
                }
            }
        wave_sync();   // c~ goes over the gated columns
#pragma unroll
        for (int ct = 0; ct < MT; ++ct) {
            const int m = 16 * ct + r;
#pragma unroll
            for (int pt = 0; pt < QT; ++pt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int p = 16 * pt + 4 * g + v;
                    cb[p * kCB + m] = acc2[ct][pt][v];
                    if (a.ct && p < Q && m < M) a.ct[(i * Q + p) * int64_t(L2) + b + m] = acc2[ct][pt][v];
                }
        }
        if (a.pt) {
            wave_sync();
            spectrum_out<MT, QT>(cb, Q, r, g, a.pt + (i * (lmax + 1) + l) * int64_t(QQ));
        }
    };
    const int one = lmax < 7 ? lmax : 7;   // degrees whose columns fit one tile
    for (int l = 0; l <= one; ++l) degree(std::integral_constant<int, 1>{}, l);
    for (int l = 8; l <= lmax; ++l) degree(std::integral_constant<int, 2>{}, l);
}

template <int QT, int KS, int HT>
hipError_t launch_infer_t(const CompressArgs& a, const InferLayout& L, hipStream_t stream)
{
    auto kernel = k_cmp_infer<QT, KS, HT>;
    // (at most 51 KB of LDS: K = 128, lmax 12)
    hipLaunchKernelGGL(kernel, dim3(unsigned(a.n)), dim3(64), size_t(L.total), stream, a, L);
    return hipGetLastError();
}

template <int QT, int KS>
hipError_t launch_infer_h(const CompressArgs& a, const InferLayout& L, hipStream_t stream)
{
    return L.HT == 4 ? launch_infer_t<QT, KS, 4>(a, L, stream) : launch_infer_t<QT, KS, 8>(a, L, stream);
}

template <int QT>
hipError_t launch_infer_q(const CompressArgs& a, const InferLayout& L, hipStream_t stream)
{
    return L.KS == 1   ? launch_infer_h<QT, 1>(a, L, stream)
           : L.KS == 2 ? launch_infer_h<QT, 2>(a, L, stream)
           : L.KS == 3 ? launch_infer_h<QT, 3>(a, L, stream)
                       : launch_infer_h<QT, 4>(a, L, stream);
}

}  // namespace

size_t compress_image_bytes(int K, int Q, int H, int lmax)
{
    if (K > 128 || H > 128 || Q > 32 || lmax < 1 || lmax > 12 || K % 4 != 0 || H % 4 != 0) return 0;
    return size_t(lmax + 1) * infer_layout(K, Q, H, lmax).frags * 1024;
}

hipError_t launch_compress_infer(const CompressArgs& a, hipStream_t stream)
{
    const InferLayout L = infer_layout(a.K, a.Q, a.H, a.lmax);
    hipLaunchKernelGGL(k_cmp_image, dim3(unsigned((L.frags * 64 + 255) / 256), unsigned(a.lmax + 1)), dim3(256), 0, stream,
                       a, L);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return L.QT == 1 ? launch_infer_q<1>(a, L, stream) : launch_infer_q<2>(a, L, stream);
}

}  // namespace soap
