// The compression network in float on the FP32 matrix cores: forward pass
// and weight gradient (training, and inference without bfloat16) for
// K, H <= 128 channels and hidden units and Q <= 32 outputs.
//
// Every product of degree l is a small matrix times the columns (centre, m)
// of a group of centres: G centres with G (2l+1) <= 32 columns per group
// (G <= 8), two tiles of 16.  A work-group of four waves takes groups of one
// degree in turn and keeps that degree's weights in registers as MFMA
// operands (v_mfma_f32_16x16x4_f32: lane (r, g) = (lane & 15, lane >> 4)
// supplies A[r][g], B[g][r] and holds D[4g + v][r]; step s of a 16-wide
// chunk of the inner dimension takes index 4g + s on both sides).  Wave w
// owns the hidden tiles w and w + 4.  Per group:
//   X    [column][k]            c_{k,lm} in LDS
//   h    = W1 X                 -> LDS [hidden][column]
//   g    = h 2 sigma(alpha |h| + beta), one lane per (unit, centre)
//   c~   = W2 g                 -> LDS [output][column]
// forward: p~ of each centre from c~; backward, with G~ the symmetric
// unpacking of dL/dp~ (doubled diagonal):
//   dc~  = G~ c~                one lane per (column, output)
//   dW2 += dc~ g^T,  dg = W2^T dc~
//   dh   from dg through the gate (|h| and sigma formed again)
//   dW1 += dh X^T
// dW1 and dW2 stay in registers as accumulators over all groups of the
// work-group and leave as one partial sum; k_train_reduce adds the partial
// sums of a degree in order, so results are bitwise reproducible.
//
// The flops are few (0.4 GFLOP forward, 1.1 backward for 512 centres at
// K = 72, H = 128, Q = 32, lmax 6); the kernels are bound by the latency of
// the chain of products and barriers, which two work-groups per CU share
// (80 KB of LDS at the largest shape).  The form before (one work-group per
// centre or per (degree, slice), one lane per output looping over scalar
// products from global memory) took 329 us forward and 1518 us backward for
// that batch; now 45 and 95 us, and 7.5 us for adding the partial sums
// (17 us before, 64 serial loads per lane).  That form is kept (compress.hip)
// for the shapes whose operands do not fit here, K or H over 128, Q over 32,
// and for small networks of many centres, which these tiles pad.
#include "soap_internal.hpp"

namespace soap {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kCols = 32;        // columns of a group
constexpr int kMaxG = 8;         // centres of a group
constexpr int kHid = 128;        // hidden units, at most
constexpr int kHS = kCols + 1;   // row stride of the [hidden][column] arrays (odd: rows on distinct banks)
constexpr int kCS = kCols + 4;   // row stride of the [output][column] arrays

// work-groups first[l] .. first[l + 1] take the groups of degree l
struct TrainPlan {
    int g[13];        // centres per group
    int first[14];
    int64_t per;      // groups per work-group
};

struct TrainLayout {
    int xs, x, h, gb, ct, dct, gp, total;   // row stride of X, offsets in floats
};

__host__ __device__ inline TrainLayout train_layout(int KT, int Q, bool bwd)
{
    const int QP = (Q + 15) / 16 * 16;
    TrainLayout L;
    L.xs = KT * 16 + 4;
    int o = 0;
    L.x = o; o += kCols * L.xs;
    L.ct = o; o += QP * kCS;
    L.dct = o; o += bwd ? QP * kCS : 0;
    L.gp = o; o += bwd ? (kMaxG * (Q * (Q + 1) / 2) + 3) / 4 * 4 : 0;
    L.h = o; o += kHid * kHS;
    L.gb = o; o += bwd ? kHid * kHS : 0;
    L.total = o;
    return L;
}

__device__ __forceinline__ float sigm(float x) { return 1.0f / (1.0f + expf(-x)); }

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// KT: tiles of 16 input channels (K <= 16 KT); QT: tiles of 16 outputs
template <bool BWD, int KT, int QT>
__global__ void __launch_bounds__(256, 2) k_train(CompressArgs a, TrainPlan pl)
{
    extern __shared__ __align__(16) float sm[];
    const int K = a.K, Q = a.Q, H = a.H, lmax = a.lmax, L2 = (lmax + 1) * (lmax + 1);
    const int QQ = Q * (Q + 1) / 2, tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const TrainLayout L = train_layout(KT, Q, BWD);
    float* X = sm + L.x;
    float* hb = sm + L.h;
    float* gb = BWD ? sm + L.gb : hb;   // g (forward: in place of h), then dg and dh
    float* ct = sm + L.ct;
    float* dct = sm + L.dct;
    float* gp = sm + L.gp;

    int l = 0;
    while (int(blockIdx.x) >= pl.first[l + 1]) ++l;
    const int M = 2 * l + 1, b = l * l, G = pl.g[l];
    const int64_t groups = (a.n + G - 1) / G;
    const int64_t lo = (int64_t(blockIdx.x) - pl.first[l]) * pl.per;
    const int64_t hi = lo + pl.per < groups ? lo + pl.per : groups;
    const int64_t lsize = int64_t(H) * K + Q * H + 2 * H;
    const float* W1 = a.w + l * lsize;
    const float* W2 = W1 + H * K;
    const float* al = W2 + Q * H;
    const float* be = al + H;

    // the degree's weights as operands, zero outside the matrices
    f32x4 w1[2][KT], w2[kHid / 16];
    float w2t[2][4 * QT];
    const int pt = QT > 1 ? wave >> 1 : 0, cw = wave & 1;   // this wave's tile of c~ (QT = 1: waves 0 and 1)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int q = 16 * (wave + 4 * t) + r;
#pragma unroll
        for (int c = 0; c < KT; ++c)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = 16 * c + 4 * g + s;
                w1[t][c][s] = q < H && k < K ? W1[q * K + k] : 0.0f;
            }
        if (BWD)
#pragma unroll
            for (int c = 0; c < QT; ++c)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int p = 16 * c + 4 * g + s;
                    w2t[t][4 * c + s] = q < H && p < Q ? W2[p * H + q] : 0.0f;
                }
    }
#pragma unroll
    for (int c = 0; c < kHid / 16; ++c)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int p = 16 * pt + r, q = 16 * c + 4 * g + s;
            w2[c][s] = p < Q && q < H ? W2[p * H + q] : 0.0f;
        }
    const int hq = tid & (kHid - 1), half = tid >> 7;   // gate: this lane's unit, centres half, half + 2, ...
    const float alq = hq < H ? al[hq] : 0.0f, beq = hq < H ? be[hq] : 0.0f;

    f32x4 dw1[2][KT], dw2[2][QT];
    float gal = 0.0f, gbe = 0.0f;
    if (BWD) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int c = 0; c < KT; ++c) dw1[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < QT; ++c) dw2[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        for (int e = tid; e < QT * 16 * kCS; e += 256) dct[e] = 0.0f;   // rows past Q stay zero
    }
    // forward: the packed outputs of this lane
    int pq1[3], pq2[3];
    if (!BWD) {
        int t = tid, q1 = 0, start = 0;   // start: packed position of (q1, q1)
#pragma unroll
        for (int u = 0; u < 3; ++u, t += 256) {
            while (q1 < Q && t >= start + Q - q1) {
                start += Q - q1;
                ++q1;
            }
            pq1[u] = q1;
            pq2[u] = q1 + (t - start);
        }
    }

    const int col = tid & (kCols - 1), kr = tid >> 5;   // staging: this lane's column, channels kr, kr + 8, ...
    const int ic_col = col / M, m_col = col - ic_col * M;
    for (int64_t gr = lo; gr < hi; ++gr) {
        const int64_t i0 = gr * G;
        const int nc = a.n - i0 < G ? int(a.n - i0) : G;
        // X, and the upstream gradient of the group's centres
        {
            const bool in = ic_col < nc;
            const float* src = a.c + (i0 + (in ? ic_col : 0)) * int64_t(K) * L2 + b + m_col;
            float v[2 * KT];
#pragma unroll
            for (int u = 0; u < 2 * KT; ++u) {
                const int k = kr + 8 * u;
                v[u] = in && k < K ? src[k * L2] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 2 * KT; ++u) X[col * L.xs + kr + 8 * u] = v[u];
        }
        if (BWD)
            for (int ic = 0; ic < nc; ++ic) {
                const float* src = a.gpt + ((i0 + ic) * (lmax + 1) + l) * int64_t(QQ);
                for (int t = tid; t < QQ; t += 256) gp[ic * QQ + t] = src[t];
            }
        __syncthreads();
        // h
        {
            f32x4 acc[2][2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < KT; ++c) {
                f32x4 x[2];
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    x[j] = *reinterpret_cast<const f32x4*>(&X[(16 * j + r) * L.xs + 16 * c + 4 * g]);
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int j = 0; j < 2; ++j) acc[t][j] = mfma(w1[t][c][s], x[j][s], acc[t][j]);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int q = 16 * (wave + 4 * t) + 4 * g + v;
                        const float hv = q < H ? acc[t][j][v] : 0.0f;
                        hb[q * kHS + 16 * j + r] = hv;
                        if (BWD) gb[q * kHS + 16 * j + r] = hv;
                    }
        }
        __syncthreads();
        // g
        if (hq < H)
            for (int ic = half; ic < nc; ic += 2) {
                const float* hc = hb + hq * kHS + ic * M;
                float* gc = gb + hq * kHS + ic * M;
                float s = 0.0f;
                for (int m = 0; m < M; ++m) s += hc[m] * hc[m];
                const float f = 2.0f * sigm(alq * sqrtf(s) + beq);
                for (int m = 0; m < M; ++m) gc[m] = f * hc[m];
            }
        __syncthreads();
        // c~
        if (QT > 1 || wave < 2) {
            f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int c = 0; c < kHid / 16; ++c)
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    acc[s & 1] = mfma(w2[c][s], gb[(16 * c + 4 * g + s) * kHS + 16 * cw + r], acc[s & 1]);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int p = 16 * pt + 4 * g + v;
                ct[p * kCS + 16 * cw + r] = acc[0][v] + acc[1][v];
            }
        }
        __syncthreads();
        if (!BWD) {
            if (a.ct)
                for (int e = tid; e < Q * nc * M; e += 256) {
                    const int p = e / (nc * M), cm = e - p * (nc * M), ic = cm / M, m = cm - ic * M;
                    a.ct[((i0 + ic) * Q + p) * L2 + b + m] = ct[p * kCS + cm];
                }
            if (a.pt)
                for (int ic = 0; ic < nc; ++ic) {
                    float* out = a.pt + ((i0 + ic) * (lmax + 1) + l) * int64_t(QQ);
#pragma unroll
                    for (int u = 0; u < 3; ++u) {
                        if (tid + 256 * u >= QQ) continue;
                        const float* c1 = ct + pq1[u] * kCS + ic * M;
                        const float* c2 = ct + pq2[u] * kCS + ic * M;
                        float s = 0.0f;
                        for (int m = 0; m < M; ++m) s += c1[m] * c2[m];
                        out[tid + 256 * u] = s;
                    }
                }
            __syncthreads();   // c~ and X are written again
            continue;
        }
        // dc~_{p,col} = sum_q G~_pq c~_{q,col}: the packed position of (q, p)
        // grows by Q - q - 1 from q to q + 1 below the diagonal, by 1 above
        for (int p = tid >> 5; p < Q; p += 8) {
            float s = 0.0f;
            if (ic_col < nc) {
                const float* gc = gp + ic_col * QQ;
                int at = p;
                for (int q = 0; q < p; ++q) {
                    s += gc[at] * ct[q * kCS + col];
                    at += Q - q - 1;
                }
                s += 2.0f * gc[at] * ct[p * kCS + col];
                for (int q = p + 1; q < Q; ++q) s += gc[++at] * ct[q * kCS + col];
            }
            dct[p * kCS + col] = s;
        }
        __syncthreads();
        // dW2 += dc~ g^T and dg = W2^T dc~
        f32x4 dg[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j) dg[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < kCols / 16; ++c) {
            f32x4 d[QT];
#pragma unroll
            for (int p = 0; p < QT; ++p)
                d[p] = *reinterpret_cast<const f32x4*>(&dct[(16 * p + r) * kCS + 16 * c + 4 * g]);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float gv = gb[(16 * (wave + 4 * t) + r) * kHS + 16 * c + 4 * g + s];
#pragma unroll
                    for (int p = 0; p < QT; ++p) dw2[t][p] = mfma(d[p][s], gv, dw2[t][p]);
                }
        }
#pragma unroll
        for (int c = 0; c < QT; ++c)
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const float d = dct[(16 * c + 4 * g + s) * kCS + 16 * j + r];
#pragma unroll
                    for (int t = 0; t < 2; ++t) dg[t][j] = mfma(w2t[t][4 * c + s], d, dg[t][j]);
                }
        // a wave reads and writes only its own units' rows of gb here
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    gb[(16 * (wave + 4 * t) + 4 * g + v) * kHS + 16 * j + r] = dg[t][j][v];
        __syncthreads();
        // through the gate: g = 2 s h, s = sigma(alpha |h| + beta)
        if (hq < H)
            for (int ic = half; ic < nc; ic += 2) {
                const float* hc = hb + hq * kHS + ic * M;
                float* dc = gb + hq * kHS + ic * M;
                float ss = 0.0f, dG = 0.0f;
                for (int m = 0; m < M; ++m) {
                    ss += hc[m] * hc[m];
                    dG += dc[m] * hc[m];
                }
                const float nrm = sqrtf(ss), s = sigm(alq * nrm + beq);
                const float dz = dG * 2.0f * s * (1.0f - s);
                gal += dz * nrm;
                gbe += dz;
                const float cf = nrm > 0.0f ? dz * alq / nrm : 0.0f;
                for (int m = 0; m < M; ++m) dc[m] = dc[m] * (2.0f * s) + cf * hc[m];
            }
        __syncthreads();
        // dW1 += dh X^T
#pragma unroll
        for (int c = 0; c < kCols / 4; ++c) {
            const int cc = 4 * c + g;
            float d[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) d[t] = gb[(16 * (wave + 4 * t) + r) * kHS + cc];
#pragma unroll
            for (int k = 0; k < KT; ++k) {
                const float x = X[cc * L.xs + 16 * k + r];
#pragma unroll
                for (int t = 0; t < 2; ++t) dw1[t][k] = mfma(d[t], x, dw1[t][k]);
            }
        }
        __syncthreads();   // X, gp and the h arrays are written again
    }
    if (!BWD) return;
    float* out = a.gpart + int64_t(blockIdx.x) * lsize;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int c = 0; c < KT; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int q = 16 * (wave + 4 * t) + 4 * g + v, k = 16 * c + r;
                if (q < H && k < K) out[q * K + k] = dw1[t][c][v];
            }
#pragma unroll
        for (int p = 0; p < QT; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int pp = 16 * p + 4 * g + v, q = 16 * (wave + 4 * t) + r;
                if (pp < Q && q < H) out[H * K + pp * H + q] = dw2[t][p][v];
            }
    }
    // the two halves of each unit's gate gradients
    float* red = sm + L.ct;   // at least 16 kCS >= 4 kHid floats
    red[tid] = gal;
    red[256 + tid] = gbe;
    __syncthreads();
    if (tid < H) {
        out[H * K + Q * H + tid] = red[tid] + red[tid + kHid];
        out[H * K + Q * H + H + tid] = red[256 + tid] + red[256 + tid + kHid];
    }
}

// adds the partial sums of a degree's work-groups in order
__global__ void __launch_bounds__(256) k_train_reduce(TrainPlan pl, int lmax, int64_t lsize, const float* part,
                                                      float* out)
{
    const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
    const int l = blockIdx.y;
    if (e >= lsize) return;
    const float* src = part + int64_t(pl.first[l]) * lsize + e;
    const int n = pl.first[l + 1] - pl.first[l];
    float s = 0.0f;
    int k = 0;
    for (; k + 8 <= n; k += 8) {   // eight loads in flight
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[(k + u) * lsize];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; k < n; ++k) s += src[k * lsize];
    out[l * lsize + e] = s;
}

bool train_fits(const CompressArgs& a) { return a.K <= 128 && a.H <= kHid && a.Q <= 32; }

// work-groups: at most `want` (and, for the gradient, the workspace's
// partial sums), every one with the same number of groups
TrainPlan train_plan(const CompressArgs& a, int64_t want)
{
    TrainPlan pl;
    int64_t groups[13], total = 0;
    for (int l = 0; l <= a.lmax; ++l) {
        const int g = kCols / (2 * l + 1);
        pl.g[l] = g < kMaxG ? g : kMaxG;
        groups[l] = (a.n + pl.g[l] - 1) / pl.g[l];
        total += groups[l];
    }
    pl.per = (total + want - 1) / want;
    if (pl.per < 1) pl.per = 1;
    for (;; ++pl.per) {
        int64_t o = 0;
        for (int l = 0; l <= a.lmax; ++l) {
            pl.first[l] = int(o);
            o += (groups[l] + pl.per - 1) / pl.per;
        }
        for (int l = a.lmax + 1; l < 14; ++l) pl.first[l] = int(o);
        if (o <= want) return pl;
    }
}

template <bool BWD, int KT, int QT>
hipError_t launch_train_t(const CompressArgs& a, const TrainPlan& pl, hipStream_t stream)
{
    const int blocks = pl.first[a.lmax + 1];
    if (blocks == 0) return hipSuccess;
    const int lds = train_layout(KT, a.Q, BWD).total * int(sizeof(float));
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_train<BWD, KT, QT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_train<BWD, KT, QT>), dim3(unsigned(blocks)), dim3(256), size_t(lds), stream, a,
                       pl);
    return hipGetLastError();
}

template <bool BWD, int QT>
hipError_t launch_train_q(const CompressArgs& a, const TrainPlan& pl, hipStream_t stream)
{
    const int kt = (a.K + 15) / 16;
    if (kt <= 2) return launch_train_t<BWD, 2, QT>(a, pl, stream);
    if (kt <= 4) return launch_train_t<BWD, 4, QT>(a, pl, stream);
    if (kt <= 5) return launch_train_t<BWD, 5, QT>(a, pl, stream);
    if (kt <= 6) return launch_train_t<BWD, 6, QT>(a, pl, stream);
    return launch_train_t<BWD, 8, QT>(a, pl, stream);
}

}  // namespace

hipError_t launch_train_forward(const CompressArgs& a, hipStream_t stream)
{
    if (!train_fits(a)) return hipErrorNotSupported;
    // four work-groups per CU at most; more groups than that loop
    const TrainPlan pl = train_plan(a, 1024);
    return a.Q <= 16 ? launch_train_q<false, 1>(a, pl, stream) : launch_train_q<false, 2>(a, pl, stream);
}

hipError_t launch_train_backward(const CompressArgs& a, float* grad, hipStream_t stream)
{
    if (!train_fits(a)) return hipErrorNotSupported;
    // two work-groups per CU, within the partial sums the workspace holds
    // (a.slices per degree on average)
    const int64_t room = int64_t(a.slices) * (a.lmax + 1);
    const TrainPlan pl = train_plan(a, room < 512 ? room : 512);
    hipError_t e = a.Q <= 16 ? launch_train_q<true, 1>(a, pl, stream) : launch_train_q<true, 2>(a, pl, stream);
    if (e != hipSuccess) return e;
    const int64_t lsize = int64_t(a.H) * a.K + int64_t(a.Q) * a.H + 2 * int64_t(a.H);
    hipLaunchKernelGGL(k_train_reduce, dim3(unsigned((lsize + 255) / 256), unsigned(a.lmax + 1)), dim3(256), 0, stream, pl,
                       a.lmax, lsize, a.gpart, grad);
    return hipGetLastError();
}

}  // namespace soap
