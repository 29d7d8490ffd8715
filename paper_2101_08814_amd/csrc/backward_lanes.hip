// Adjoint of the expansion with respect to positions with one or two lanes
// per pair.
//
// Adjoint (App. B Eq. energy-derivative), k_exp_backward_lanes: one wave per
// centre i, one lane per pair q = (i, j, s).  With G = dL/dc_i (the
// neighbour's species block, staged once per wave in LDS) the lane forms
//   A_lm = sum_n G_{n,lm} (f I~)'_nl,   B_lm = sum_n G_{n,lm} f I~_nl
// degree by degree while the harmonics of that degree come out of the
// recurrence, and
//   g_q = dL/dr_ji = u sum_lm A_lm Y_lm + sum_lm B_lm grad Y_lm
//       = u (sA - sL / r) + t / r,
//   sA = sum A Y, sL = sum l B Y, t = sum B grad Z
// (grad Y_lm = (grad Z_lm - l Y_lm u) / r).  Nothing per pair is staged and
// no lane decodes an index; the per-atom sums stay in the gather kernel of
// backward.hip.
//
// The cubics come a group of two at a time, the next group loading meanwhile,
// and the reads of G of a group's two rows go out together.  4096 centres of
// some 70 pairs at n=10, lmax=8 took 60 us with single cubics two ahead, and
// the wave waiting 55% of its cycles; 51 now, 33 of it vector instructions
// (at lmax 8 the launch bound keeps the second wave a SIMD: 79 us without).
//
// Where the registers leave one wave a SIMD, a chunk of at most 32 pairs gives
// each pair two lanes, 32 apart, each with half of the n: A, B and the five
// sums are linear in G, so the halves add at the end, and only the harmonics
// are formed twice.  1024 centres of 28 pairs at n=10, lmax=12 took 48 us,
// 42 with the groups, 32 with the halves (in double at lmax 8 36, 33 and 25).
// At lower degrees, where two waves and more hide each other's waits, the
// halves gain less (26.6, 22.1 and 19.1 at lmax 8 in float) and one lane keeps
// the order of the sum over n.  At lmax 9 in float the halves cost the second
// wave that whole pairs keep, so they serve while every centre has a SIMD to
// itself: 1024 centres of 28 pairs at n=9 take 21.1 us with them and 22.3
// without, 4096 76 and 50.  With one n there is nothing to halve, and the
// kernel without the code for it is the faster one (4096 centres at lmax 12:
// 49.9 and 46.9 us).  In double the groups of two cost the second wave at lmax
// 5 (4096 centres of 50 pairs at n=7: 48.7 us, 45.9 with single cubics); below
// they gain (16,384 of 28 at n=4, lmax=2: 46.5, singly 51.5).
#include "lane_pair.hpp"

namespace soap {
namespace {

using namespace dev;

// The degrees above which the registers leave one wave a SIMD.
template <typename T>
constexpr bool one_wave(int lmax) { return lmax > (sizeof(T) == 4 ? 8 : 5); }

// GR: cubics per group; HALVES: two lanes per pair in chunks of at most 32;
// WAVES: waves per SIMD that the registers keep
template <typename T, int LMAX, int GR, bool HALVES, int WAVES>
__global__ void __launch_bounds__(64, WAVES)
k_exp_backward_lanes(FeatureArgs a, const T* __restrict__ grad_c, T* __restrict__ grad_pair)
{
    constexpr int LM1 = LMAX + 1, L2 = LM1 * LM1;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* G = reinterpret_cast<T*>(smem_raw);
    const int lane = threadIdx.x;
    const int64_t i = blockIdx.x;
    if (a.pair_offsets[a.n_atoms] > a.pair_capacity) {
        if (lane == 0) put_status(a.status, SOAP_ECAPACITY);
        return;
    }
    const int nmax = a.nmax;
    const int nL2 = nmax * L2, KL2 = a.S * nL2;
    {
        const T* gi = grad_c + i * int64_t(KL2);
        for (int e0 = lane; e0 < KL2; e0 += 4 * 64) {
            T v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = e0 + 64 * u < KL2 ? gi[e0 + 64 * u] : T(0);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (e0 + 64 * u < KL2) G[e0 + 64 * u] = v[u];
        }
    }
    wave_sync();
    const int64_t qb = a.pair_offsets[i], qe = a.pair_offsets[i + 1];
    const V4<T>* __restrict__ coef = static_cast<const V4<T>*>(a.coef_ln);
    const T* __restrict__ vec = static_cast<const T*>(a.pair_vec);
    const T inv_delta = T(a.inv_delta);
    // pairs q0 .. q0 + np - 1, one lane each or (SPLIT) two
    auto chunk = [&](auto Split, int64_t q0, int np) __attribute__((always_inline)) {
        constexpr bool SPLIT = decltype(Split)::value;
        const int p = SPLIT ? lane & 31 : lane;
        const int64_t q = q0 + p;
        const bool live = p < np;
        const int64_t qq = live ? q : q0;   // the lanes past the chunk follow its first pair and write nothing
        const PairGeom<T> g = pair_geometry<T>(a, vec[3 * qq], vec[3 * qq + 1], vec[3 * qq + 2]);
        const int sp = pair_species(a, qq);
        // this lane's n: nb .. nb + cnt - 1 below nmax
        const int cnt = SPLIT ? (nmax + 1) >> 1 : nmax, nb = SPLIT && lane >= 32 ? cnt : 0;
        const T t3 = T(3) * g.t;
        const int full = SPLIT ? nmax >> 1 : nmax;   // both halves have that many
        const T* Gs = G + sp * nL2 + nb * L2;
        const V4<T>* cf = coef + int64_t(g.k) * (LM1 * nmax) + nb;
        YlmStream<T, LMAX> ys(g.ux, g.uy, g.uz);
        T sA = T(0), sL = T(0), tx = T(0), ty = T(0), tz = T(0);
        // the interval's cubics are contiguous ([l][n]; past a degree's end
        // the next one's, past the table's end its zeros, not used)
        V4<T> nxt[GR];
#pragma unroll
        for (int u = 0; u < GR; ++u) nxt[u] = cf[u];
        static_for<0, LM1>([&](auto Lc) __attribute__((always_inline)) {
            constexpr int L = decltype(Lc)::value;
            constexpr int NM = 2 * L + 1;
            T A[NM], B[NM];
#pragma unroll
            for (int m = 0; m < NM; ++m) A[m] = B[m] = T(0);
            const T* gr = Gs + L * L;
            for (int k0 = 0; k0 < cnt; k0 += GR) {
                V4<T> cur[GR];
#pragma unroll
                for (int u = 0; u < GR; ++u) cur[u] = nxt[u];
                if (k0 + GR < cnt || L < LMAX) {
                    const V4<T>* nx = cf + (k0 + GR < cnt ? L * nmax + k0 + GR : (L + 1) * nmax);
#pragma unroll
                    for (int u = 0; u < GR; ++u) nxt[u] = nx[u];
                }
                auto add = [&](int u) __attribute__((always_inline)) {
                    const V4<T> c = cur[u];
                    // the spline's value and slope with every rounding pinned,
                    // whichever way the loop around it is unrolled
                    const T v = fma(g.t, fma(g.t, fma(g.t, c.w, c.z), c.y), c.x);
                    const T dv = fma(g.t, fma(T(2), c.z, t3 * c.w), c.y) * inv_delta;
                    const T R = g.f * v, dR = fma(g.f, dv, g.df * v);
                    const T* gu = gr + (k0 + u) * L2;
#pragma unroll
                    for (int m = 0; m < NM; ++m) {
                        const T gv = gu[m];
                        A[m] = fma(gv, dR, A[m]);
                        B[m] = fma(gv, R, B[m]);
                    }
                };
                if (k0 + GR <= full) {
#pragma unroll
                    for (int u = 0; u < GR; ++u) add(u);
                } else {
#pragma unroll
                    for (int u = 0; u < GR; ++u)
                        if (k0 + u < cnt && (!SPLIT || nb + k0 + u < nmax)) add(u);
                }
            }
            T sB = T(0);
            ys.template degree<L, true>([&](int mi, T Y, T zx, T zy, T zz) __attribute__((always_inline)) {
                sA += A[mi] * Y;
                sB += B[mi] * Y;
                tx += B[mi] * zx;
                ty += B[mi] * zy;
                tz += B[mi] * zz;
            });
            sL += T(L) * sB;
        });
        if (SPLIT) {
            sA += __shfl_xor(sA, 32, 64);
            sL += __shfl_xor(sL, 32, 64);
            tx += __shfl_xor(tx, 32, 64);
            ty += __shfl_xor(ty, 32, 64);
            tz += __shfl_xor(tz, 32, 64);
        }
        const T radial = sA - sL * g.rinv;
        if (live && (!SPLIT || lane < 32)) {
            grad_pair[3 * q] = g.ux * radial + tx * g.rinv;
            grad_pair[3 * q + 1] = g.uy * radial + ty * g.rinv;
            grad_pair[3 * q + 2] = g.uz * radial + tz * g.rinv;
        }
    };
    for (int64_t q0 = qb; q0 < qe; q0 += 64) {
        const int np = qe - q0 < 64 ? int(qe - q0) : 64;
        if constexpr (HALVES) {
            if (np <= 32 && nmax > 1) {
                chunk(std::true_type{}, q0, np);
                continue;
            }
        }
        chunk(std::false_type{}, q0, np);
    }
}

template <typename T, int LM>
struct BackLanesFn {
    template <int GR, bool HALVES, int WAVES>
    static hipError_t launch(const FeatureArgs& a, const void* grad_c, void* grad_pair, hipStream_t st)
    {
        const size_t lds = size_t(a.S) * a.nmax * (LM + 1) * (LM + 1) * sizeof(T);
        auto kernel = k_exp_backward_lanes<T, LM, GR, HALVES, WAVES>;
        hipLaunchKernelGGL(kernel, dim3(unsigned(a.n_atoms)), dim3(64), lds, st, a, static_cast<const T*>(grad_c),
                           static_cast<T*>(grad_pair));
        return hipGetLastError();
    }
    static hipError_t run(const FeatureArgs& a, const void* grad_c, void* grad_pair, hipStream_t st)
    {
        constexpr bool f32 = sizeof(T) == 4;
        if constexpr (LM < 0) {
            return hipErrorNotSupported;
        } else if constexpr (!one_wave<T>(LM)) {
            return launch<f32 || LM < 5 ? 2 : 1, false, 2>(a, grad_c, grad_pair, st);
        } else {
            if constexpr (f32 && LM == 9) {
                if (a.n_atoms > 1024 || a.nmax == 1) return launch<2, false, 2>(a, grad_c, grad_pair, st);
            }
            if constexpr (f32 && LM > 9) {
                if (a.nmax == 1) return launch<1, false, 1>(a, grad_c, grad_pair, st);
            }
            return launch<2, true, 1>(a, grad_c, grad_pair, st);
        }
    }
};

}  // namespace

bool expansion_backward_lanes_fits(const FeatureArgs& a, bool f64)
{
    const size_t lds = size_t(a.S) * a.nmax * (a.lmax + 1) * (a.lmax + 1) * (f64 ? 8 : 4);
    return lds <= 64 * 1024;
}

hipError_t launch_expansion_backward_lanes(const FeatureArgs& a, bool f64, const void* grad_c, void* grad_pair,
                                           hipStream_t stream)
{
    if (!expansion_backward_lanes_fits(a, f64)) return hipErrorNotSupported;
    if (a.n_atoms == 0) return hipSuccess;
    return f64 ? by_degree<double, BackLanesFn>(a.lmax, a, grad_c, grad_pair, stream)
               : by_degree<float, BackLanesFn>(a.lmax, a, grad_c, grad_pair, stream);
}

}  // namespace soap
