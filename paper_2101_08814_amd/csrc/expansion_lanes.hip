// Spherical expansion and power spectrum of a centre by one to four waves.
//
// Expansion (Sec. 4.A Eq. spherical_expansion_coefficients_gaussians, Sec.
// 4.F), k_expansion_lanes: one work-group of one, two or four waves per
// centre.  For a chunk of up to 64 of its pairs, one to sixteen lanes per
// pair form its harmonics Y_lm and radial values R_nl = f I~_nl in registers
// and put them in the centre's LDS rows; then each lane owns items (four n,
// one lm) of a species block and sums R_{n..n+3,l} Y_lm over the pairs of that
// species (one 16-byte and one 4-byte LDS read per four FMAs).  Pairs arrive
// grouped by neighbour species (the order soap_compute_neighbors writes), so a
// block is complete when the species changes and is written then; a list that
// is not grouped is detected and the centre is redone one species at a time.
// The blocks stay in LDS as a copy of c_i, and the power spectrum
// p_{l,k1<=k2} = sum_m c_{k1,lm} c_{k2,lm} (Sec. 2 Eq. nu2-basis-coupled up
// to the factor of reading R4) is formed from it, one lane per (k1, k2).
// Each output element has one owner: no atomics.
#include "lane_pair.hpp"

namespace soap {
namespace {

using namespace dev;

// ------------------------------------------------------------- expansion
template <typename T, int LMAX, int NW>
__global__ void __launch_bounds__(64 * NW) k_expansion_lanes(FeatureArgs a, LaneLayout W)
{
    constexpr int LM1 = LMAX + 1, L2 = LM1 * LM1;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* base = reinterpret_cast<T*>(smem_raw);
    T* Rs = base + W.rs;
    T* Ys = base + W.ys;
    T* Cs = base + W.cs;
    constexpr int NT = 64 * NW;
    const int tid = threadIdx.x, lane = tid & 63;
    auto sync = [&]() __attribute__((always_inline)) {
        if constexpr (NW == 1) wave_sync();
        else __syncthreads();
    };
    const int64_t i = blockIdx.x;
    if (a.pair_offsets[a.n_atoms] > a.pair_capacity) {
        if (tid == 0) put_status(a.status, SOAP_ECAPACITY);
        return;
    }
    const int nmax = a.nmax, S = a.S;
    const int nL2 = nmax * L2, KL2 = S * nL2;
    const int NI = ((nmax + 3) >> 2) * L2;
    const int nl = LM1 * nmax;
    const int64_t qb = a.pair_offsets[i], qe = a.pair_offsets[i + 1];
    const T* __restrict__ centre_term = static_cast<const T*>(a.center);
    const V4<T>* __restrict__ coef = static_cast<const V4<T>*>(a.coef_ln);
    const T* __restrict__ vec = static_cast<const T*>(a.pair_vec);
    int sp_i = -1;
    if (a.include_center) {
        sp_i = a.species[i];
        if (sp_i < 0 || sp_i >= S) {
            if (tid == 0) put_status(a.status, SOAP_ESPECIES);
            sp_i = -1;
        }
    }
    T* c_out = static_cast<T*>(a.coeffs) + i * int64_t(KL2);

    // Items (n group ng, lm), v = ng L2 + lm < NI: the four sums over n =
    // 4 ng..4 ng+3 of one lm, held in the block buffer blk4[v] (LDS) of the
    // species being summed; a lane takes items lane, lane + 64, ...
    V4<T>* const cs4 = reinterpret_cast<V4<T>*>(Cs);
    auto zero_blocks = [&]() __attribute__((always_inline)) {
        for (int v = tid; v < S * NI; v += NT) cs4[v] = V4<T>{T(0), T(0), T(0), T(0)};
    };
    // species block sp of c to HBM with consecutive lanes on consecutive
    // addresses; the central atom adds its term to lm = 0 of its own species
    // on the way, and to the LDS copy
    auto flush = [&](int sp) __attribute__((always_inline)) {
        T* b1 = reinterpret_cast<T*>(cs4 + sp * NI);
        sync();
        T* dst = c_out + sp * nL2;
        const bool own = sp == sp_i;
        for (int e = tid; e < nL2; e += NT) {
            const int n = e / L2, lm = e - n * L2;
            T* src = b1 + ((n >> 2) * L2 + lm) * 4 + (n & 3);
            T v = *src;
            if (own && lm == 0) {
                v += centre_term[n];
                *src = v;
            }
            dst[e] = v;
        }
        sync();
    };
    // the chunk's pairs [lo, hi) of species sp added to its block: per item
    // and pair one 4-byte and one 16-byte LDS read and four FMAs
    auto accumulate = [&](int sp, int lo, int hi) __attribute__((always_inline)) {
        V4<T>* blk = cs4 + sp * NI;
        for (int v = tid; v < NI; v += NT) {
            const int ng = v / L2, lm = v - ng * L2;
            V4<T> s4 = blk[v];
            const T* yp = Ys + lo * W.l2s + lm;
            const T* rp = Rs + lo * W.nls + l_of(lm) * W.np + 4 * ng;
#pragma unroll 4
            for (int p = lo; p < hi; ++p) {
                const T Y = yp[0];
                const V4<T> R = *reinterpret_cast<const V4<T>*>(rp);
                s4.x += R.x * Y;
                s4.y += R.y * Y;
                s4.z += R.z * Y;
                s4.w += R.w * Y;
                yp += W.l2s;
                rp += W.nls;
            }
            blk[v] = s4;
        }
    };
    zero_blocks();

    // Stages pairs q0 .. q0 + nc - 1 (harmonics and radial values in their
    // LDS rows); lane p < nc of every wave returns pair p's neighbour's
    // species (the other lanes' values mean nothing).  A pair takes one, two
    // or four lanes per wave, side by side: all of them run the harmonics (the
    // first writes them), and each forms its share of the radial values, so
    // that a chunk of few pairs does not leave most of the wave idle along one
    // lane's chain of loads.
    // The radial values are formed four n at a time: quad j = l G + n / 4 of
    // the G = np / 4 quads of every degree sits at 4 j of the pair's row
    // [l][np], its cubics at 4 j - l (np - nmax) of the interval's block
    // [l][nmax] (l = (j ceil(2^16 / G)) >> 16, exact for j < 2^12).  They
    // stream with two quads in flight, one consumed after each degree of
    // harmonics.  The quad of a degree's end may run into the next degree's
    // cubics, or the table's 32 zero entries past its end; what it puts past
    // nmax is not used.
    // One lane per pair with two batches of eight values took 38.2 us for
    // 1024 centres of 28 pairs at n=10, lmax=12 (chunks of 16 pairs by LDS),
    // with the shares of one wave 30.2, and 63.6 and 46.9 for 2048 centres of
    // 45 pairs at n=10, lmax=8, where the chunks of 32 take the wave's two
    // halves; two quads a step: 31.9 and 49.7, three: 33.7 and 50.4.
    const int rpad = W.np - nmax, G = W.np >> 2, QN = LM1 * G, rmul = (65536 + G - 1) / G;
    auto stage = [&](int64_t q0, int nc) __attribute__((always_inline)) -> int {
        constexpr int W0 = NW == 4 ? 2 : NW == 2 ? 1 : 0;
        const int sh = W0 + (nc <= 16 ? 2 : nc <= 32 ? 1 : 0);
        const int p = tid >> sh, part = tid & ((1 << sh) - 1);
        if (p < nc) {
            const int64_t q = q0 + p;
            const PairGeom<T> g = pair_geometry<T>(a, vec[3 * q], vec[3 * q + 1], vec[3 * q + 2]);
            const V4<T>* cf = coef + int64_t(g.k) * nl;
            T* yrow = Ys + p * W.l2s;
            T* rrow = Rs + p * W.nls;
            // (the place in the interval with one rounding, whatever is around it)
            const T tt = fma(g.r, T(a.inv_delta), -T(g.k)), f = g.f;
            // quad j, or quad 0 past the last one
            auto load = [&](V4<T>* c, int j) __attribute__((always_inline)) {
                const int jj = j < QN ? j : 0;
                const V4<T>* cj = cf + 4 * jj - rpad * ((jj * rmul) >> 16);
#pragma unroll
                for (int u = 0; u < 4; ++u) c[u] = cj[u];
            };
            const int step = 1 << sh;
            V4<T> A[4], B[4];
            load(A, part);
            load(B, part + step);
            int jb = 0;   // the first of the quads that the pair's lanes take now
            auto consume = [&]() __attribute__((always_inline)) {
                const int j = jb + part;
                T v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const V4<T> c = A[u];
                    v[u] = f * (c.x + tt * (c.y + tt * (c.z + tt * c.w)));
                    A[u] = B[u];
                }
                load(B, j + 2 * step);
                if (j < QN) *reinterpret_cast<V4<T>*>(rrow + 4 * j) = V4<T>{v[0], v[1], v[2], v[3]};
                jb += step;
            };
            YlmStream<T, LMAX> ys(g.ux, g.uy, g.uz);
            static_for<0, LM1>([&](auto Lc) __attribute__((always_inline)) {
                constexpr int L = decltype(Lc)::value;
                T Yd[2 * L + 1];
                ys.template degree<L, false>([&](int mi, T Y, T, T, T) __attribute__((always_inline)) { Yd[mi] = Y; });
                if (part == 0) {
#pragma unroll
                    for (int m = 0; m < 2 * L + 1; ++m) yrow[L * L + m] = Yd[m];
                }
                if (jb < QN) consume();
            });
            while (jb < QN) consume();
        }
        const int my_sp = pair_species(a, q0 + (lane < nc ? lane : 0));   // the same in every wave
        sync();
        return my_sp;
    };

    // Grouped pass: blocks written as the species changes.  A chunk whose
    // species decrease anywhere (or start below the current block) marks
    // the centre as not grouped.
    int cur = 0;
    bool grouped = true;
    for (int64_t q0 = qb; q0 < qe && grouped; q0 += W.ch) {
        const int nc = int(qe - q0 < W.ch ? qe - q0 : W.ch);
        const int my_sp = stage(q0, nc);
        const int prev = __shfl_up(my_sp, 1, 64);
        const bool bad = lane < nc && my_sp < (lane == 0 ? cur : prev);
        if (__ballot(bad)) {
            grouped = false;
            break;
        }
        for (int lo = 0; lo < nc;) {
            const int sp = __builtin_amdgcn_readlane(my_sp, lo);
            const int cnt = __popcll(__ballot(lane < nc && my_sp == sp));
            while (cur < sp) {
                flush(cur);
                ++cur;
            }
            accumulate(sp, lo, lo + cnt);
            lo += cnt;
        }
        sync();
    }
    if (grouped) {
        for (int sp = cur; sp < S; ++sp) flush(sp);
    } else {
        // pairs not grouped by species: every block, one species per pass
        zero_blocks();
        for (int sp = 0; sp < S; ++sp) {
            for (int64_t q0 = qb; q0 < qe; q0 += W.ch) {
                const int nc = int(qe - q0 < W.ch ? qe - q0 : W.ch);
                const int my_sp = stage(q0, nc);
                for (int p = 0; p < nc; ++p)
                    if (__builtin_amdgcn_readlane(my_sp, p) == sp) accumulate(sp, p, p + 1);
                sync();
            }
            flush(sp);
        }
    }
    sync();
    const int K = S * nmax, KK = K * (K + 1) / 2;
    T* p_out = static_cast<T*>(a.p) + i * int64_t(LM1 * KK);
    for (int kk = tid; kk < KK; kk += NT) {
        int k1, k2;
        tri_decode(K, kk, k1, k2);
        // c_{k, lm} sits at ((ng L2 + lm) 4 + n % 4) of species a's block
        const int s1 = k1 / nmax, n1 = k1 - s1 * nmax, s2 = k2 / nmax, n2 = k2 - s2 * nmax;
        const T* c1 = Cs + (s1 * NI + (n1 >> 2) * L2) * 4 + (n1 & 3);
        const T* c2 = Cs + (s2 * NI + (n2 >> 2) * L2) * 4 + (n2 & 3);
        static_for<0, LM1>([&](auto Lc) __attribute__((always_inline)) {
            constexpr int L = decltype(Lc)::value;
            T s = T(0);
#pragma unroll
            for (int m = L * L; m < (L + 1) * (L + 1); ++m) s += c1[4 * m] * c2[4 * m];
            p_out[L * KK + kk] = s;
        });
    }
}

template <typename T, int LM, int NW>
hipError_t launch_lanes(const FeatureArgs& a, const LaneLayout& W, hipStream_t st)
{
    auto kernel = k_expansion_lanes<T, LM, NW>;
    hipLaunchKernelGGL(kernel, dim3(unsigned(a.n_atoms)), dim3(64 * NW), size_t(W.total) * sizeof(T), st, a, W);
    return hipGetLastError();
}

// Waves per centre for c and p: with one, fewer than 4096 centres leave most
// of the chip's waves empty and each centre's sums and products run as one
// chain.  Two are faster than one (4000 centres of 45 pairs at n=10, lmax=8:
// 85 and 72 us, double 190 and 165; 1024 of 28 at n=10, lmax=12: 30.2 and
// 25.8), four only while a CU has few centres: 21 centres of four species at
// n=8, lmax=6 take 19.0 us with one, 13.4 with two and 11.2 with four, 512
// float ones at n=9, lmax=6 15.8, 12.5 and 10.2, but 512 in double at n=6,
// lmax=4 10.8, 10.0 and 10.3, and the 1024 above 33.2.  One is enough where it
// has an item for every lane and the centres are many: 3000 in double of 50
// pairs and two species at n=6, lmax=4 (50 items) take 38.8 and 46.1 us with
// one and two, 2000 33.7 and 33.0; in float two still hide each other's waits
// there (3000: 23.3 and 19.1) but not with a quarter of a wave's items (3000 of
// eight species at n=4, lmax=3: 28.0 and 31.3).
constexpr int64_t kFourWavesBytes = 2048;   // four waves up to that many centres times the element's size
constexpr int64_t kOneWaveAtoms = 2500;     // one from that many centres, for at most kOneWaveItems items a species
template <typename T>
constexpr int kOneWaveItems = sizeof(T) == 8 ? 64 : 16;

template <typename T, int LM>
struct LanesFn {
    static hipError_t run(const FeatureArgs& a, const LaneLayout& W, hipStream_t st)
    {
        if constexpr (LM < 0) {
            return hipErrorNotSupported;
        } else {
            if constexpr ((LM + 1) * (LM + 1) <= kOneWaveItems<T>) {
                if (a.n_atoms >= kOneWaveAtoms && (W.np >> 2) * (LM + 1) * (LM + 1) <= kOneWaveItems<T>)
                    return launch_lanes<T, LM, 1>(a, W, st);
            }
            return a.n_atoms * int64_t(sizeof(T)) <= kFourWavesBytes ? launch_lanes<T, LM, 4>(a, W, st)
                                                                     : launch_lanes<T, LM, 2>(a, W, st);
        }
    }
};

}  // namespace

LaneLayout lane_layout(int S, int nmax, int lmax, int ch)
{
    LaneLayout W{};
    const int lm1 = lmax + 1, L2 = lm1 * lm1;
    W.ch = ch;
    W.np = (nmax + 3) & ~3;
    W.nls = lm1 * W.np;
    W.l2s = L2 | 1;
    int o = 0;
    W.rs = o; o += ch * W.nls;
    W.ys = o; o += ch * W.l2s;
    o = (o + 3) & ~3;
    W.cs = o; o += S * W.np * L2;
    W.total = o;
    return W;
}

// Largest chunk (64, 32 or 16 pairs) whose LDS keeps at least six centres'
// work-groups per CU, else the smallest that fits 64 KB; total = 0 if none
// fits.
LaneLayout choose_lane_layout(int S, int nmax, int lmax, size_t elem)
{
    for (int ch = 64; ch >= 16; ch /= 2) {
        LaneLayout W = lane_layout(S, nmax, lmax, ch);
        if (size_t(W.total) * elem <= 24 * 1024) return W;
    }
    LaneLayout W = lane_layout(S, nmax, lmax, 16);
    if (size_t(W.total) * elem > 64 * 1024) W.total = 0;
    return W;
}

constexpr int64_t kSplitAtoms = 4096;   // c and p in two kernels from this many centres

hipError_t launch_expansion_lanes(const FeatureArgs& a, bool f64, hipStream_t stream)
{
    if (a.p == nullptr) return launch_expansion_packed(a, f64, stream);
    if (a.n_atoms >= kSplitAtoms) {
        // c with the pairs packed across centres, then p from c in HBM
        // (4096 liquid centres: 61 and 21 us against 78 for c and p in one
        // kernel, 8000 90 and 33 against 126; at n=6, lmax=4 in double 23 and
        // 9 against 39; smaller systems are faster in one launch)
        FeatureArgs c = a;
        c.p = nullptr;
        hipError_t e = launch_expansion_packed(c, f64, stream);
        if (e == hipSuccess) {
            FeatureArgs q = a;
            q.dcoeffs = q.dcoeffs_self = q.dp = q.dp_self = nullptr;
            e = launch_power_spectrum(q, f64 ? SOAP_F64 : SOAP_F32, stream);
            if (e != hipErrorNotSupported) return e;
        } else if (e != hipErrorNotSupported) {
            return e;
        }
    }
    const size_t elem = f64 ? 8 : 4;
    LaneLayout W = choose_lane_layout(a.S, a.nmax, a.lmax, elem);
    if (W.total == 0 || a.n_atoms == 0) return W.total == 0 ? hipErrorNotSupported : hipSuccess;
    return f64 ? by_degree<double, LanesFn>(a.lmax, a, W, stream)
               : by_degree<float, LanesFn>(a.lmax, a, W, stream);
}

}  // namespace soap
