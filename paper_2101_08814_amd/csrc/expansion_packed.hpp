// Spherical expansion c alone (Sec. 4.A Eq.
// spherical_expansion_coefficients_gaussians, Sec. 4.F) with the pairs of
// several centres packed into one wave's chunks.
//
// A wave takes one to four consecutive centres and walks their pairs, which
// are stored contiguously and grouped by centre and then by neighbour species,
// in chunks of CH = 16 or 32 (pack_layout says when): a chunk may hold the end
// of one centre and the start of the next, so the lanes stay busy when centres
// have few pairs.  The 64 / CH lanes of a pair all form its geometry and
// harmonics Y_lm (and write the same values to the wave's LDS rows).
//
// The radial values R_nl = f I~_nl, in chunks of 32: by two lanes per pair,
// four n at a time with one 16-byte LDS store.  In chunks of 16: by four lanes
// per pair, neighbouring lanes on neighbouring cubics of the pair's interval,
// so that a load takes 64-byte runs of 16 pairs and not 16 bytes of each of 64
// lines.  Chunks of 16 halve the LDS of a wave (12.6 KB at nmax 12, lmax 8),
// which lets twice the waves share a CU; forming the harmonics four times over
// costs less than those gain once the chip is full: 131,072 centres at nmax
// 12, lmax 8 (4.1 GB written) 1.72 -> 1.44 ms.  Either change alone is slower
// or gives a third of that (cooperative loads in chunks of 32: 1.75 ms, chunks
// of 16 with a lane per quad: 1.57).  Sums on v_mfma_f32_4x4x1 (four n and an
// m per lane): 1.46 to 1.56 ms.
//
// Each lane then owns up to pack_slots items (four n, one lm) of c and sums
// R_{n..n+3,l} Y_lm over the pairs of the current (centre, species) segment in
// registers; when the segment ends the sums go straight to HBM (consecutive
// lanes on consecutive lm) with the central atom's term added, and species
// without pairs are written as zeros.  Every output element has one owner.  A
// list whose species are not grouped within a centre is detected, and the
// wave's centres are then redone one species at a time.
//
// The groups of four n, GMAX = ceil(nmax / 4), are a template parameter, so
// that the items, the quads of a row and their degrees are constants (with the
// number of groups a run-time value up to GMAX: 300 centres of 120 pairs at
// n=10, lmax=8 35.6 us, 32.8 with the constant).
#pragma once

#include "lane_pair.hpp"
#include <cstdlib>

namespace soap {
namespace {

using namespace dev;

constexpr int kPackMaxCpw = 4;   // centres per wave
constexpr int kPackMaxN = 16;    // nmax covered by the register items

// quads of an LDS row of radial values: with four lanes per pair an odd
// number, so that the rows of 16 pairs start on distinct banks; with two a
// spare quad past the row
__host__ __device__ constexpr int pack_quads(int lm1, int gmax, int ch)
{
    return ch == 16 ? (lm1 * gmax) | 1 : lm1 * gmax + 1;
}

// items per lane with GMAX groups of four n (4 GMAX - 4 < nmax <= 4 GMAX)
template <int LMAX, int GMAX>
constexpr int pack_slots()
{
    return (GMAX * (LMAX + 1) * (LMAX + 1) + 63) / 64;
}

// waves per SIMD the register allocation aims at (where it fits without
// spilling: three at nmax <= 8, lmax <= 6 in FP32, where the LDS allows
// eleven waves per CU; two up to lmax 8)
template <typename T, int LMAX, int GMAX>
constexpr int pack_waves()
{
    return sizeof(T) != 4 ? 1 : (GMAX <= 2 && LMAX <= 6) ? 3 : LMAX <= 8 ? 2 : 1;
}

// CH: pairs per chunk, 64 / CH lanes per pair
template <typename T, int LMAX, int GMAX, int CH>
__global__ void __launch_bounds__(64, (pack_waves<T, LMAX, GMAX>())) k_expansion_packed(FeatureArgs a, PackLayout W)
{
    constexpr int LM1 = LMAX + 1, L2 = LM1 * LM1, NS = pack_slots<LMAX, GMAX>(), NI = GMAX * L2;
    // LDS rows of a pair: radial values [l][4 GMAX], and the harmonics (odd
    // stride)
    constexpr int NP = 4 * GMAX, NLS = 4 * pack_quads(LM1, GMAX, CH), L2S = L2 | 1;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* Rs = reinterpret_cast<T*>(smem_raw);   // [pair][NLS] radial values
    T* Ys = Rs + CH * NLS;                // [pair][L2S] harmonics
    const int lane = threadIdx.x;
    if (a.pair_offsets[a.n_atoms] > a.pair_capacity) {
        if (lane == 0) put_status(a.status, SOAP_ECAPACITY);
        return;
    }
    const int nmax = a.nmax, S = a.S;
    const int nL2 = nmax * L2;
    const int nl = LM1 * nmax;
    const int64_t c0 = int64_t(blockIdx.x) * W.cpw;
    const int ncw = int(a.n_atoms - c0 < W.cpw ? a.n_atoms - c0 : W.cpw);
    int64_t bnd[kPackMaxCpw + 1];   // pair range of each of the wave's centres
#pragma unroll
    for (int k = 0; k <= kPackMaxCpw; ++k) bnd[k] = a.pair_offsets[c0 + (k < ncw ? k : ncw)];
    const T* __restrict__ centre_term = static_cast<const T*>(a.center);
    const V4<T>* __restrict__ coef = static_cast<const V4<T>*>(a.coef_ln);
    const T* __restrict__ vec = static_cast<const T*>(a.pair_vec);
    T* c_out = static_cast<T*>(a.coeffs) + c0 * S * int64_t(nL2);

    // items v = lane + 64 u (u < NS, v < NI): n = 4 ng .. 4 ng + 3 of one lm;
    // lanes past NI in the last slot read row 0 and write nothing
    int yoff[NS], roff[NS];
    unsigned ooff[NS];   // bytes of the item in a block of c
    V4<T> acc[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const int v = lane + 64 * u;
        const int ng = v / L2, lm = v - ng * L2;
        const bool in = v < NI;
        yoff[u] = in ? lm : 0;
        roff[u] = in ? l_of(lm) * NP + 4 * ng : 0;
        ooff[u] = unsigned(4 * ng * L2 + lm) * unsigned(sizeof(T));
        acc[u] = V4<T>{T(0), T(0), T(0), T(0)};
    }
    // the central atom's terms in LDS, so that writing a block waits on no
    // global load
    T* Cs = Ys + CH * L2S;
    if (lane < kPackMaxN) Cs[lane] = lane < nmax ? centre_term[lane] : T(0);
    // {t, f, interval} of the chunk's pairs
    T* Gs = Cs + kPackMaxN;
    // species of the wave's centres, 16 bits each (0xFFFF: no central term)
    uint64_t cspc = ~uint64_t(0);
#pragma unroll
    for (int k = 0; k < kPackMaxCpw; ++k) {
        if (a.include_center && k < ncw) {
            const int si = a.species[c0 + k];
            if (si < 0 || si >= S) {
                if (lane == 0) put_status(a.status, SOAP_ESPECIES);
            } else {
                cspc = (cspc & ~(uint64_t(0xFFFF) << (16 * k))) | (uint64_t(si) << (16 * k));
            }
        }
    }

    // the inputs of pair q0 + p (p = lane mod CH, p < nc): vector and
    // neighbour index, loaded a chunk ahead; the neighbour's species once
    // the index has arrived
    struct PairIn {
        T x, y, z;
        int j;
    };
    auto load_in = [&](int64_t q0, int nc) __attribute__((always_inline)) -> PairIn {
        PairIn r{T(0), T(0), T(1), 0};
        const int p = lane & (CH - 1);
        if (p < nc) {
            const int64_t q = q0 + p;
            r.x = vec[3 * q];
            r.y = vec[3 * q + 1];
            r.z = vec[3 * q + 2];
            r.j = a.pair_j[q];
        }
        return r;
    };
    // species of neighbour j, checked (an invalid j stores SOAP_EINVAL, an
    // invalid species SOAP_ESPECIES; both count as species 0)
    auto species_of = [&](int j, bool valid) __attribute__((always_inline)) -> int {
        if (!valid) return 0;
        if (j < 0 || j >= a.n_atoms) {
            put_status(a.status, SOAP_EINVAL);
            return 0;
        }
        const int sp = a.species[j];
        if (sp < 0 || sp >= S) {
            put_status(a.status, SOAP_ESPECIES);
            return 0;
        }
        return sp;
    };
    // Pair q0 + p (p = lane mod CH) staged by its lanes; returns its key
    // (centre of the wave) S + (neighbour species), -1 past the chunk.
    auto stage = [&](int64_t q0, int nc, const PairIn& in, int spq) __attribute__((always_inline)) -> int {
        const int p = lane & (CH - 1);
        int key = -1;
        T t = T(0), f = T(0), ux = T(0), uy = T(0), uz = T(1);
        int k = 0;
        if (p < nc) {
            const int64_t q = q0 + p;
            const PairGeom<T> g = pair_geometry<T>(a, in.x, in.y, in.z);
            int cl = 0;
#pragma unroll
            for (int c = 1; c < kPackMaxCpw; ++c) cl += q >= bnd[c] ? 1 : 0;
            key = cl * S + spq;
            ux = g.ux; uy = g.uy; uz = g.uz;
            t = g.t; f = g.f; k = g.k;
        }
        auto harmonics = [&]() __attribute__((always_inline)) {
            T* yrow = Ys + p * L2S;
            YlmStream<T, LMAX> ys(ux, uy, uz);
            static_for<0, LM1>([&](auto Lc) __attribute__((always_inline)) {
                constexpr int L = decltype(Lc)::value;
                ys.template degree<L, false>([&](int mi, T Y, T, T, T) __attribute__((always_inline)) {
                    yrow[L * L + mi] = Y;
                });
            });
        };
        if constexpr (CH == 16) {
            if (lane < CH) *reinterpret_cast<V4<T>*>(Gs + 4 * p) = V4<T>{t, f, T(k), T(0)};
            wave_sync();
            // radial values: lane = 4 pl + part takes the cubics j = part + 4 i of
            // pair pl (past the interval: the next one's, or the table's zero
            // tail, not stored), kNB at a time, the first in flight during the
            // harmonics and each next batch during the last
            constexpr int NQ = LM1 * GMAX, kNB = 6, NBAT = (NQ + kNB - 1) / kNB;
            const int part = lane & 3, pl = lane >> 2, ni = (nl + 3) >> 2;
            const V4<T> gq = *reinterpret_cast<const V4<T>*>(Gs + 4 * pl);
            const T tt = gq.x, ff = gq.y;
            const V4<T>* cf = coef + int64_t(int(gq.z)) * nl + part;
            V4<T> A[2][kNB];
            auto fetch = [&](int b) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < kNB; ++i) A[b & 1][i] = cf[4 * (b * kNB + i)];
            };
            // LDS position of the lane's next value: l NP + n for j = l nmax + n
            int rn = part, ro = part;
            auto settle = [&]() __attribute__((always_inline)) {
                const bool w = rn >= nmax;
                rn -= w ? nmax : 0;
                ro += w ? NP - nmax : 0;
                if (nmax < 4)   // up to four degrees per step
                    while (rn >= nmax) {
                        rn -= nmax;
                        ro += NP - nmax;
                    }
            };
            settle();
            T* rrow = Rs + pl * NLS;
            auto use = [&](int b) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < kNB; ++i) {
                    const V4<T> c = A[b & 1][i];
                    if (ro < LM1 * NP) rrow[ro] = ff * (c.x + tt * (c.y + tt * (c.z + tt * c.w)));
                    rn += 4;
                    ro += 4;
                    settle();
                }
            };
            fetch(0);
            harmonics();
            static_for<0, NBAT>([&](auto Bc) __attribute__((always_inline)) {
                constexpr int b = decltype(Bc)::value;
                if (b * kNB < ni) {
                    if constexpr (b + 1 < NBAT) {
                        if ((b + 1) * kNB < ni) fetch(b + 1);
                    }
                    use(b);
                }
            });
        } else if (p < nc) {
            // radial quads u = h + 2 i: four n of one l, coefficient
            // j = l nmax + 4 (u - l GMAX) = 4 u - l pad, at 4 u of the row.
            // The last quad of a degree may read up to three values past it
            // (the next interval's, or the table's zero tail), which land in
            // the row's padding.  Every lane takes QH quads: those past the
            // last one read its coefficients and write the row's spare quad,
            // so that each load is used on every path.
            constexpr int NQ = LM1 * GMAX, QH = (NQ + 1) / 2, kNB = GMAX <= 2 ? 3 : 2, NB = QH < kNB ? QH : kNB;
            constexpr int gmul = (65536 + GMAX - 1) / GMAX;   // l of quad u: (u * gmul) >> 16
            const int h = lane >> 5, pad = 4 * GMAX - nmax;
            const V4<T>* cf = coef + int64_t(k) * nl;
            T* rrow = Rs + p * NLS;
            auto coefs = [&](int u, V4<T>* A) __attribute__((always_inline)) {
                u = u < NQ ? u : NQ - 1;
                const int j = 4 * u - ((u * gmul) >> 16) * pad;
#pragma unroll
                for (int x = 0; x < 4; ++x) A[x] = cf[j + x];
            };
            auto put = [&](int u, const V4<T>* A) __attribute__((always_inline)) {
                V4<T> r;
                r.x = f * (A[0].x + t * (A[0].y + t * (A[0].z + t * A[0].w)));
                r.y = f * (A[1].x + t * (A[1].y + t * (A[1].z + t * A[1].w)));
                r.z = f * (A[2].x + t * (A[2].y + t * (A[2].z + t * A[2].w)));
                r.w = f * (A[3].x + t * (A[3].y + t * (A[3].z + t * A[3].w)));
                *reinterpret_cast<V4<T>*>(rrow + 4 * (u < NQ ? u : NQ)) = r;
            };
            // the first quads in flight during the harmonics, then each buffer
            // refilled with the quad NB ahead
            V4<T> Bf[NB][4];
            static_for<0, NB>([&](auto I) __attribute__((always_inline)) {
                constexpr int i = decltype(I)::value;
                coefs(h + 2 * i, Bf[i]);
            });
            harmonics();
            static_for<0, QH>([&](auto I) __attribute__((always_inline)) {
                constexpr int i = decltype(I)::value;
                put(h + 2 * i, Bf[i % NB]);
                if constexpr (i + NB < QH) coefs(h + 2 * (i + NB), Bf[i % NB]);
            });
        }
        wave_sync();
        return key;
    };
    // pairs [lo, hi) of the chunk added to the lane's items
    // (per pair, the lane's slots together: their LDS reads in flight at once)
    auto accumulate = [&](int lo, int hi) __attribute__((always_inline)) {
        const T* yb = Ys + lo * L2S;
        const T* rb = Rs + lo * NLS;
        auto pair = [&](int k) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                const T Y = yb[k * L2S + yoff[u]];
                const V4<T> R = *reinterpret_cast<const V4<T>*>(rb + k * NLS + roff[u]);
                acc[u].x += R.x * Y;
                acc[u].y += R.y * Y;
                acc[u].z += R.z * Y;
                acc[u].w += R.w * Y;
            }
        };
        // four pairs per step at fixed offsets from one address per slot
        int p = lo;
        for (; p + 4 <= hi; p += 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) pair(k);
            yb += 4 * L2S;
            rb += 4 * NLS;
        }
        for (; p < hi; ++p) {
            pair(0);
            yb += L2S;
            rb += NLS;
        }
    };
    // block key = cl S + sp of c to HBM and the sums cleared; the central
    // atom adds its term to lm = 0 of its own species
    auto flush = [&](int cl, int sp) __attribute__((always_inline)) {
        const int key = cl * S + sp;
        const bool own = int((cspc >> (16 * cl)) & 0xFFFF) == sp;
        T* out = c_out + int64_t(key) * nL2;
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int v = lane + 64 * u;
            const int ng = v / L2, lm = v - ng * L2;
            const int nn = v < NI ? min(4, nmax - 4 * ng) : 0;   // n of the item that exist
            T x4[4] = {acc[u].x, acc[u].y, acc[u].z, acc[u].w};
            if (own) {   // the same for the whole wave
                const bool cen = lm == 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const T ck = Cs[min(4 * ng + k, kPackMaxN - 1)];
                    x4[k] += cen ? ck : T(0);
                }
            }
            T* o = reinterpret_cast<T*>(reinterpret_cast<char*>(out) + ooff[u]);
            if (nn == 4) {
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k * L2] = x4[k];
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k < nn) o[k * L2] = x4[k];
            }
            acc[u] = V4<T>{T(0), T(0), T(0), T(0)};
        }
    };

    const int nkeys = ncw * S;
    int cur = 0, ccl = 0, csp = 0;   // blocks below cur = ccl S + csp are written
    auto flush_cur = [&]() __attribute__((always_inline)) {
        flush(ccl, csp);
        ++cur;
        if (++csp == S) {
            csp = 0;
            ++ccl;
        }
    };
    bool grouped = true;
    const int64_t pe = bnd[kPackMaxCpw];
    auto chunk_n = [&](int64_t q0) __attribute__((always_inline)) {
        return int(pe - q0 < CH ? pe - q0 : CH);
    };
    // The next chunk's inputs are loaded after this chunk's coefficient
    // loads have been used (vector loads complete in order, so loads issued
    // before them would hold them up) and arrive during the sums.
    PairIn nxt = load_in(bnd[0], chunk_n(bnd[0]));
    int nsp = species_of(nxt.j, (lane & (CH - 1)) < chunk_n(bnd[0]));
    for (int64_t q0 = bnd[0]; q0 < pe; q0 += CH) {
        const int nc = chunk_n(q0);
        const PairIn in = nxt;
        const int spq = nsp;
        const bool more = q0 + CH < pe;
        const int nc1 = more ? chunk_n(q0 + CH) : 0;
        const int key = stage(q0, nc, in, spq);
        if (more) nxt = load_in(q0 + CH, nc1);
        const int prev = __shfl_up(key, 1, 64);
        if (__ballot(lane < nc && key < (lane == 0 ? cur : prev))) {
            grouped = false;
            break;
        }
        for (int lo = 0; lo < nc;) {
            const int k = __builtin_amdgcn_readlane(key, lo);
            const int cnt = __popcll(__ballot(lane < nc && key == k));
            while (cur < k) flush_cur();
            accumulate(lo, lo + cnt);
            lo += cnt;
        }
        if (more) nsp = species_of(nxt.j, (lane & (CH - 1)) < nc1);
        wave_sync();   // the rows are read before the next chunk overwrites them
    }
    if (grouped) {
        while (cur < nkeys) flush_cur();
        return;
    }
    // species not grouped within a centre: each centre again, one species
    // per pass over its pairs
#pragma unroll
    for (int u = 0; u < NS; ++u) acc[u] = V4<T>{T(0), T(0), T(0), T(0)};
    for (int cl = 0; cl < ncw; ++cl) {
        for (int sp = 0; sp < S; ++sp) {
            for (int64_t q0 = bnd[cl]; q0 < bnd[cl + 1]; q0 += CH) {
                const int nc = int(bnd[cl + 1] - q0 < CH ? bnd[cl + 1] - q0 : CH);
                const PairIn in = load_in(q0, nc);
                const int key = stage(q0, nc, in, species_of(in.j, (lane & (CH - 1)) < nc));
                for (int p = 0; p < nc; ++p)
                    if (__builtin_amdgcn_readlane(key, p) == cl * S + sp) accumulate(p, p + 1);
                wave_sync();
            }
            flush(cl, sp);
        }
    }
}

template <typename T, int LM>
struct PackedFn {
    template <int GMAX, int CH>
    static hipError_t launch(const FeatureArgs& a, const PackLayout& W, hipStream_t st)
    {
        const size_t lds = size_t(W.total) * sizeof(T);
        const int64_t waves = (a.n_atoms + W.cpw - 1) / W.cpw;
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_expansion_packed<T, LM, GMAX, CH>), dim3(unsigned(waves)), dim3(64), lds, st,
                           a, W);
        return hipGetLastError();
    }
    template <int CH>
    static hipError_t run_ch(const FeatureArgs& a, const PackLayout& W, hipStream_t st)
    {
        if (W.gmax == 1) return launch<1, CH>(a, W, st);
        if (W.gmax == 2) return launch<2, CH>(a, W, st);
        if (W.gmax == 3) return launch<3, CH>(a, W, st);
        return launch<4, CH>(a, W, st);
    }
    static hipError_t run(const FeatureArgs& a, const PackLayout& W, hipStream_t st)
    {
        if constexpr (LM < 0) {
            return hipErrorNotSupported;
        } else {
            if (W.ch == 16) return run_ch<16>(a, W, st);
            return run_ch<32>(a, W, st);
        }
    }
};

template <typename T>
hipError_t launch_packed(const FeatureArgs& a, const PackLayout& W, hipStream_t st)
{
    return by_degree<T, PackedFn>(a.lmax, a, W, st);
}

}  // namespace
}  // namespace soap
