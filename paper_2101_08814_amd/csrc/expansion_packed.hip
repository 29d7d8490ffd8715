// Layout and launch of the packed expansion (expansion_packed.hpp).
#include "expansion_packed.hpp"

namespace soap {

hipError_t launch_packed_f64(const FeatureArgs& a, const PackLayout& W, hipStream_t st);

// Pairs per chunk and centres per wave; the results do not depend on them.
// Chunks of 16 fit 64 KB of LDS at every nmax up to kPackMaxN, lmax and
// precision (49 KB in double at nmax 16, lmax 12).
//
// Chunks of 32 pairs take half the steps of chunks of 16 and hold twice the
// LDS.  While every centre has a wave of its own on the chip at once (256 CUs,
// as many waves each as their LDS allows, 16 at most) the steps count: 300
// centres of 45 pairs at n=10, lmax=8 take 16.7 us in chunks of 32, 23.0 of
// 16, 1000 centres 21.4 and 28.1.  Beyond that the waves in flight count: 2048
// centres 36.6 and 28.5, 8192 104 and 74 (of 120 pairs 219 and 174).  Where a
// pair has few radial values its geometry and harmonics are what it costs, and
// 32 pairs form them twice instead of 16 four times: 16,384 centres of 120
// pairs at n=3, lmax=2 take 53 and 71 us, of 12 pairs in double at n=6, lmax=4
// 41.6 and 42.8 (four centres a wave; 4096 centres, two a wave, 13.3 and 14.6).
//
// Several centres share a wave's set-up and its last, partly filled chunk, but
// fewer waves balance worse at the end: 8192 centres of 45 pairs at n=10,
// lmax=8 take 74, 90 and 88 us at one, two and four centres per wave, 16,384
// of 30 pairs at n=8, lmax=6 58, 56 and 54 (of 12 pairs 41, 38 and 36), 32,768
// of 45 at n=10, lmax=8 262, 261 and 256, 131,072 of 31 at n=12, lmax=8 1.72
// and 1.58 ms at one and four (in chunks of 32).
PackLayout pack_layout(int nmax, int lmax, int64_t n_atoms, int64_t pair_capacity, size_t elem)
{
    PackLayout W{};
    const int lm1 = lmax + 1;
    W.gmax = (nmax + 3) / 4;
    auto set = [&](int ch, int cpw) {
        W.ch = ch;
        W.cpw = cpw;
        W.total = ch * (4 * pack_quads(lm1, W.gmax, ch) + ((lm1 * lm1) | 1)) + kPackMaxN + 4 * ch;
    };
    const int nl = lm1 * nmax;   // radial values of a pair
    const bool long_envs = pair_capacity >= 32 * n_atoms;
    set(32, 1);
    const int64_t wave = int64_t(W.total) * int64_t(elem), cu = 160 * 1024 / wave;
    if (wave > 64 * 1024) {
        set(16, 1);
    } else if (n_atoms > 256 * (cu < 16 ? cu : 16)) {
        if (nl <= 16 || (nl <= 32 && !long_envs)) {
            W.cpw = long_envs ? 1 : n_atoms >= 8192 ? 4 : n_atoms >= 2048 ? 2 : 1;
            return W;
        }
        set(16, 1);
    } else {
        return W;
    }
    W.cpw = n_atoms >= 32768 ? 4 : n_atoms >= 16384 ? 2 : 1;
    return W;
}

hipError_t launch_expansion_packed(const FeatureArgs& a, bool f64, hipStream_t stream)
{
    if (a.p != nullptr || a.nmax > kPackMaxN) return hipErrorNotSupported;
    if (a.n_atoms == 0) return hipSuccess;
    const size_t elem = f64 ? 8 : 4;
    const PackLayout W = pack_layout(a.nmax, a.lmax, a.n_atoms, a.pair_capacity, elem);
    return f64 ? launch_packed_f64(a, W, stream) : launch_packed<float>(a, W, stream);
}

}  // namespace soap
