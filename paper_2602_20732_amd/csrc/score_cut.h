// Scores as ordered keys, and the search for a cut among them: the part of the selection's arithmetic that has nothing
// of the GPU in it (plain C++ as well, so that the CPU tests run this code and not a copy).
#pragma once

#include <cmath>
#include <cstdint>

#ifdef __HIPCC__
#define CHESS_HD __host__ __device__ __forceinline__
#else
#define CHESS_HD inline
#endif

namespace chess {

// Monotone map double -> uint64 (larger score = larger key); every finite or infinite score maps
// to a key >= 2^52 - 1, so 0 can mark "not published yet" and 1 "no unit".  -0.0 is folded onto +0.0.  A NaN gets a
// key beyond the infinity of its sign.
CHESS_HD uint64_t order_key(double s)
{
    s += 0.0;
    const uint64_t u = __builtin_bit_cast(uint64_t, s);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// A float that never decreases when the key grows: the score with its lower 32 bits dropped, rounded to fp32,
// kept finite.  All the binning of a cut needs is this monotonicity (a higher bin then means a strictly larger
// score); the exact order inside a bin is settled on the 64-bit keys.
// The key is clamped, not the float, to the keys of -2^126 and 2^126: infinities and NaNs of either sign then keep
// their places at the ends (clamped as a float, a positive NaN -- the largest key there is -- fell to the bottom, and a
// cut that took its bounds from the smallest and the largest key kept nearly everything), and the difference of two
// such floats is finite.
CHESS_HD float key_float(unsigned key_hi)
{
    constexpr unsigned kTop = 0xC7D00000u;            // upper half of order_key(2^126)
    const unsigned k = key_hi < ~kTop ? ~kTop : key_hi > kTop ? kTop : key_hi;
    const unsigned u = (k >> 31) ? (k & 0x7fffffffu) : ~k;
    return (float)__builtin_bit_cast(double, (uint64_t)u << 32);
}

// What the search for a cut ends with: slots with f > above are kept for sure; the cnt slots with from < f <= above
// still have to be ranked on their 64-bit keys, want of them are kept.  cnt = 0: the cut falls between two keys.
struct Bracket {
    float above, from;
    int want, cnt;
};

constexpr int kSearchBits = 24;             // thresholds the search tells apart: 2^24 steps from the smallest to the largest score

// The bracket of the k-th largest of n_valid scores f (0 < k < n_valid; fmin and fmax: the smallest and the largest of
// them, finite).  count(t1, t2, t3, c1, c2, c3) says how many scores are above each of three thresholds.  The number of the
// highest threshold with at least k scores above it, two bits a step, the highest first, until a threshold has exactly k (5 steps
// for 256 normally distributed scores).  Two bits, because a step is a chain of dependent instructions whatever it
// counts; thresholds by number (they never decrease with it, whatever is rounded), so that all a step decides is scalar and
// nothing in it branches: as a search that kept the bounds themselves a step took 600 cycles of a wave with 256 keys.
template <class Count>
CHESS_HD Bracket search_cut(Count count, int k, int n_valid, float fmin, float fmax)
{
    const float step = (fmax - fmin) * (1.f / (float)(1 << kSearchBits));
    const auto threshold = [&](unsigned j) { return __builtin_fmaf((float)j, step, fmin); };
    unsigned t = 0;                                   // at least k scores above threshold t; 0: all of them
    int c_t = n_valid;
#pragma unroll 1
    for (unsigned h = 1u << (kSearchBits - 2); h != 0; h >>= 2) {
        int c1 = 0, c2 = 0, c3 = 0;
        count(threshold(t + h), threshold(t + 2 * h), threshold(t + 3 * h), c1, c2, c3);
        const int n1 = c1 >= k, n2 = c2 >= k, n3 = c3 >= k;                // n3 implies n2 implies n1
        t += h * (unsigned)(n1 + n2 + n3);
        c_t = n3 ? c3 : n2 ? c2 : n1 ? c1 : c_t;
        if (c_t == k) break;
    }
    const float from = t == 0 ? -INFINITY : threshold(t);
    if (c_t == k) return Bracket{from, from, 0, 0};
    const float above = t + 1 == 1u << kSearchBits ? fmax : threshold(t + 1);
    int c1 = 0, c2 = 0, c3 = 0;
    count(above, above, above, c1, c2, c3);
    return Bracket{above, from, k - c1, c_t - c1};
}

}  // namespace chess
