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

constexpr int kSearchSteps = 14;            // steps (of two bits) a search for the cut takes before it leaves the rest to ranking

// What the search for a cut ends with: slots with f > above are kept for sure; the cnt slots with from < f <= above
// still have to be ranked on their 64-bit keys, want of them are kept.  cnt = 0: the cut falls between two keys.
struct Bracket {
    float above, from;
    int want, cnt;
};

// The bracket of the k-th largest of n_valid scores f (0 < k < n_valid; fmin and fmax: the smallest and the largest of
// them, finite).  count(t1, t2, t3, c1, c2, c3) says how many scores are above each of three thresholds.  A search by
// value, three thresholds a step, that ends as soon as a threshold has exactly k scores above it (4 steps for 256 normally
// distributed scores, 10 at most in 400 draws).  Three thresholds, because a step is a chain of dependent instructions
// whatever it counts.
template <class Count>
CHESS_HD Bracket search_cut(Count count, int k, int n_valid, float fmin, float fmax)
{
    float lo = fmin, hi = fmax;                       // more than k scores above lo (at or above it until it moves), fewer above hi
    float from = -INFINITY;                           // lo once it has moved
    int c_lo = n_valid, c_hi = 0;
#pragma unroll 1
    for (int step = 0; step < kSearchSteps; ++step) {
        const float t2 = 0.5f * lo + 0.5f * hi, t1 = 0.5f * lo + 0.5f * t2, t3 = 0.5f * t2 + 0.5f * hi;
        if (!(lo < t2 && t2 < hi)) break;             // neighbouring floats (or one value): ranked by key
        int c1 = 0, c2 = 0, c3 = 0;
        count(t1, t2, t3, c1, c2, c3);
        if ((c1 == k) | (c2 == k) | (c3 == k)) {
            hi = from = c1 == k ? t1 : c2 == k ? t2 : t3;
            c_lo = c_hi = k;
            break;
        }
        const bool g1 = c1 > k, g2 = c2 > k, g3 = c3 > k;                 // g3 implies g2 implies g1
        hi = g3 ? hi : g2 ? t3 : g1 ? t2 : t1;
        c_hi = g3 ? c_hi : g2 ? c3 : g1 ? c2 : c1;
        lo = g3 ? t3 : g2 ? t2 : g1 ? t1 : lo;
        from = g1 ? lo : from;
        c_lo = g3 ? c3 : g2 ? c2 : g1 ? c1 : c_lo;
    }
    return Bracket{hi, from, k - c_hi, c_lo - c_hi};
}

}  // namespace chess
