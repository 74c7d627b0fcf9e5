// Runs the product's score keys and cut search (score_cut.h) on the host against sorting.  Exit code 0: all hold.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <limits>
#include <random>
#include <vector>

#include "score_cut.h"

using namespace chess;

static int fail(const char* what, int a, int b)
{
    std::printf("FAILED: %s (%d, %d)\n", what, a, b);
    return 1;
}

int main()
{
    const double inf = std::numeric_limits<double>::infinity(), nan = std::numeric_limits<double>::quiet_NaN();
    const double special[] = {nan, -nan, inf, -inf, 0.0, -0.0, 1e300, -1e300, 3.5e38, -3.5e38, 1e37, -1e37, 5e-324, -5e-324, 1.0, -1.0};
    std::mt19937_64 rng(1);
    std::normal_distribution<double> normal;

    // the float of a key never decreases when the key grows, and differences of two of them are finite
    std::vector<uint64_t> keys;
    for (double s : special) keys.push_back(order_key(s));
    for (int i = 0; i < 20000; ++i) keys.push_back(order_key(__builtin_bit_cast(double, rng())));
    for (int i = 0; i < 20000; ++i) keys.push_back(order_key(normal(rng)));
    std::sort(keys.begin(), keys.end());
    for (size_t i = 0; i < keys.size(); ++i) {
        const float f = key_float((unsigned)(keys[i] >> 32));
        if (!std::isfinite(f)) return fail("finite", (int)i, 0);
        if (i > 0 && !(key_float((unsigned)(keys[i - 1] >> 32)) <= f)) return fail("monotone", (int)i, 0);
    }
    if (!std::isfinite(key_float((unsigned)(keys.back() >> 32)) - key_float((unsigned)(keys[0] >> 32)))) return fail("difference", 0, 0);

    // the search: what lies above the bracket and `want` of the bracket's own are the k largest, and the bracket's count is right
    for (int round = 0; round < 4000; ++round) {
        const int n = 2 + (int)(rng() % 255), kind = round % 5;
        std::vector<uint64_t> key(n);
        for (auto& x : key) x = order_key(kind == 1 ? (double)(int)(rng() % 3) : normal(rng) * (kind == 2 ? 1e36 : 1.0));
        if (kind >= 2)                                // a few special values among them (all of them in the last kind)
            for (int i = 0; i < n; ++i)
                if (kind == 4 || rng() % 8 == 0) key[i] = order_key(special[rng() % 16]);
        std::vector<float> f(n);
        for (int i = 0; i < n; ++i) f[i] = key_float((unsigned)(key[i] >> 32));
        const uint64_t lo = *std::min_element(key.begin(), key.end()), hi = *std::max_element(key.begin(), key.end());
        std::vector<uint64_t> order(key);
        std::sort(order.begin(), order.end(), std::greater<uint64_t>());
        const auto count = [&](float t1, float t2, float t3, int& c1, int& c2, int& c3) {
            for (float x : f) { c1 += x > t1; c2 += x > t2; c3 += x > t3; }
        };
        for (int k = 1; k < n; k += 1 + (int)(rng() % 7)) {
            const Bracket br = search_cut(count, k, n, key_float((unsigned)(lo >> 32)), key_float((unsigned)(hi >> 32)));
            int sure = 0, in = 0;
            for (int i = 0; i < n; ++i) {
                sure += f[i] > br.above;
                in += f[i] > br.from && !(f[i] > br.above);
            }
            if (sure + br.want != k || br.want < 0) return fail("kept for sure + wanted = k", round, k);
            if (br.cnt > 0 && in != br.cnt) return fail("members of the bracket", round, k);
            if (br.want > br.cnt) return fail("wanted of the bracket", round, k);
            for (int i = 0; i < n; ++i) {
                if (f[i] > br.above && key[i] < order[k - 1]) return fail("a kept slot is not among the k largest", round, k);
                if (!(f[i] > br.from) && key[i] > order[k - 1]) return fail("a dropped slot is among the k largest", round, k);
            }
        }
    }
    std::printf("ok\n");
    return 0;
}
