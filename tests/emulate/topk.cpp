// k_topk and k_regret of select.hip on the CPU, with one wave held back or run
// ahead at every point where it can be: the picks and regrets have to be those
// of a plain sort each time.  Prints "topk ok" at the end.
#include KERNELS

#include <algorithm>
#include <cmath>
#include <random>

using namespace hwsel;

static uint64_t order(float s, uint32_t i)
{
    uint32_t b = s != s ? 0u : (s == 0.0f ? 0x80000000u : 0u);
    if (!b && s == s) b = (__float_as_uint(s) >> 31) ? ~__float_as_uint(s) : __float_as_uint(s) | 0x80000000u;
    return (uint64_t)b << 32 | (0xffffffffu - i);
}

template <int NT>
static void topk(const char *what, const std::vector<float> &s, int k, const std::vector<int> &priority)
{
    const int64_t seg[2] = {0, (int64_t)s.size()};
    std::vector<int32_t> idx(k, -7);
    std::vector<float> vals(k, 7.0f);
    lanes::run(NT, 0, priority, [&] { k_topk<NT>(s.data(), seg, k, idx.data(), vals.data()); });
    std::vector<uint64_t> keys;
    for (size_t i = 0; i < s.size(); ++i) keys.push_back(order(s[i], (uint32_t)i));
    std::sort(keys.rbegin(), keys.rend());
    for (int j = 0; j < k; ++j) {
        const int32_t want = j < (int)keys.size() ? (int32_t)(0xffffffffu - (uint32_t)keys[j]) : -1;
        if (idx[j] != want) {
            printf("%s, %zu rows, k %d, %d threads: pick %d is %d, not %d\n", what, s.size(), k, NT, j, idx[j], want);
            lanes::fail("wrong pick");
        }
    }
}

template <int NT>
static void all_orders(const char *what, const std::vector<float> &s, int k)
{
    const int waves = NT / 64;
    for (int w = 0; w < waves; w += waves > 4 ? 5 : 1)
        for (const int p : {-1, 1}) {                      // wave w last, then first
            std::vector<int> priority(waves, 0);
            priority[w] = p;
            topk<NT>(what, s, k, priority);
        }
}

int main()
{
    std::mt19937 g(1);
    std::normal_distribution<float> normal;
    auto some = [&](int n, auto &&f) {
        std::vector<float> s(n);
        for (int i = 0; i < n; ++i) s[i] = f(i);
        return s;
    };
    // one tile; several whose best rows lie in the first (nothing above the
    // floor later on), in the last, in all; more rows above the floor than the list holds
    const struct {
        const char *what;
        std::vector<float> s;
        int k;
    } cases[] = {
        {"one tile", some(700, [&](int) { return normal(g); }), 7},
        {"falling", some(3 * 8192 + 5, [&](int i) { return -(float)i; }), 3},
        {"rising", some(3 * 8192 + 5, [&](int i) { return (float)i; }), 16},
        {"random", some(4 * 8192, [&](int) { return normal(g); }), 5},
        {"equal", some(2 * 8192 + 1, [&](int) { return 1.0f; }), 33},
        {"few", some(9, [&](int) { return normal(g); }), 64},
        {"one wave", some(64, [&](int) { return normal(g); }), 5},
        {"past one wave", some(65, [&](int) { return normal(g); }), 64},
        {"short", some(1024, [&](int i) { return (float)(i % 5); }), 9},
        {"past short", some(1025, [&](int i) { return (float)(i % 5); }), 9},
        {"flood, then not", some(5 * 8192, [&](int i) { return i < 4 * 8192 ? (float)i : -(float)i; }), 16},
        {"one wave", some(64, [&](int) { return normal(g); }), 5},
        {"past one wave", some(65, [&](int) { return normal(g); }), 64},
        {"flood, then not", some(5 * 8192, [&](int i) { return i < 4 * 8192 ? (float)i : -(float)i; }), 16},
        {"nan", some(8192 + 9, [&](int i) { return i % 3 ? NAN : normal(g); }), 64},
    };
    for (const auto &c : cases) {
        all_orders<256>(c.what, c.s, c.k);
        all_orders<1024>(c.what, c.s, c.k);
        printf("%s: ok\n", c.what);
        fflush(stdout);
    }
    // regrets, a pick of runtime -0 behind a negative one among them
    const std::vector<float> t = {3.0f, -0.0f, -1.0f, 2.0f};
    for (int w = 0; w < 4; ++w) {
        std::vector<int> priority(4, 0);
        priority[w] = -1;
        const int64_t seg[2] = {0, 4};
        const int32_t idx[3] = {3, 1, -1};
        float r1 = 0, rk = 0;
        int32_t best = 0;
        lanes::run(256, 0, priority, [&] { k_regret<256>(t.data(), seg, idx, 3, &r1, &rk, &best); });
        if (best != 2 || r1 != 1.5f || rk != (float)(1.0 - (double)t[2] / (double)t[1])) {
            printf("best %d regret %g, best of 3 %g\n", best, (double)r1, (double)rk);
            lanes::fail("wrong regret");
        }
    }
    printf("topk ok\n");
    return 0;
}
