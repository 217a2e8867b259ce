// The kernels' quotient (csrc/plane.h) on the device against the division of
// the host, over classes of operands: prints, per class, the largest
// difference in units in the last place (NaN against NaN counts as none) and
// the number of operands.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#include "plane.h"

enum { SINGLE, PAIR, FIELD };
template <typename T>
__global__ void k_quot(const T* a, const T* b, T* q, int n, int form) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= n) return;
    if (form == FIELD) {
        q[t] = ptk::quot_field(a[t], b[t]);
        return;
    }
    if constexpr (sizeof(T) == 8)
        if (form == PAIR) {
            double other;
            ptk::quot2(a[t], 0.75 * a[t], b[t], q[t], other);
            return;
        }
    q[t] = ptk::quot(a[t], b[t]);
}

template <typename T>
int64_t ordered(T v) {   // neighbours differ by 1
    std::conditional_t<sizeof(T) == 8, int64_t, int32_t> i;
    std::memcpy(&i, &v, sizeof v);
    const int64_t mag = i & (sizeof(T) == 8 ? INT64_MAX : INT32_MAX);
    return std::signbit(v) ? -mag : mag;
}

template <typename T>
void check(const char* name, const std::vector<T>& a, const std::vector<T>& b, int form = SINGLE) {
    const int n = (int)a.size();
    T *da, *db, *dq;
    auto ok = [](hipError_t e) {
        if (e != hipSuccess) {
            std::fprintf(stderr, "%s\n", hipGetErrorString(e));
            std::exit(2);
        }
    };
    ok(hipMalloc(&da, n * sizeof(T)));
    ok(hipMalloc(&db, n * sizeof(T)));
    ok(hipMalloc(&dq, n * sizeof(T)));
    ok(hipMemcpy(da, a.data(), n * sizeof(T), hipMemcpyHostToDevice));
    ok(hipMemcpy(db, b.data(), n * sizeof(T), hipMemcpyHostToDevice));
    hipLaunchKernelGGL(k_quot<T>, dim3((n + 255) / 256), dim3(256), 0, 0, da, db, dq, n, form);
    ok(hipGetLastError());
    std::vector<T> q(n);
    ok(hipMemcpy(q.data(), dq, n * sizeof(T), hipMemcpyDeviceToHost));
    int64_t worst = 0;
    int at = 0;
    for (int t = 0; t < n; ++t) {
        const T e = a[t] / b[t];
        int64_t d;
        if (std::isnan(e) || std::isnan(q[t])) d = std::isnan(e) && std::isnan(q[t]) ? 0 : INT64_MAX / 2;
        else d = std::llabs(ordered(e) - ordered(q[t]));
        if (d > worst) {
            worst = d;
            at = t;
        }
    }
    std::printf("%s %lld %d\n", name, (long long)worst, n);
    if (worst) std::fprintf(stderr, "%s: %a / %a = %a, not %a\n", name, (double)a[at], (double)b[at], (double)q[at], (double)(a[at] / b[at]));
    ok(hipFree(da));
    ok(hipFree(db));
    ok(hipFree(dq));
}

int main() {
    std::mt19937_64 rng(7);
    constexpr int N = 1 << 20;
    // a value of a random sign, significand and binary exponent of [lo, hi]
    auto value = [&](int lo, int hi) {
        std::uniform_int_distribution<int> ex(lo, hi);
        std::uniform_real_distribution<double> m(1.0, 2.0);
        const double v = std::ldexp(m(rng), ex(rng));
        return rng() & 1 ? -v : v;
    };
    // operands of a class, their quotients normal numbers of the type
    auto operands = [&](auto one, int a_lo, int a_hi, int b_lo, int b_hi) {
        using T = decltype(one);
        constexpr double lo = sizeof(T) == 8 ? 0x1p-1021 : 0x1p-125, hi = sizeof(T) == 8 ? 0x1p1023 : 0x1p127;
        std::vector<T> a, b;
        while ((int)a.size() < N) {
            const T n = (T)value(a_lo, a_hi), d = (T)value(b_lo, b_hi);
            const double e = std::fabs((double)n / (double)d);
            if (!(e >= lo && e <= hi)) continue;
            a.push_back(n);
            b.push_back(d);
        }
        return std::make_pair(a, b);
    };
    auto run = [&](const char* name, const auto& ab, int form = SINGLE) { check(name, ab.first, ab.second, form); };
    run("double_range", operands(1.0, -969, 1022, -1022, 1021));
    run("double_range_pair", operands(1.0, -969, 1022, -1022, 1021), PAIR);
    run("double_range_low_end", operands(1.0, -1000, 0, -1022, -1021));
    run("double_range_high_end", operands(1.0, 2, 1022, 1020, 1021));
    run("double_small_dividends", operands(1.0, -1074, -970, -1022, 0));
    run("float_range", operands(1.0f, -102, 126, -126, 125));
    run("float_range_low_end", operands(1.0f, -102, 0, -126, -125));
    run("float_range_high_end", operands(1.0f, 2, 126, 124, 125));
    run("float_small_dividends", operands(1.0f, -149, -103, -126, 0));
    run("float_field_subnormal", operands(1.0f, -149, 0, -149, -127), FIELD);
    run("float_field", operands(1.0f, -149, 126, -149, 127), FIELD);
    run("double_field", operands(1.0, -969, 1022, -1022, 1021), FIELD);
    // zeros, infinities and NaN with each other and with ordinary values
    auto specials = [&](auto one, const char* name, int form) {
        using T = decltype(one);
        const T s[] = {T(0), -T(0), T(INFINITY), -T(INFINITY), T(NAN), T(1), T(-3.5), T(1e-30), T(1e30)};
        std::vector<T> a, b;
        for (T x : s)
            for (T y : s) {
                a.push_back(x);
                b.push_back(y);
            }
        check(name, a, b, form);
    };
    specials(1.0, "double_specials", SINGLE);
    specials(1.0, "double_pair_specials", PAIR);
    specials(1.0f, "float_specials", SINGLE);
    specials(1.0f, "float_field_specials", FIELD);
    return 0;
}
