// Checks the generator's binary64 functions (kb_math.hpp) on the host against
// 80-bit long double: the largest error of each, in units in the last place
// of binary64, on the ends of every reduction interval and on words spread
// over the range.  The seeds are off by 2^-23 either way, twice what the
// device's reciprocal and inverse square root instructions may be off.
// Prints one line per function: name, largest error, word (pair) it was at.
// With an argument instead: the binary32 functions of the 16-bit first pass
// (rho32, sincos32) where they are sure, against binary64, as relative errors
// in units of 2^-24; rho32 with the logarithm and the root as rounded, then
// both one unit in the last place too large, and too small.
#include <cmath>
#include <cstdio>
#include <vector>

#include "../paper_2608_02611_amd/csrc/kb_math.hpp"

namespace {

template <int SIGN>
struct Seed {
    static constexpr double off = 1.0 + SIGN * 0x1p-23;
    static double rcp(double x) { return 1.0 / x * off; }
    static double rsq(double x) { return 1.0 / std::sqrt(x) * off; }
    static double frexp_mant(double x) { int e; return std::frexp(x, &e); }
    static int frexp_exp(double x) { int e; std::frexp(x, &e); return e; }
    static double ldexp(double x, int n) { return std::ldexp(x, n); }
    // binary32: correctly rounded, then off by one unit in the last place
    // (SIGN 0: as rounded), as the device's logarithm and root may be
    static float step(float x) { return SIGN == 0 ? x : std::nextafter(x, SIGN > 0 ? INFINITY : -INFINITY); }
    static uint32_t to_u32(float x) { return x >= 0x1p32f ? 0xFFFFFFFFu : (uint32_t)x; }
    static float log2(float x) { return step((float)std::log2((double)x)); }
    static float sqrt32(float x) { return step((float)std::sqrt((double)x)); }
};

// |got - want| in units in the last place of binary64 at want.
double ulps(double got, long double want) {
    if (want == 0.0L) return got == 0.0 ? 0.0 : 1e300;
    int e;
    std::frexp((double)want, &e);
    return (double)(std::fabs((long double)got - want) / std::ldexp(1.0L, e - 53));
}

struct Worst {
    double u = 0.0;
    uint32_t at = 0;
    void see(double v, uint32_t x) {
        if (!(v <= u)) { u = v; at = x; }
    }
};

template <int SIGN>
void check(const std::vector<uint32_t>& words) {
    using S = Seed<SIGN>;
    Worst lg, root, sn, cs, t3;
    for (uint32_t x : words) {
        const double t = kb::neg2_log_u01<S>(x);
        // (log1p keeps the accuracy of the oracle value itself near u = 1)
        const long double m = (long double)x + 1.0L;
        const long double want = -2.0L * (x > 0xF0000000u ? log1pl((m - 0x1p32L) * 0x1p-32L) : logl(m * 0x1p-32L));
        lg.see(ulps(t, want), x);
        root.see(ulps(kb::math_sqrt<S>(t), sqrtl((long double)t)), x);
        double s, c;
        kb::sincos_2pi_u(x, s, c);
        const double theta = 6.283185307179586476925286766559 * ((double)x * 0x1p-32);
        sn.see(ulps(s, sinl((long double)theta)), x);
        cs.see(ulps(c, cosl((long double)theta)), x);
    }
    // Student-t: words three apart in the list, against the definition with
    // all four normals (any second angle)
    auto log2u = [](uint32_t x) {
        const long double m = (long double)x + 1.0L;
        return -2.0L * (x > 0xF0000000u ? log1pl((m - 0x1p32L) * 0x1p-32L) : logl(m * 0x1p-32L));
    };
    auto literal = [&](uint32_t x, uint32_t y, uint32_t z, uint32_t w) {
        const long double th = 6.283185307179586476925286766559 * ((double)y * 0x1p-32), ph = (long double)w * 1e-9L;
        const long double r1 = sqrtl(log2u(x)), r2 = sqrtl(log2u(z));
        const long double z1 = r1 * sinl(th), z2 = r2 * cosl(ph), z3 = r2 * sinl(ph);
        return r1 * cosl(th) / sqrtl((z1 * z1 + z2 * z2 + z3 * z3) / 3.0L);
    };
    for (size_t i = 0; i + 3 < words.size(); ++i) {
        const uint32_t x = words[i], y = words[i + 1], z = words[i + 2], w = words[i + 3];
        t3.see(ulps(kb::student_t3_64<S>(x, y, z), literal(x, y, z, w)), x);
    }
    // u = 1 in the first pair: zero; in the second with z1 = 0: a quotient by zero
    const uint32_t one = 0xFFFFFFFFu;
    const bool edges = kb::student_t3_64<S>(one, 77u, 5u) == 0.0 && std::isinf(kb::student_t3_64<S>(5u, 0u, one)) &&
                       std::isnan(kb::student_t3_64<S>(one, 0u, one));
    std::printf("edges %d 0\nstudent_t3 %.3f %08x\n", edges ? 0 : 1, t3.u, t3.at);
    std::printf("neg2_log %.3f %08x\nsqrt %.3f %08x\nsin %.3f %08x\ncos %.3f %08x\n", lg.u, lg.at, root.u, root.at,
                sn.u, sn.at, cs.u, cs.at);
}

}  // namespace

// The largest relative errors of the binary32 functions, over every 61st word
// and all words next to the multiples of 1/8 turn and the ends of the range.
template <int SIGN>
void check32() {
    double rho = 0.0, angle = 0.0;
    uint32_t rho_at = 0, angle_at = 0;
    auto see = [&](uint32_t x) {
        bool sure;
        const float r = kb::rho32<Seed<SIGN>>(x, sure);
        if (sure) {
            const double u = ((double)x + 1.0) * 0x1p-32;
            const double want = std::sqrt(-2.0 * (u > 0.75 ? std::log1p(((double)x + 1.0 - 0x1p32) * 0x1p-32) : std::log(u)));
            const double e = std::fabs((double)r - want) / want;
            if (!(e <= rho)) { rho = e; rho_at = x; }
        }
        if (SIGN != 0) return;
        float s, c;
        kb::sincos32(x, s, c, sure);
        if (sure) {
            const double theta = 6.283185307179586476925286766559 * ((double)x * 0x1p-32);
            const double e = std::fmax(std::fabs((s - std::sin(theta)) / std::sin(theta)),
                                       std::fabs((c - std::cos(theta)) / std::cos(theta)));
            if (!(e <= angle)) { angle = e; angle_at = x; }
        }
    };
    for (uint64_t x = 0; x < (1ull << 32); x += 61) see((uint32_t)x);
    for (uint32_t o = 0; o < 8; ++o)
        for (int32_t d = -100000; d <= 100000; ++d) see((o << 29) + (uint32_t)d);
    std::printf("rho32 %.3f %08x\n", rho * 0x1p24, rho_at);
    if (SIGN == 0) std::printf("sincos32 %.3f %08x\n", angle * 0x1p24, angle_at);
}

int main(int argc, char**) {
    if (argc > 1) {  // the binary32 functions only
        check32<0>();
        check32<1>();
        check32<-1>();
        return 0;
    }
    std::vector<uint32_t> words;
    // every power of two and every eighth of the circle, with neighbours
    for (int k = 0; k < 32; ++k)
        for (int d = -70; d <= 70; ++d) words.push_back((1u << k) + (uint32_t)d);
    for (uint32_t o = 0; o < 16; ++o)
        for (int d = -70; d <= 70; ++d) words.push_back((o << 28) + (uint32_t)d);
    // sqrt(1/2) of every binade, where the logarithm changes its exponent
    for (int k = 1; k < 33; ++k) {
        const uint32_t m = (uint32_t)(0.70710678118654752 * std::ldexp(1.0, k));
        for (int d = -70; d <= 70; ++d) words.push_back(m + (uint32_t)d);
    }
    uint64_t s = 0x9E3779B97F4A7C15ull;
    for (int i = 0; i < 1000000; ++i) {
        s ^= s << 13; s ^= s >> 7; s ^= s << 17;  // xorshift64
        words.push_back((uint32_t)(s >> 32));
        words.push_back((uint32_t)(s >> 32) >> (s & 31));
    }
    check<1>(words);
    check<-1>(words);
    return 0;
}
