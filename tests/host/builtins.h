// The gfx950 builtins that the device headers use, for a host compiler: rounded to
// nearest, or (ULP) now to one and now to the other of the two floats around the exact
// value, always the same one for the same value, as the instructions may be.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

using std::isfinite;
using std::max;
using std::min;

inline float rounded(double v) {
    const float near = (float)v;
#ifdef ULP
    // the other float around v, one time in two, unless v is a float to a tenth of a unit
    const float other = std::nextafterf(near, v > (double)near ? INFINITY : -INFINITY);
    uint64_t h;
    std::memcpy(&h, &v, 8);
    h *= 0x9E3779B97F4A7C15ull;
    if (std::isfinite(near) && near != 0.0f && (h >> 63) && std::fabs(v - near) > 0.1 * std::fabs((double)other - near))
        return other;
#endif
    return near;
}

inline float __builtin_amdgcn_rcpf(float x) { return rounded(1.0 / (double)x); }
inline double __builtin_amdgcn_rcp(double x) { return 1.0 / x; }
inline float __builtin_amdgcn_logf(float x) { return rounded(std::log2((double)x)); }
inline float __builtin_amdgcn_exp2f(float x) { return rounded(std::exp2((double)x)); }
inline float __builtin_amdgcn_sqrtf(float x) { return rounded(std::sqrt((double)x)); }
inline float __builtin_amdgcn_ldexpf(float x, int n) { return std::ldexp(x, n); }
inline int __builtin_amdgcn_frexp_exp(double x) { int e; std::frexp(x, &e); return e; }
inline double __builtin_amdgcn_frexp_mant(double x) { int e; return std::frexp(x, &e); }
inline float cospif(float x) { return (float)std::cos(3.141592653589793 * (double)x); }

// Lanes of a quad run one after the other, in passes: a permutation gives the value that
// the other lane had at the same call in the pass before.
struct Quad {
    int lane = 0, at = 0;
    int now[4][64] = {}, before[4][64] = {};
    template <class F>
    void run(F&& lane_body, int passes) {
        for (int k = 0; k < passes; ++k) {
            std::memcpy(before, now, sizeof now);
            for (lane = 0; lane < 4; ++lane) {
                at = 0;
                lane_body(lane);
            }
        }
    }
};
inline Quad quad;

inline int __builtin_amdgcn_update_dpp(int, int v, int ctrl, int, int, bool) {
    const int from = ctrl == 0x00 ? 0 : ctrl == 0xB1 ? quad.lane ^ 1 : ctrl == 0x4E ? quad.lane ^ 2 : quad.lane;
    quad.now[quad.lane][quad.at] = v;
    return quad.before[from][quad.at++];
}
