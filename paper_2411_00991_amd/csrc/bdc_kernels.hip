// bdc_kernels.hip -- gfx950 kernels of the posterior sampler.
//
// One sweep = forward_propose (mu = P (x) rho from scratch, plus this sweep's
// proposals for every pixel) -> the colour or block-phase passes (footprint
// likelihood deltas, Metropolis decisions, mu commits) -> moments (Welford,
// batched R-hat statistics, per-chain log-posterior partials) -> finalize
// (deterministic reduction of the log-posterior, sweep index + 1).
// The sweep index lives in device memory so a captured sweep replays as is.
#include "bdc_bounds.h"
#include "bdc_conv.h"
#include "bdc_device.h"
#include "bdc_kernels.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace bdc {

namespace {

__device__ inline PixConst pc_of(float4 u) {
    PixConst p;
    p.c = u.x; p.a2 = u.y; p.L0 = u.z; p.iB = u.w;
    p.ks = fmaxf(p.c, 0.0f);
    p.inv2a = __builtin_amdgcn_rcpf(p.a2);
    p.h0 = __builtin_amdgcn_sqrtf(2.0f * TAIL_T * p.inv2a);
    return p;
}

__device__ inline PixConst load_pc(const float4* pc, int64_t n) {
    // 16-byte records; frames stay below 2^27 pixels, so a 32-bit byte offset
    // from the base suffices
    return pc_of(*reinterpret_cast<const float4*>(reinterpret_cast<const char*>(pc) + ((uint32_t)n << 4)));
}

// Per-pixel constants of the phi window from c and a (see PixConst).
__device__ inline PixConst make_pc(double c, double a) {
    PixConst p;
    const double ks = c > 0.0 ? c : 0.0;
    p.c = (float)c;
    p.a2 = (float)(2.0 * a);
    p.inv2a = (float)(0.5 / a);
    p.ks = (float)ks;
    p.L0 = (float)(2.0 * a * (c - ks) - log(ks + 1.0));
    p.iB = (float)(1.0 / (2.0 * a + 1.0 / (ks + 1.0)));
    p.h0 = (float)sqrt((double)TAIL_T / a);
    return p;
}

__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Workgroups go to the XCDs round-robin in dispatch order, and each XCD has
// its own L2.  The chains of one block of a block scan read the same per-pixel
// records, so the block scans map workgroup id to (block, chain) with id mod
// XCDS the XCD: the C chains of block XCDS * q + x are consecutive workgroups
// of XCD x, resident together, and the first chain's record reads leave the
// lines in that XCD's L2 for the others.  Ids past the last block get false
// (the workgroup exits at once).  Grid: xcd_grid(nblk, C).
__device__ inline bool xcd_block(int nblk, int C, int& bi, int& chain) {
    const int64_t id = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;   // dispatch order
    const int x = (int)(id % XCDS);
    const int64_t j = id / XCDS;
    const int64_t bl = XCDS * (j / C) + x;
    chain = (int)(j % C);
    bi = (int)min(bl, (int64_t)nblk);
    return bl < nblk;
}

// Camera value of pixel n (map or scalar).
__device__ inline float cam(const float* p, int per_pixel, int64_t n) { return per_pixel ? p[n] : p[0]; }

// log n! for an integer n >= 0: the log of the exact product below 20 (every
// partial product is exact in double), Stirling's series through the n^-7
// term from 20 on (truncation error below 2e-15).
__device__ inline double log_factorial(int n) {
    if (n < 20) {
        double p = 1.0;
        for (int i = 2; i <= n; ++i) p *= (double)i;
        return log(p);
    }
    const double x = (double)n, ix = rcp_nr(x), ix2 = ix * ix;
    const double corr = ix * (1.0 / 12.0 - ix2 * (1.0 / 360.0 - ix2 * (1.0 / 1260.0 - ix2 * (1.0 / 1680.0))));
    return (x + 0.5) * log(x) - x + 0.91893853320467274178 + corr;   // + log(2 pi) / 2
}

// Sharper read noise than the recurrence takes (a > A_RECUR_MAX, rare): a
// max-shifted log-sum-exp over the (short) window.
__device__ __noinline__ double ell_abs_sharp(double mu, double c, double a, double lnorm, int lo, int hi) {
    const double lmud = log(mu), lf_lo = log_factorial(lo);
    double mx = -INFINITY, lf = lf_lo;                 // lf = log k!
    for (int k = lo; k <= hi; ++k) {
        if (k > lo) lf += log((double)k);
        mx = fmax(mx, -a * (k - c) * (k - c) + k * lmud - lf);
    }
    double s = 0.0;
    lf = lf_lo;
    for (int k = lo; k <= hi; ++k) {
        if (k > lo) lf += log((double)k);
        s += exp(-a * (k - c) * (k - c) + k * lmud - lf - mx);
    }
    return lnorm - mu + mx + log(s);
}

// Absolute log-likelihood of one pixel in double precision (parity output and
// log-posterior trace).  a <= A_RECUR_MAX: Horner from the window top,
//   ell = lnorm - mu + log W_lo + log(1 + sum_{k>lo} W_k / W_lo),
//   log W_lo = -a (lo - c)^2 + lo log mu - log(lo!);
// sharper read noise: ell_abs_sharp.
__device__ inline double ell_abs(float muf, float wv, float gain, float o, float sig) {
    const double c = ((double)wv - (double)o) / (double)gain;
    const double a = (double)gain * (double)gain / (2.0 * (double)sig * (double)sig);
    const double lnorm = -0.5 * log(2.0 * M_PI * (double)sig * (double)sig);
    const double mu = (double)muf;
    if (!(mu > 0.0)) return lnorm - a * c * c;
    const PixConst pc = make_pc(c, a);
    const float lmu = logf(muf);
    const Window win = phi_window(lmu, lmu, pc);
    if (!win.ok) return __builtin_nan("");
    if (a > (double)A_RECUR_MAX) return ell_abs_sharp(mu, c, a, lnorm, win.lo, win.hi);
    const double lmud = log(mu);
    const double qi = exp(2.0 * a);
    double G = mu * exp(-a * (2.0 * (win.hi - 1) + 1.0 - 2.0 * c));
    double acc = 0.0;
#pragma unroll 1
    for (int k = win.hi - 1; k >= win.lo; --k) {
        const double r = G * rcp_nr((double)(k + 1));
        G *= qi;
        acc = fma(r, acc, r);
    }
    const double lo = (double)win.lo;
    const double logw_lo = -a * (lo - c) * (lo - c) + lo * lmud - log_factorial(win.lo);
    return lnorm - mu + logw_lo + log1p(acc);
}

// The same for an EMCCD pixel (bdc_device.h), in double from the raw inputs.
__device__ __noinline__ double ell_abs_emccd(float muf, float wv, float gain, float o, float sig) {
    const double c = ((double)wv - (double)o) / (double)gain;
    const double dw = (double)wv - (double)o, s2 = (double)sig * (double)sig;
    const double lA = -0.5 * log(2.0 * M_PI * s2) - dw * dw / (2.0 * s2);
    const double mu = (double)muf;
    if (!(mu > 0.0)) return lA;
    return emccd_lse(mu, c, lA, -c - log((double)gain)) - mu;
}

template <bool EM>
__device__ inline double ell_abs_cam(const Frame& f, float mu, int64_t n) {
    const float w = f.w[n], G = cam(f.gain, f.cam_per_pixel, n), o = cam(f.offset, f.cam_per_pixel, n),
                sg = cam(f.sigma, f.cam_per_pixel, n);
    if constexpr (EM) return ell_abs_emccd(mu, w, G, o, sg);
    else return ell_abs(mu, w, G, o, sg);
}

// ---------------------------------------------------------------------------
// Frame setup
// ---------------------------------------------------------------------------
__global__ void k_pixel_consts(Frame f, float4* pc, int* bad) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= f.Np) return;
    const float wv = f.w[n];
    const float G = cam(f.gain, f.cam_per_pixel, n);
    const float o = cam(f.offset, f.cam_per_pixel, n);
    const float sg = cam(f.sigma, f.cam_per_pixel, n);
    if (!isfinite(wv) || !isfinite(o) || !isfinite(G) || !isfinite(sg)) { atomicAdd(&bad[0], 1); return; }
    if (!(G > 0.0f) || !(sg > 0.0f)) { atomicAdd(&bad[1], 1); return; }
    const double c = ((double)wv - (double)o) / (double)G;
    if (f.camera == 1) {
        const double dw = (double)wv - (double)o, s2 = (double)sg * (double)sg;
        const double lA = -0.5 * log(2.0 * M_PI * s2) - dw * dw / (2.0 * s2);
        const double lB = c > 0.0 ? -c - log((double)G) : -INFINITY;
        pc[n] = make_float4((float)c, -1.0f, (float)lA, (float)lB);
        return;
    }
    const double a = (double)G * (double)G / (2.0 * (double)sg * (double)sg);
    const PixConst p = make_pc(c, a);
    pc[n] = make_float4(p.c, record_a2(p.a2), p.L0, p.iB);
}

__global__ void k_init_state(Frame f, State S, const float* rho0, float log_step0, int* bad) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int chain = blockIdx.y;
    if (n >= f.N) return;
    const int64_t i = (int64_t)chain * f.N + n;
    float v;
    if (rho0) {
        v = rho0[i];
        if (!(v > 0.0f) || !isfinite(v)) { atomicAdd(&bad[0], 1); v = 1.0f; }
    } else if (f.sub == 1) {
        const float c = f.pc[n].x;
        const float xi = box_muller(draw(f.key, (uint32_t)n, 0u, (uint32_t)chain, STREAM_INIT));
        v = fmaxf(c, 0.5f) * expf(0.5f * xi);
    } else {
        // a pixel's photon estimate shared by its k x k cells
        const int y = (int)(n / f.W), x = (int)(n % f.W);
        const float c = f.pc[(int64_t)(y / f.sub) * f.Wp + x / f.sub].x;
        const float xi = box_muller(draw(f.key, (uint32_t)n, 0u, (uint32_t)chain, STREAM_INIT));
        v = fmaxf(c, 0.5f) / (float)(f.sub * f.sub) * expf(0.5f * xi);
    }
    S.rho[i] = v;
    S.log_step[i] = log_step0;
}

// ---------------------------------------------------------------------------
// mu = P (x) rho (bdc_conv.h, double accumulation) and this sweep's
// proposals: rho' = rho exp(step xi), step = exp(log_step), xi ~ N(0, 1) from
// stream 0; Hastings + prior terms; log u from stream 1.
// ---------------------------------------------------------------------------
// This sweep's proposal for object cell m of one chain (current value r0).
__device__ inline void propose_cell(const Frame& f, const State& S, const Prior& pr, int64_t m, int chain,
                                    int64_t t, float r0) {
    const int64_t i = (int64_t)chain * f.N + m;
    const float xi = box_muller(draw(f.key, (uint32_t)m, (uint32_t)t, (uint32_t)chain, STREAM_PROPOSAL));
    const float step = expf(S.log_step[i]);
    const float hs = step * xi;                 // log rho' - log rho
    const float e = expf(hs), rp = mul_rn(r0, e);
    float hast = hs;
    if (pr.kind == 1) hast = fmaf(step, xi, fmaf(pr.a - 1.0f, hs, -(pr.b * fmaf(r0, e, -r0))));
    if (!(rp > 0.0f) || !isfinite(rp)) hast = -INFINITY;
    S.prop[i] = make_float4(rp, hast, logf(u01(draw(f.key, (uint32_t)m, (uint32_t)t, (uint32_t)chain, STREAM_ACCEPT).x)),
                            add_rn(rp, -r0));
}

// One output tile of one chain.
template <class T>
__device__ inline void forward_tile(const Frame& f, const State& S, const Prior& pr, int propose, int tile, int chain,
                                    int64_t t, float* lds) {
    const float* rho = S.rho + (int64_t)chain * f.N;
    T::run(f.H, f.W, f.r, f.psf64, tile, lds, [&](int y, int x) { return rho[(int64_t)y * f.W + x]; },
           [&](int y, int x, double sum) {
               const int64_t m = (int64_t)y * f.W + x;
               S.mu[(int64_t)chain * f.N + m] = (float)sum;
               if (propose) propose_cell(f, S, pr, m, chain, t, rho[m]);
           });
}

template <class T>
__global__ void __launch_bounds__(WG) k_forward_propose(Frame f, State S, Prior pr, int propose) {
    extern __shared__ float lds_f[];
    forward_tile<T>(f, S, pr, propose, blockIdx.x, blockIdx.y, *S.t, lds_f);
}

// Finer object lattice (sub = k > 1): pixel n's mean, FP64 accumulation over
// the k^2 phases and the footprint, mu_n = sum_phase sum_d T_phase[d] rho(cell
// of that phase in pixel n - d).
__global__ void __launch_bounds__(WG) k_forward_sub(Frame f, State S) {
    const int64_t n = (int64_t)blockIdx.x * WG + threadIdx.x;
    const int chain = blockIdx.y;
    if (n >= f.Np) return;
    const int k = f.sub, s = f.s, r = f.r;
    const int py = (int)(n / f.Wp), px = (int)(n % f.Wp);
    const float* rho = S.rho + (int64_t)chain * f.N;
    double acc = 0.0;
    for (int ph = 0; ph < k * k; ++ph) {
        const float* T = f.psf + (int64_t)ph * s * s;
        const int a = ph / k, b = ph % k;
        for (int dy = -r; dy <= r; ++dy) {
            const int qy = py - dy;
            if (qy < 0 || qy >= f.Hp) continue;
            for (int dx = -r; dx <= r; ++dx) {
                const int qx = px - dx;
                if (qx < 0 || qx >= f.Wp) continue;
                acc = fma((double)T[(dy + r) * s + dx + r], (double)rho[(int64_t)(qy * k + a) * f.W + qx * k + b], acc);
            }
        }
    }
    S.mu[(int64_t)chain * f.Np + n] = (float)acc;
}

// This sweep's proposals for every object cell (sub > 1).
__global__ void __launch_bounds__(WG) k_propose_sub(Frame f, State S, Prior pr) {
    const int64_t m = (int64_t)blockIdx.x * WG + threadIdx.x;
    const int chain = blockIdx.y;
    if (m >= f.N) return;
    propose_cell(f, S, pr, m, chain, *S.t, S.rho[(int64_t)chain * f.N + m]);
}

// Decision shared by both scans: accept iff Delta finite and log u < Delta;
// commits rho, adapts the step during burn-in, counts, records for parity.
// hast, logu, rp: this pixel's Hastings + prior term, log u and proposal
// (loaded ahead by the caller, off the decision's critical path).
__device__ inline bool decide_commit(const Frame& f, const State& S, int chain, int64_t m, int64_t t, int burn_in,
                                     double tot, bool writer, float hast, float logu, float rp, float* dbg_delta,
                                     uint8_t* dbg_acc) {
    const int64_t i = (int64_t)chain * f.N + m;
    const double delta = tot + (double)hast;
    const bool acc = isfinite(delta) && ((double)logu < delta);
    if (writer) {
        if (acc) {
            S.rho[i] = rp;
            atomicAdd(&S.accepts[chain], 1ull);
        }
        if (t < burn_in) {
            const float gain = exp2f(-0.6f * log2f((float)t + 1.0f));
            S.log_step[i] = fmaf(gain, (acc ? 1.0f : 0.0f) - 0.44f, S.log_step[i]);
        }
        if (dbg_delta) dbg_delta[i] = (float)delta;
        if (dbg_acc) dbg_acc[i] = acc ? 1 : 0;
    }
    return acc;
}

__device__ inline bool decide_and_commit(const Frame& f, const State& S, int chain, int64_t m, int64_t t,
                                         int burn_in, double tot, bool writer,
                                         float* dbg_delta, uint8_t* dbg_acc) {
    const int64_t i = (int64_t)chain * f.N + m;
    const float4 pr = S.prop[i];
    return decide_commit(f, S, chain, m, t, burn_in, tot, writer, pr.y, pr.z, pr.x, dbg_delta, dbg_acc);
}

// ---------------------------------------------------------------------------
// Pixel-chromatic pass: one colour (cy, cx) of the s x s colouring; one
// workgroup per (active pixel, chain); footprint spread over the workgroup.
// ---------------------------------------------------------------------------
__device__ inline void count_work(unsigned long long* ctr, int terms, int evals) {
    unsigned long long t = (unsigned long long)terms, e = (unsigned long long)evals;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        t += __shfl_xor(t, off, 64);
        e += __shfl_xor(e, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&ctr[0], t);
        atomicAdd(&ctr[1], e);
    }
}

template <bool EM>
__global__ void __launch_bounds__(WG) k_colour_pass(Frame f, State S, int burn_in, const double* inv_tab,
                                                    int cy, int cx, float* dbg_delta, uint8_t* dbg_acc) {
    __shared__ double s_red[WG / 64];
    __shared__ int s_acc;
    const int s = f.s, r = f.r, F = s * s;
    const int ncol = (f.W - cx + s - 1) / s;
    const int y = cy + s * (blockIdx.x / ncol), x = cx + s * (blockIdx.x % ncol);
    const int chain = blockIdx.y;
    const int64_t m = (int64_t)y * f.W + x;
    const int64_t base = (int64_t)chain * f.N;
    const float d = S.prop[base + m].w;
    const float* mu = S.mu + base;
    double part = 0.0;
    int nterms = 0, nevals = 0;
    for (int j = threadIdx.x; j < F; j += WG) {
        const int ny = y + j / s - r, nx = x + j % s - r;
        if (ny < 0 || ny >= f.H || nx < 0 || nx >= f.W) continue;
        const int64_t n = (int64_t)ny * f.W + nx;
        part += delta_pix<EM>(mu[n], mul_rn(d, f.psf[j]), load_pc(f.pc, n), inv_tab, nterms);
        ++nevals;
    }
    count_work(S.counters, nterms, nevals);
    part = wave_sum(part);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = part;
    __syncthreads();
    const int64_t t = *S.t;
    if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int w = 0; w < WG / 64; ++w) tot += s_red[w];
        s_acc = decide_and_commit(f, S, chain, m, t, burn_in, tot, true, dbg_delta, dbg_acc) ? 1 : 0;
    }
    __syncthreads();
    if (s_acc) {
        float* muw = S.mu + base;
        for (int j = threadIdx.x; j < F; j += WG) {
            const int ny = y + j / s - r, nx = x + j % s - r;
            if (ny < 0 || ny >= f.H || nx < 0 || nx >= f.W) continue;
            float& m = muw[(int64_t)ny * f.W + nx];
            m = fmaf(d, f.psf[j], m);
        }
    }
}

// Pixel-chromatic pass over a finer object lattice (sub = k > 1): the cells of
// one phase (a, b) in the pixels (cy + s i, cx + s j); cell m's footprint is
// the s x s pixels around its own with weights T_phase.
template <bool EM>
__global__ void __launch_bounds__(WG) k_colour_pass_sub(Frame f, State S, int burn_in, const double* inv_tab,
                                                        int phase, int cy, int cx, float* dbg_delta,
                                                        uint8_t* dbg_acc) {
    __shared__ double s_red[WG / 64];
    __shared__ int s_acc;
    const int s = f.s, r = f.r, F = s * s, k = f.sub;
    const int ncol = (f.Wp - cx + s - 1) / s;
    const int py = cy + s * (blockIdx.x / ncol), px = cx + s * (blockIdx.x % ncol);
    const int chain = blockIdx.y;
    const int64_t m = (int64_t)(py * k + phase / k) * f.W + (px * k + phase % k);
    const int64_t base = (int64_t)chain * f.N, pbase = (int64_t)chain * f.Np;
    const float* T = f.psf + (int64_t)phase * F;
    const float d = S.prop[base + m].w;
    const float* mu = S.mu + pbase;
    double part = 0.0;
    int nterms = 0, nevals = 0;
    for (int j = threadIdx.x; j < F; j += WG) {
        const int ny = py + j / s - r, nx = px + j % s - r;
        if (ny < 0 || ny >= f.Hp || nx < 0 || nx >= f.Wp) continue;
        const int64_t n = (int64_t)ny * f.Wp + nx;
        part += delta_pix<EM>(mu[n], mul_rn(d, T[j]), load_pc(f.pc, n), inv_tab, nterms);
        ++nevals;
    }
    count_work(S.counters, nterms, nevals);
    part = wave_sum(part);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = part;
    __syncthreads();
    const int64_t t = *S.t;
    if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int w = 0; w < WG / 64; ++w) tot += s_red[w];
        s_acc = decide_and_commit(f, S, chain, m, t, burn_in, tot, true, dbg_delta, dbg_acc) ? 1 : 0;
    }
    __syncthreads();
    if (s_acc) {
        float* muw = S.mu + pbase;
        for (int j = threadIdx.x; j < F; j += WG) {
            const int ny = py + j / s - r, nx = px + j % s - r;
            if (ny < 0 || ny >= f.Hp || nx < 0 || nx >= f.Wp) continue;
            float& m = muw[(int64_t)ny * f.Wp + nx];
            m = fmaf(d, T[j], m);
        }
    }
}

// ---------------------------------------------------------------------------
// Block-phase pass.  The frame is cut into B x B blocks; blocks whose
// (row, col) parities equal the phase are >= B + 1 >= s pixels apart, so their
// footprint regions (block + r halo) are disjoint and each workgroup owns its
// region's mu in LDS for the whole phase, running the s*s intra-block colours
// [k0, k1) in order with workgroup barriers only.
// ---------------------------------------------------------------------------
constexpr int MAX_ACT = 16;   // active pixels per colour per block (B <= 4 s)

// Divergence control.  A wave's phi-term loop runs as long as its longest
// window, and a pixel's window length is set mostly by a per-pixel constant,
// the half-width h0 = sqrt(T / a) of its read noise.  With one active pixel
// per colour (B <= s, the usual block), every wave sorts its own footprint
// evaluations by the class floor(h0) (a counting sort in wave-private LDS, no
// workgroup barrier) and its lanes take them in that order, so the 64 windows
// evaluated together have nearly the same length.
constexpr int NCLS = 16;           // window classes
constexpr int SORT_MAX_F = 4 * WG; // footprints up to 32 x 32 take the sorted path
constexpr int WAVES = WG / 64;

struct WaveSort {                  // per-wave scratch in LDS
    int hist[NCLS];
    int base[NCLS];
    int count;
    uint16_t order[SORT_MAX_F / WAVES];
};

// (EMCCD pixels carry no window: their h0 is NaN, class 0)
__device__ inline int window_class(float h0) { return h0 >= 0.0f ? min(NCLS - 1, (int)h0) : 0; }

__device__ inline void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Workgroup barrier that orders LDS only.  __syncthreads() also waits for every
// outstanding global load and store of the wave; the block-series pass passes
// no global data between its threads, so its barriers leave global traffic
// (the decision inputs fetched one update ahead, thread 0's commits) in flight.
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---------------------------------------------------------------------------
// Dirichlet-OTF prior per chunk (Methods, Prior, Eqs. 7-8).  A chunk is one
// B x B block of the block-phase scan (edge chunks smaller); its prior is the
// Dirichlet of x_k = |F_k| / sum_j |F_j| with concentration alpha_k (the
// normalised |OTF| on the chunk's grid, tabulated per chunk shape by the host),
//   F_k = sum_m rho_m exp(-2 pi i (ky y / th + kx x / tw)).
// A move rho_m -> rho_m + d changes every F_k by d w_k(m), w_k(m) =
// exp(-2 pi i (ky y_m / th + kx x_m / tw)), so with p_k = Re(F_k conj(w_k)),
//   |F_k'|^2 = |F_k|^2 (1 + u_k),  u_k = d (2 p_k + d) / |F_k|^2,
// and the change of the log prior is
//   sum_k (alpha_k - 1) log(1 + u_k) / 2  -  (sum_k (alpha_k - 1)) log(S' / S)
// with S = sum_k |F_k|, S' - S = sum_k d (2 p_k + d) / (|F_k'| + |F_k|): both
// sums free of cancellation, so FP32 terms keep their relative accuracy.  The
// spectrum is kept in FP64: a move can nearly cancel a component (|F'| << |F|),
// and log|F'| then needs F' to more digits than FP32 holds.
// ---------------------------------------------------------------------------
constexpr int DIR_MAX_B = 32;                 // chunk side (B <= s <= 31 with this prior)

struct ChunkGeom { int y0, x0, th, tw, shape; };

__device__ inline ChunkGeom chunk_geom(const Frame& f, int ci) {
    const int B = f.dir_B, ncx = (f.W + B - 1) / B;
    const int cy = ci / ncx, cx = ci - cy * ncx;
    ChunkGeom g;
    g.y0 = cy * B;
    g.x0 = cx * B;
    g.th = min(B, f.H - g.y0);
    g.tw = min(B, f.W - g.x0);
    g.shape = (g.th < B ? 2 : 0) + (g.tw < B ? 1 : 0);
    return g;
}

// a - b floor(a / b) for 0 <= a < 2^20, b >= 1 (exact in FP32 arithmetic)
__device__ inline int small_mod(int a, int b, float inv_b) {
    const int q = (int)(((float)a + 0.5f) * inv_b);
    return a - b * q;
}

// One block (index bi among the blocks of phase (py, px)) of one chain.
// lds: block_phase_lds(B, s) bytes, 8-byte aligned.
template <bool EM>
__device__ void block_phase_block(const Frame& f, const State& S, int burn_in, const double* inv_tab, int B,
                                  int py, int px, int bi, int chain, int64_t t, int k0, int k1,
                                  float* dbg_delta, uint8_t* dbg_acc, double* lds_d) {
    const int s = f.s, r = f.r, F = s * s;
    const int RW = B + 2 * r;
    double* s_inv = lds_d;                                   // [INV_TABLE]
    double* s_red = s_inv + INV_TABLE;                       // [MAX_ACT][WG/64]
    float* s_psf = (float*)(s_red + MAX_ACT * (WG / 64));   // [F]
    float* s_mu = s_psf + F;                                 // [RW*RW], -1 outside the frame
    uint16_t* s_off = (uint16_t*)(s_mu + RW * RW);           // [F]: (dy + r) | (dx + r) << 8
    uint8_t* s_cls = (uint8_t*)(s_off + F);                  // [RW*RW] window class
    __shared__ float s_d[MAX_ACT];                           // rho' - rho of the colour's pixels
    __shared__ WaveSort s_ws[WAVES];

    const int nbx = (f.W + B - 1) / B;
    const int nbx_p = (nbx - px + 1) / 2;
    const int by = py + 2 * (bi / nbx_p), bx = px + 2 * (bi % nbx_p);
    const int by0 = by * B, bx0 = bx * B;
    const int bh = min(B, f.H - by0), bw = min(B, f.W - bx0);
    const int64_t base = (int64_t)chain * f.N;
    const int ry0 = by0 - r, rx0 = bx0 - r;
    const bool sorted = F <= SORT_MAX_F;

    for (int i = threadIdx.x; i < INV_TABLE; i += WG) s_inv[i] = inv_tab[i];
    for (int j = threadIdx.x; j < F; j += WG) {
        s_psf[j] = f.psf[j];
        s_off[j] = (uint16_t)((j / s) | ((j % s) << 8));
    }
    for (int i = threadIdx.x; i < RW * RW; i += WG) {
        const int yy = ry0 + i / RW, xx = rx0 + i % RW;
        const bool in = yy >= 0 && yy < f.H && xx >= 0 && xx < f.W;
        const int64_t n = (int64_t)yy * f.W + xx;
        s_mu[i] = in ? S.mu[base + n] : -1.0f;
        if (sorted)
            s_cls[i] = in ? (uint8_t)window_class(__builtin_amdgcn_sqrtf(2.0f * TAIL_T / f.pc[n].y)) : 0;
    }
    __syncthreads();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    WaveSort& ws = s_ws[wave];
    int nterms = 0, nevals = 0;

    for (int k = k0; k < k1; ++k) {
        const int ky = k / s, kx = k - (k / s) * s;
        const int nay = bh > ky ? (bh - 1 - ky) / s + 1 : 0;
        const int nax = bw > kx ? (bw - 1 - kx) / s + 1 : 0;
        const int nact = nay * nax;
        if (nact == 0) continue;                              // uniform over the workgroup
        float pre_hast = 0.0f, pre_logu = 0.0f, pre_rp = 0.0f;   // the single pixel's decision inputs
        if (nact == 1 && sorted) {
            const int ly = ky, lx = kx;
            const int64_t m = (int64_t)(by0 + ly) * f.W + (bx0 + lx);
            const float4 pr = S.prop[base + m];
            pre_rp = pr.x;
            pre_hast = pr.y;
            pre_logu = pr.z;
            const float d = pr.w;
            if (threadIdx.x == 0) s_d[0] = d;
            const int rbase = ly * RW + lx;
            // counting sort of this wave's evaluations by window class
            if (lane < NCLS) ws.hist[lane] = 0;
            wave_fence();
            int key[SORT_MAX_F / WG], rank[SORT_MAX_F / WG];
#pragma unroll
            for (int q = 0; q < SORT_MAX_F / WG; ++q) {
                const int j = threadIdx.x + q * WG;
                key[q] = -1;
                rank[q] = 0;
                if (j < F) {
                    const int o = s_off[j];
                    const int ri = rbase + (o & 0xFF) * RW + (o >> 8);
                    if (s_mu[ri] >= 0.0f) {
                        key[q] = s_cls[ri];
                        rank[q] = atomicAdd(&ws.hist[key[q]], 1);
                    }
                }
            }
            wave_fence();
            if (lane < NCLS) {
                int b = 0;
                for (int c = 0; c < lane; ++c) b += ws.hist[c];
                ws.base[lane] = b;
                if (lane == NCLS - 1) ws.count = b + ws.hist[NCLS - 1];
            }
            wave_fence();
#pragma unroll
            for (int q = 0; q < SORT_MAX_F / WG; ++q)
                if (key[q] >= 0) ws.order[ws.base[key[q]] + rank[q]] = (uint16_t)(threadIdx.x + q * WG);
            wave_fence();
            const int V = ws.count;
            double part = 0.0;
            for (int p = lane; p < V; p += 64) {
                const int j = ws.order[p];
                const int o = s_off[j], oy = o & 0xFF, ox = o >> 8;
                const float muv = s_mu[rbase + oy * RW + ox];
                const int64_t n = m + (int64_t)(oy - r) * f.W + (ox - r);
                part += delta_pix<EM>(muv, mul_rn(d, s_psf[j]), load_pc(f.pc, n), s_inv, nterms);
                ++nevals;
            }
            part = wave_sum(part);
            if (lane == 0) s_red[wave] = part;
        } else {
            for (int a = 0; a < nact; ++a) {
                const int ly = ky + s * (a / nax), lx = kx + s * (a % nax);
                const int64_t m = (int64_t)(by0 + ly) * f.W + (bx0 + lx);
                const float d = S.prop[base + m].w;
                if (threadIdx.x == 0) s_d[a] = d;
                const int rbase = ly * RW + lx;                   // footprint origin in the region
                double part = 0.0;
                for (int j = threadIdx.x; j < F; j += WG) {
                    const int o = s_off[j], oy = o & 0xFF, ox = o >> 8;
                    const float muv = s_mu[rbase + oy * RW + ox];
                    if (muv < 0.0f) continue;                     // outside the frame
                    const int64_t n = m + (int64_t)(oy - r) * f.W + (ox - r);
                    part += delta_pix<EM>(muv, mul_rn(d, s_psf[j]), load_pc(f.pc, n), s_inv, nterms);
                    ++nevals;
                }
                part = wave_sum(part);
                if ((threadIdx.x & 63) == 0) s_red[a * (WG / 64) + wave] = part;
            }
        }
        __syncthreads();
        for (int a = 0; a < nact; ++a) {
            const int ly = ky + s * (a / nax), lx = kx + s * (a % nax);
            const int64_t m = (int64_t)(by0 + ly) * f.W + (bx0 + lx);
            double tot = 0.0;
            for (int w = 0; w < WG / 64; ++w) tot += s_red[a * (WG / 64) + w];
            const float d = s_d[a];
            const bool acc = (nact == 1 && sorted)
                ? decide_commit(f, S, chain, m, t, burn_in, tot, threadIdx.x == 0, pre_hast, pre_logu, pre_rp,
                                dbg_delta, dbg_acc)
                : decide_and_commit(f, S, chain, m, t, burn_in, tot, threadIdx.x == 0, dbg_delta, dbg_acc);
            if (acc) {
                const int rbase = ly * RW + lx;
                for (int j = threadIdx.x; j < F; j += WG) {
                    const int o = s_off[j];
                    const int ri = rbase + (o & 0xFF) * RW + (o >> 8);
                    const float muv = s_mu[ri];
                    if (muv < 0.0f) continue;
                    s_mu[ri] = fmaf(d, s_psf[j], muv);
                }
            }
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < RW * RW; i += WG) {
        const int yy = ry0 + i / RW, xx = rx0 + i % RW;
        if (yy >= 0 && yy < f.H && xx >= 0 && xx < f.W) S.mu[base + (int64_t)yy * f.W + xx] = s_mu[i];
    }
    count_work(S.counters, nterms, nevals);
}

template <bool EM>
__global__ void __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(5))) k_block_phase(Frame f, State S, int burn_in, const double* inv_tab,
                                                    int B, int py, int px, int k0, int k1,
                                                    float* dbg_delta, uint8_t* dbg_acc, int nblk) {
    extern __shared__ double lds_d[];
    int bi, chain;
    if (!xcd_block(nblk, f.C, bi, chain)) return;
    block_phase_block<EM>(f, S, burn_in, inv_tab, B, py, px, bi, chain, *S.t, k0, k1, dbg_delta, dbg_acc,
                                 lds_d);
}

// Block-phase pass over a finer object lattice (sub = k > 1): blocks of B x B
// pixels of one phase (py, px); the block's region of pixel means (block plus
// an r halo) lives in LDS for the whole phase, and the colours [k0, k1) of the
// k^2 s^2 within-block colours (cell phase major, then the pixel position mod
// s, as in the pixel-chromatic scan) run in order, each with one cell per
// active pixel position, the footprint weighted by its phase's table.
// lds: block_phase_sub_lds(B, s, k) bytes.
template <bool EM>
__global__ void __launch_bounds__(WG) k_block_phase_sub(Frame f, State S, int burn_in, const double* inv_tab, int B,
                                                        int py, int px, int k0, int k1, float* dbg_delta,
                                                        uint8_t* dbg_acc, int nblk) {
    extern __shared__ double lds_d[];
    const int s = f.s, r = f.r, F = s * s, k = f.sub, KF = k * k * F;
    const int RW = B + 2 * r;
    double* s_inv = lds_d;                                   // [INV_TABLE]
    double* s_red = s_inv + INV_TABLE;                       // [MAX_ACT][WAVES]
    float* s_psf = (float*)(s_red + MAX_ACT * WAVES);        // [k^2][F]
    float* s_mu = s_psf + KF;                                // [RW*RW], -1 outside the frame
    uint16_t* s_off = (uint16_t*)(s_mu + RW * RW);           // [F]: (dy + r) | (dx + r) << 8
    __shared__ float s_d[MAX_ACT];
    int bi, chain;
    if (!xcd_block(nblk, f.C, bi, chain)) return;
    const int nbx = (f.Wp + B - 1) / B;
    const int nbx_p = (nbx - px + 1) / 2;
    const int by = py + 2 * (bi / nbx_p), bx = px + 2 * (bi % nbx_p);
    const int by0 = by * B, bx0 = bx * B;
    const int bh = min(B, f.Hp - by0), bw = min(B, f.Wp - bx0);
    const int64_t base = (int64_t)chain * f.N, pbase = (int64_t)chain * f.Np;
    const int ry0 = by0 - r, rx0 = bx0 - r;
    const int64_t t = *S.t;
    const int wave = threadIdx.x >> 6;

    for (int i = threadIdx.x; i < INV_TABLE; i += WG) s_inv[i] = inv_tab[i];
    for (int j = threadIdx.x; j < KF; j += WG) s_psf[j] = f.psf[j];
    for (int j = threadIdx.x; j < F; j += WG) s_off[j] = (uint16_t)((j / s) | ((j % s) << 8));
    for (int i = threadIdx.x; i < RW * RW; i += WG) {
        const int yy = ry0 + i / RW, xx = rx0 + i % RW;
        const bool in = yy >= 0 && yy < f.Hp && xx >= 0 && xx < f.Wp;
        s_mu[i] = in ? S.mu[pbase + (int64_t)yy * f.Wp + xx] : -1.0f;
    }
    __syncthreads();
    int nterms = 0, nevals = 0;
    for (int c = k0; c < k1; ++c) {
        const int ph = c / F, kk = c - ph * F;
        const int ky = kk / s, kx = kk - (kk / s) * s;
        const int nay = bh > ky ? (bh - 1 - ky) / s + 1 : 0;
        const int nax = bw > kx ? (bw - 1 - kx) / s + 1 : 0;
        const int nact = nay * nax;
        if (nact == 0) continue;                              // uniform over the workgroup
        const float* T = s_psf + ph * F;
        for (int a = 0; a < nact; ++a) {
            const int ly = ky + s * (a / nax), lx = kx + s * (a % nax);
            const int64_t m = (int64_t)((by0 + ly) * k + ph / k) * f.W + ((bx0 + lx) * k + ph % k);
            const float d = S.prop[base + m].w;
            if (threadIdx.x == 0) s_d[a] = d;
            const int rbase = ly * RW + lx;                   // footprint origin in the region
            double part = 0.0;
            for (int j = threadIdx.x; j < F; j += WG) {
                const int o = s_off[j], oy = o & 0xFF, ox = o >> 8;
                const float muv = s_mu[rbase + oy * RW + ox];
                if (muv < 0.0f) continue;                     // outside the frame
                const int64_t n = (int64_t)(by0 + ly + oy - r) * f.Wp + (bx0 + lx + ox - r);
                part += delta_pix<EM>(muv, mul_rn(d, T[j]), load_pc(f.pc, n), s_inv, nterms);
                ++nevals;
            }
            part = wave_sum(part);
            if ((threadIdx.x & 63) == 0) s_red[a * WAVES + wave] = part;
        }
        __syncthreads();
        for (int a = 0; a < nact; ++a) {
            const int ly = ky + s * (a / nax), lx = kx + s * (a % nax);
            const int64_t m = (int64_t)((by0 + ly) * k + ph / k) * f.W + ((bx0 + lx) * k + ph % k);
            double tot = 0.0;
            for (int w = 0; w < WAVES; ++w) tot += s_red[a * WAVES + w];
            const float d = s_d[a];
            if (decide_and_commit(f, S, chain, m, t, burn_in, tot, threadIdx.x == 0, dbg_delta, dbg_acc)) {
                const int rbase = ly * RW + lx;
                for (int j = threadIdx.x; j < F; j += WG) {
                    const int o = s_off[j];
                    const int ri = rbase + (o & 0xFF) * RW + (o >> 8);
                    const float muv = s_mu[ri];
                    if (muv < 0.0f) continue;
                    s_mu[ri] = fmaf(d, T[j], muv);
                }
            }
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < RW * RW; i += WG) {
        const int yy = ry0 + i / RW, xx = rx0 + i % RW;
        if (yy >= 0 && yy < f.Hp && xx >= 0 && xx < f.Wp) S.mu[pbase + (int64_t)yy * f.Wp + xx] = s_mu[i];
    }
    count_work(S.counters, nterms, nevals);
}

// Every chunk's spectrum (MODE 0: into f.dir_F) or log prior (MODE 1: into
// M.dir_part) for one chain: DFT sums in FP64, rows then columns.  One
// workgroup per (chunk, chain).  LDS: chunk_fourier_lds(B) bytes.
template <int MODE>
__global__ void __launch_bounds__(WG) k_chunk_fourier(Frame f, State S, MomentBufs M) {
    extern __shared__ double lds_c[];
    const int ci = blockIdx.x, chain = blockIdx.y;
    const ChunkGeom g = chunk_geom(f, ci);
    const int K = g.th * g.tw;
    double* r = lds_c;                         // [K] rho, later |F|
    double* gre = r + K;                       // [K] row transforms
    double* gim = gre + K;
    double* cth = gim + K;                     // cos, sin (2 pi j / th), (2 pi j / tw)
    double* sth = cth + g.th;
    double* ctw = sth + g.th;
    double* stw = ctw + g.tw;
    double* red = stw + g.tw;                  // [WAVES]
    const int64_t base = (int64_t)chain * f.N;
    for (int i = threadIdx.x; i < K; i += WG) {
        const int y = i / g.tw, x = i - (i / g.tw) * g.tw;
        r[i] = (double)S.rho[base + (int64_t)(g.y0 + y) * f.W + (g.x0 + x)];
    }
    for (int j = threadIdx.x; j < g.th; j += WG) sincospi(2.0 * j / g.th, &sth[j], &cth[j]);
    for (int j = threadIdx.x; j < g.tw; j += WG) sincospi(2.0 * j / g.tw, &stw[j], &ctw[j]);
    __syncthreads();
    for (int i = threadIdx.x; i < K; i += WG) {
        const int y = i / g.tw, kx = i - (i / g.tw) * g.tw;
        double re = 0.0, im = 0.0;
        int idx = 0;
        for (int x = 0; x < g.tw; ++x) {
            const double v = r[y * g.tw + x];
            re = fma(v, ctw[idx], re);
            im = fma(-v, stw[idx], im);
            idx += kx;
            if (idx >= g.tw) idx -= g.tw;
        }
        gre[i] = re;
        gim[i] = im;
    }
    __syncthreads();
    double sab = 0.0;
    for (int i = threadIdx.x; i < K; i += WG) {
        const int ky = i / g.tw, kx = i - (i / g.tw) * g.tw;
        double re = 0.0, im = 0.0;
        int idx = 0;
        for (int y = 0; y < g.th; ++y) {
            const double a = gre[y * g.tw + kx], b = gim[y * g.tw + kx], cs = cth[idx], sn = sth[idx];
            re += a * cs + b * sn;
            im += b * cs - a * sn;
            idx += ky;
            if (idx >= g.th) idx -= g.th;
        }
        if (MODE == 0) {
            f.dir_F[base + (int64_t)(g.y0 + ky) * f.W + (g.x0 + kx)] = make_double2(re, im);
        } else {
            r[i] = sqrt(re * re + im * im);
            sab += r[i];
        }
    }
    if (MODE == 0) return;
    sab = wave_sum(sab);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sab;
    __syncthreads();
    double Ssum = 0.0;
    for (int w = 0; w < WAVES; ++w) Ssum += red[w];
    __syncthreads();
    const float* am = f.dir_am1 + (size_t)g.shape * f.dir_B * f.dir_B;
    double lp = 0.0;
    for (int i = threadIdx.x; i < K; i += WG) lp += (double)am[i] * log(r[i] / Ssum);
    lp = wave_sum(lp);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = lp;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = f.dir_const[g.shape];
        for (int w = 0; w < WAVES; ++w) t += red[w];
        M.dir_part[(int64_t)ci * f.C + chain] = t;
    }
}

// ---------------------------------------------------------------------------
// Block-series pass: the block-phase scan for blocks with one active pixel per
// colour (B <= s), where each footprint pixel's likelihood change comes from a
// cached local series (series_at) whenever the move stays inside the series'
// radius, and from delta_ell otherwise.
//
// LDS ring: the s region rows that the footprints of one block row cover
// (region row y in slot y mod s), two 16-byte records per pixel:
//   st = (mu, D, R, -): the current mean (< 0 outside the frame), its
//   displacement from the series anchor mu - D, and the series radius;
//   b = (b1..b4), the series coefficients at the anchor.
// Moving to the next block row writes the oldest row back to mu and loads the
// next region row with fresh series.  Each thread holds SER_Q footprint
// entries, in descending PSF weight: the first (q = 0) covers the PSF core,
// where relative moves are large and terms leave their radius.
//
// Decisions.  A term outside its radius still has its series' coefficients, and
// they give an interval that holds the direct evaluation (series_bound).  The
// update sums every term's series or interval centre and the half-widths; when
// log u lies farther from Delta than their sum, the direct evaluations could
// not change the decision and none is made.  Otherwise (and when Delta itself is asked for)
// the terms outside are evaluated directly, as a pass without bounds would
// always do, so the chain is the same bit for bit.  What an update waited for
// was one dependent chain of direct evaluations on a few lanes; 2048 x 2048, 4
// chains, Airy 31 x 31: 147.6 to 121.1 ms for two sweeps (17.9 to 14.7 ms per
// launch), direct evaluations 32 to 0.02 per update; 512 x 512, one chain (one
// workgroup per CU, all latency): 46.1 to 35.5 ms for four sweeps.
// An accepted move re-anchors the pixels that left their radius (|D + d| > R:
// the old series is spent).  Those of the PSF core are queued in LDS with their
// record before the decision, and after it consecutive threads of one wave take
// one each, rather than every wave running the whole series for its few lanes;
// the wave that does it differs between neighbouring blocks.
// Counters: [0] phi terms of direct evaluations, [1] footprint evaluations,
// [2] direct evaluations, [3] series anchored (new ring rows, accepted moves
// out of the radius), [4] their phi terms.
// ---------------------------------------------------------------------------
constexpr int SER_Q = 4;                      // footprint entries per thread, at most (F <= SER_Q * WG)
constexpr int SER_JOBS = 48;                  // queued pixels to re-anchor; beyond, the owner lanes

__device__ inline void count_work5(unsigned long long* ctr, int terms, int evals, int direct, int anchors,
                                   int anchor_terms) {
    unsigned long long v[5] = {(unsigned long long)terms, (unsigned long long)evals, (unsigned long long)direct,
                               (unsigned long long)anchors, (unsigned long long)anchor_terms};
#pragma unroll
    for (int k = 0; k < 5; ++k) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < 5; ++k) atomicAdd(&ctr[k], v[k]);
    }
}

__device__ inline double readlane_d(double v, int lane) {
    const int2 u = __builtin_bit_cast(int2, v);
    int2 w;
    w.x = __builtin_amdgcn_readlane(u.x, lane);
    w.y = __builtin_amdgcn_readlane(u.y, lane);
    return __builtin_bit_cast(double, w);
}

// Sum over the 64 lanes, the same value in every lane: pairs, quads, half rows
// and rows by DPP, then rows into the next (row_bcast15, row_bcast31), so that
// lane 63 holds the sum.
template <int CTRL, int ROWS>
__device__ inline double dpp_rows(double v) {
    const int2 u = __builtin_bit_cast(int2, v);
    int2 w;
    w.x = __builtin_amdgcn_update_dpp(0, u.x, CTRL, ROWS, 0xF, false);
    w.y = __builtin_amdgcn_update_dpp(0, u.y, CTRL, ROWS, 0xF, false);
    return __builtin_bit_cast(double, w);
}

__device__ inline double wave_sum_dpp(double v) {
    v += dpp_d<0xB1>(v);      // quad_perm [1,0,3,2]
    v += dpp_d<0x4E>(v);      // quad_perm [2,3,0,1]
    v += dpp_d<0x141>(v);     // row_half_mirror
    v += dpp_d<0x140>(v);     // row_mirror
    v += dpp_rows<0x142, 0xA>(v);
    v += dpp_rows<0x143, 0xC>(v);
    return readlane_d(v, 63);
}

__device__ inline int lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

template <int CTRL, int ROWS>
__device__ inline float dpp_f(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xF, false));
}

__device__ inline float wave_sum_dpp_f(float v) {
    v += dpp_f<0xB1, 0xF>(v);
    v += dpp_f<0x4E, 0xF>(v);
    v += dpp_f<0x141, 0xF>(v);
    v += dpp_f<0x140, 0xF>(v);
    v += dpp_f<0x142, 0xA>(v);
    v += dpp_f<0x143, 0xC>(v);
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// Whether Delta, known to within err (0: exactly), decides against log u: the
// sums of the two evaluations round apart by far less than the 1e-7 kept.
__device__ inline bool decided(double delta, float logu, float err) {
    return err == 0.0f || fabs(delta - (double)logu) > fma(1.02, (double)err, 1e-7);
}

// LDS ring of one block: per region pixel (slot * RW + x), 28 bytes in three
// arrays: A = (D, R, b1, b2), B = (b3, b4), and the series anchor ma; the
// current mean is ma + D.  R < 0 marks pixels outside the frame.
struct Ring {
    float4* A;
    float2* B;
    float* ma;
};

// Load region rows [y0, y0 + n) (block-local, possibly outside the frame) into
// their ring slots with fresh series, spread over the workgroup's NT threads.
template <int NT = WG>
__device__ inline void series_load_rows(const Frame& f, const State& S, int64_t base, int ry0, int rx0, int RW, int y0,
                                        int n, const Ring& ring, int& nterms, int& nanch) {
    for (int i = threadIdx.x; i < n * RW; i += NT) {
        const int y = y0 + i / RW, xx = i - (i / RW) * RW;
        const int gy = ry0 + y, gx = rx0 + xx;
        float4 A = make_float4(0.0f, -1.0f, 0.0f, 0.0f);
        float2 Bv = make_float2(0.0f, 0.0f);
        float mu = -1.0f;
        if (gy >= 0 && gy < f.H && gx >= 0 && gx < f.W) {
            const int64_t pn = (int64_t)gy * f.W + gx;
            mu = S.mu[base + pn];
            const Series sr = series_at(mu, load_pc(f.pc, pn), nterms);
            A = make_float4(0.0f, sr.R, sr.b.x, sr.b.y);
            Bv = make_float2(sr.b.z, sr.b.w);
            ++nanch;
        }
        const int ri = (y % f.s) * RW + xx;
        ring.A[ri] = A;
        ring.B[ri] = Bv;
        ring.ma[ri] = mu;
    }
}

// Write the means of region rows [y0, y0 + n) back to the frame.
template <int NT = WG>
__device__ inline void series_store_rows(const Frame& f, const State& S, int64_t base, int ry0, int rx0, int RW, int y0,
                                         int n, const Ring& ring) {
    for (int i = threadIdx.x; i < n * RW; i += NT) {
        const int y = y0 + i / RW, xx = i - (i / RW) * RW;
        const int gy = ry0 + y, gx = rx0 + xx;
        if (gy >= 0 && gy < f.H && gx >= 0 && gx < f.W) {
            const int ri = (y % f.s) * RW + xx;
            S.mu[base + (int64_t)gy * f.W + gx] = add_rn(ring.ma[ri], ring.A[ri].x);
        }
    }
}

// D + d of a term, d = d0 w: fused for a thread's first entry.
__device__ inline float entry_y(bool first, float D, float d0, float w) {
    return first ? fmaf(w, d0, D) : add_rn(D, mul_rn(d0, w));
}

// Footprint entry e (in descending PSF weight) of the update at block column lx
// of block row ly: offset (oy | ox << 8), ring index and the move's change.
__device__ inline void footprint_entry(const Frame& f, int RW, int ly, int lx, int e, int& o, int& ri, float& w) {
    const int s = f.s, j = f.psf_order[e], oy = j / s, ox = j - oy * s;
    int slot = ly % s + oy;
    slot = slot >= s ? slot - s : slot;
    o = oy | ox << 8;
    ri = slot * RW + ox + lx;
    w = f.psf[j];
}

// This thread's share of Delta with the terms outside their radius evaluated
// directly (rare: everything is read again rather than kept for it).
struct DirectPart { double sum; int terms, n; };

__device__ inline DirectPart block_direct_part(const Frame& f, const Ring& ring, int RW, int ly, int lx,
                                                     int64_t m, float d0) {
    const int F = f.s * f.s, r = f.r;
    DirectPart p = {0.0, 0, 0};
    float fpart = 0.0f;
#pragma unroll 1
    for (int e = threadIdx.x; e < F; e += WG) {
        int o, i;
        float w;
        footprint_entry(f, RW, ly, lx, e, o, i, w);
        const float4 A = ring.A[i];
        if (!(A.y >= 0.0f)) continue;
        const float dj = mul_rn(d0, w), y = entry_y(e < WG, A.x, d0, w);
        if (fabsf(y) <= A.y) {
            const float2 Bv = ring.B[i];
            fpart = fmaf(dj, series_slope(make_float4(A.z, A.w, Bv.x, Bv.y), A.x, y), fpart);
        } else {
            const PixConst pc = load_pc(f.pc, m + (int64_t)((o & 0xFF) - r) * f.W + ((o >> 8) - r));
            const float mu = add_rn(ring.ma[i], A.x);
            // a thread's first by the grouped recurrence, further ones term by term
            p.sum += p.n == 0 ? delta_ell_direct(mu, dj, pc, p.terms) : delta_ell_notab(mu, dj, pc, p.terms);
            ++p.n;
        }
    }
    p.sum += (double)fpart;
    return p;
}

// Slots of the re-anchoring queue: up to SER_JOBS, fewer where the ring leaves
// less room below the LDS size at which one more workgroup fits on a CU (the
// ring of a 31 x 31 PSF at B = 31 leaves 24).
constexpr int SER_JOB_BYTES = sizeof(float4) + sizeof(float2) + sizeof(int);
__host__ __device__ inline size_t block_series_fixed(int B, int s) {
    const int RW = B + 2 * (s / 2);
    return (size_t)2 * WAVES * (sizeof(double) + sizeof(float)) + 4 * sizeof(int) +
           ((size_t)s * RW + 1) * (sizeof(float4) + sizeof(float2) + sizeof(float));
}
__host__ __device__ inline int block_series_jobs(int B, int s) {
    constexpr size_t CU = 160 * 1024, GRAIN = 1280;                // LDS of a CU, its allocation grain
    const size_t fixed = block_series_fixed(B, s);
    const size_t room = CU / (CU / ((fixed + 16 * SER_JOB_BYTES + GRAIN - 1) / GRAIN * GRAIN)) / GRAIN * GRAIN;
    const size_t n = (room - fixed) / SER_JOB_BYTES;
    return n < SER_JOBS ? (int)n : SER_JOBS;
}

template <int NQ>
__device__ void block_series_block(const Frame& f, const State& S, int burn_in, int B,
                                   int py, int px, int bi, int chain, int64_t t, int k0, int k1, float* dbg_delta,
                                   uint8_t* dbg_acc, double* lds_d) {
    const int cap = block_series_jobs(B, f.s);
    const int s = f.s, r = f.r, F = s * s;
    const int RW = B + 2 * r, NR = s * RW;
    double* s_red = lds_d;                                          // [2][WAVES]
    float* s_err = reinterpret_cast<float*>(s_red + 2 * WAVES);     // [2][WAVES]
    int* s_cnt = reinterpret_cast<int*>(s_err + 2 * WAVES);         // [4]: queued pixels, three updates in turn
    float4* job_pc = reinterpret_cast<float4*>(s_cnt + 4);          // [cap] the queue: per-pixel record,
    Ring ring;
    ring.A = job_pc + cap;                                          // [NR + 1]
    ring.B = reinterpret_cast<float2*>(ring.A + NR + 1);            // [NR + 1]
    float2* job_md = ring.B + NR + 1;                               // [cap] (mu, d),
    ring.ma = reinterpret_cast<float*>(job_md + cap);               // [NR + 1]
    int* job_ri = reinterpret_cast<int*>(ring.ma + NR + 1);         // [cap] ring index

    const int nbx = (f.W + B - 1) / B;
    const int nbx_p = (nbx - px + 1) / 2;
    const int by = py + 2 * (bi / nbx_p), bx = px + 2 * (bi % nbx_p);
    const int by0 = by * B, bx0 = bx * B;
    const int bh = min(B, f.H - by0), bw = min(B, f.W - bx0);
    const int64_t base = (int64_t)chain * f.N;
    const int ry0 = by0 - r, rx0 = bx0 - r;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;

    // this thread's footprint entries, the heaviest PSF weights first:
    // offsets (oy, ox) packed as oy | ox << 8, and the weight
    int off[NQ];
    float pw[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int e = threadIdx.x + q * WG;
        const int j = e < F ? (int)f.psf_order[e] : -1;
        off[q] = j >= 0 ? ((j / s) | ((j % s) << 8)) : -1;
        pw[q] = j >= 0 ? f.psf[j] : 0.0f;
    }
    const int oy0 = off[0] & 0xFF, ox0 = (off[0] >> 8) & 0xFF;
    // padding entries (F < NQ * WG) read the sink cell: outside the frame
    if (threadIdx.x == 0) {
        ring.A[NR] = make_float4(0.0f, -1.0f, 0.0f, 0.0f);
        ring.B[NR] = make_float2(0.0f, 0.0f);
        ring.ma[NR] = 0.0f;
    }
    int nterms = 0, nevals = 0, ndirect = 0, nanch = 0, aterms = 0;
    // the colours [k0, k1) visit rows ly of the block, columns [lx_lo, lx_hi)
    auto lx_lo = [&](int y) { return max(0, k0 - y * s); };
    auto lx_hi = [&](int y) { return min(bw, k1 - y * s); };
    int ly = k0 / s, lx = lx_lo(ly);
    while (ly < bh && lx >= lx_hi(ly)) { ++ly; lx = lx_lo(ly); }
    if (ly >= bh) {
        count_work5(S.counters, 0, 0, 0, 0, 0);
        return;
    }
    int ly_cur = ly;
    // ring index of each entry at column 0 of the current block row
    int rb[NQ];
    auto row_bases = [&](int y) {
        const int slot0 = y % s;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int oy = off[q] & 0xFF, ox = (off[q] >> 8) & 0xFF;
            int slot = slot0 + oy;
            slot = slot >= s ? slot - s : slot;
            rb[q] = off[q] >= 0 ? slot * RW + ox : NR;
        }
    };
    row_bases(ly_cur);
    series_load_rows(f, S, base, ry0, rx0, RW, ly_cur, s, ring, aterms, nanch);
    if (threadIdx.x < 4) s_cnt[threadIdx.x] = 0;
    lds_barrier();
    // the wave that re-anchors: another one in the next block of a launch
    const int job0 = ((threadIdx.x + 64 * (bi & (WAVES - 1))) & (WG - 1)) >> 2;
    // inputs of the next update, loaded one update ahead: the decision inputs,
    // and the per-pixel constants of this thread's PSF-core entry (q = 0),
    // where direct evaluations fall
    float4 n_pr;
    float4 n_pc = make_float4(0.0f, 1.0f, 0.0f, 0.0f);
    auto prefetch = [&](int y, int x) {
        const int64_t i = base + (int64_t)(by0 + y) * f.W + (bx0 + x);
        n_pr = S.prop[i];
        const int gy = by0 + y + oy0 - r, gx = bx0 + x + ox0 - r;
        if (off[0] >= 0 && gy >= 0 && gy < f.H && gx >= 0 && gx < f.W) n_pc = f.pc[(int64_t)gy * f.W + gx];
    };
    prefetch(ly, lx);
    const float gain = t < burn_in ? exp2f(-0.6f * log2f((float)t + 1.0f)) : 0.0f;
    // Commits of rho and of the step adaptation are kept per block row: thread
    // x < bw holds pixel (row, x) and writes it back when the row is done, so
    // no global store is outstanding while a wave waits for its next inputs.
    const bool row_owner = threadIdx.x < bw;
    float row_rho = 0.0f, row_ls = 0.0f;
    bool row_acc = false;
    int row_y = -1;
    unsigned long long n_acc = 0;
    auto row_begin = [&](int y) {
        row_y = y;
        row_acc = false;
        if (row_owner && t < burn_in) row_ls = S.log_step[base + (int64_t)(by0 + y) * f.W + (bx0 + threadIdx.x)];
    };
    auto row_end = [&]() {
        if (row_y < 0 || !row_owner) return;
        const int64_t i = base + (int64_t)(by0 + row_y) * f.W + (bx0 + threadIdx.x);
        if (row_acc) S.rho[i] = row_rho;
        if (t < burn_in) S.log_step[i] = row_ls;
    };
    row_begin(ly);
    int par = 0, cq = 0;
    while (ly < bh) {
        const float rp = n_pr.x, hast = n_pr.y, logu = n_pr.z, d0 = n_pr.w;
        const float4 pcv0 = n_pc;
        int nly = ly, nlx = lx + 1;
        while (nly < bh && nlx >= lx_hi(nly)) { ++nly; nlx = lx_lo(nly); }
        if (nly < bh) prefetch(nly, nlx);                           // another pixel: no conflict with this commit
        if (ly != row_y) {
            row_end();
            row_begin(ly);
        }
        if (ly != ly_cur) {
            // rows ly_cur .. ly - 1 retire; their slots take the rows s below
            const int nr = min(ly - ly_cur, s);
            series_store_rows(f, S, base, ry0, rx0, RW, ly_cur, nr, ring);
            lds_barrier();
            series_load_rows(f, S, base, ry0, rx0, RW, ly - nr + s, nr, ring, aterms, nanch);
            ly_cur = ly;
            row_bases(ly);
            lds_barrier();
        }
        const int64_t m = (int64_t)(by0 + ly) * f.W + (bx0 + lx);
        // 1. every entry's records, loads issued together
        int ri[NQ];
        float4 Aq[NQ];
        float2 Bq[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            ri[q] = off[q] >= 0 ? rb[q] + lx : NR;
            Aq[q] = ring.A[ri[q]];
            Bq[q] = ring.B[ri[q]];
        }
        const float ma0 = ring.ma[ri[0]];                           // the PSF-core entry may leave its radius
        // 2. every term's series or, outside its radius, its bound.  (A lane's
        // few terms in FP32: their rounding stays relative to the sum of the
        // terms' magnitudes.)  A pixel that an accepted move takes out of its
        // radius is queued: for the PSF core with the record fetched an update
        // ahead, else with its pixel (marked by a negative 2a).
        bool fast[NQ], any = false;
        unsigned left = 0;                                          // entries beyond the queue; bit 8: the first is one
        float y[NQ], fpart = 0.0f, gpart = 0.0f, err = 0.0f;
        // slot i of the queue's round: (mu, d) for a lane's first such pixel,
        // re-anchored over the window of its move, (mu + d, 0) for further ones,
        // over that of the new mean
        auto queue = [&](int q, int i, float mu, float dq, bool first) {
            const int pix = (int)m + ((off[q] & 0xFF) - r) * f.W + ((off[q] >> 8) - r);
            job_pc[i] = make_float4(__int_as_float(pix), -2.0f, 0.0f, 0.0f);
            job_md[i] = first ? make_float2(mu, dq) : make_float2(add_rn(mu, dq), 0.0f);
            job_ri[i] = ri[q];
        };
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const float dq = mul_rn(d0, pw[q]);
            y[q] = entry_y(q == 0, Aq[q].x, d0, pw[q]);
            const bool valid = Aq[q].y >= 0.0f;
            fast[q] = fabsf(y[q]) <= Aq[q].y;
            const float4 b = make_float4(Aq[q].z, Aq[q].w, Bq[q].x, Bq[q].y);
            nevals += valid ? 1 : 0;
            const float slope = series_slope(b, Aq[q].x, y[q]);
            if (fast[q]) fpart = fmaf(dq, slope, fpart);
            const bool need = valid && !fast[q];
            const uint64_t bal = __ballot(need);
            if (bal) {
                int first = 0;
                if (lane == 0) first = atomicAdd(&s_cnt[cq], __popcll(bal));
                const float ma = q == 0 ? ma0 : ring.ma[ri[q]];
                if (need) {
                    const TermBound tb = series_bound(ma, b, Aq[q].x, y[q], dq * slope);
                    gpart += tb.c;
                    err += tb.e;
                }
                first = __builtin_amdgcn_readfirstlane(first) + lanes_below(bal);
                if (need) {
                    if (first < cap) {
                        queue(q, first, add_rn(ma, Aq[q].x), dq, !any);
                        if (q == 0) job_pc[first] = pcv0;
                    } else left |= any ? 1u << q : 0x100u | 1u << q;
                    any = true;
                }
            }
        }
        const int cq1 = cq == 2 ? 0 : cq + 1;
        if (threadIdx.x == 0) s_cnt[cq1] = 0;                       // read last before the previous update's barrier
        double part = wave_sum_dpp((double)fpart + (double)gpart);
        if (__any(err != 0.0f)) err = wave_sum_dpp_f(err);
        if (lane == 0) {
            s_red[par * WAVES + wave] = part;
            s_err[par * WAVES + wave] = err;
        }
        lds_barrier();
        double tot = 0.0;
        float etot = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            tot += s_red[par * WAVES + w];
            etot += s_err[par * WAVES + w];
        }
        par ^= 1;
        // 4. too close to call (or Delta asked for): the direct evaluations
        if (!decided(tot + (double)hast, logu, etot) || (dbg_delta && etot != 0.0f)) {
            const DirectPart dp = block_direct_part(f, ring, RW, ly, lx, m, d0);
            nterms += dp.terms;
            ndirect += dp.n;
            part = wave_sum_dpp(dp.sum);
            if (lane == 0) s_red[par * WAVES + wave] = part;
            lds_barrier();
            tot = 0.0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) tot += s_red[par * WAVES + w];
            par ^= 1;
        }
        // the decision (identical in every thread)
        const double delta = tot + (double)hast;
        const bool acc = isfinite(delta) && ((double)logu < delta);
        if (threadIdx.x == lx) {
            if (acc) {
                row_rho = rp;
                row_acc = true;
            }
            row_ls = fmaf(gain, (acc ? 1.0f : 0.0f) - 0.44f, row_ls);
        }
        n_acc += acc ? 1 : 0;
        if (threadIdx.x == 0) {
            if (dbg_delta) dbg_delta[base + m] = (float)delta;
            if (dbg_acc) dbg_acc[base + m] = acc ? 1 : 0;
        }
        if (acc) {
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (fast[q]) ring.A[ri[q]].x = y[q];
            // pixels that left their series' radius: re-anchor at the new mean
            auto anchor = [&](int i, const Series& nx, float mu1) {
                ring.A[i] = make_float4(0.0f, nx.R, nx.b.x, nx.b.y);
                ring.B[i] = make_float2(nx.b.z, nx.b.w);
                ring.ma[i] = mu1;
                ++nanch;
            };
            // (more than the queue holds, on bright frames: in rounds)
            for (int n = s_cnt[cq], n0 = 0;;) {
                if (job0 < min(n - n0, cap)) {
                    const float2 md = job_md[job0];
                    float4 rec = job_pc[job0];
                    if (rec.y == -2.0f) rec = f.pc[__float_as_int(rec.x)];
                    const Series nx = series_after(md.x, md.y, pc_of(rec), threadIdx.x & 3, aterms);
                    if ((threadIdx.x & 3) == 0) anchor(job_ri[job0], nx, add_rn(md.x, md.y));
                }
                n0 += cap;
                if (n <= n0) break;
                if (threadIdx.x == 0) s_cnt[3] = 0;
                lds_barrier();
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const uint64_t bal = __ballot((left >> q) & 1);
                    if (!bal) continue;
                    int i = 0;
                    if (lane == 0) i = atomicAdd(&s_cnt[3], __popcll(bal));
                    i = __builtin_amdgcn_readfirstlane(i) + lanes_below(bal);
                    if (((left >> q) & 1) && i < cap) {
                        queue(q, i, add_rn(ring.ma[ri[q]], ring.A[ri[q]].x), mul_rn(d0, pw[q]), left & 0x100);
                        left &= ~(0x100u | 1u << q);
                    }
                }
                lds_barrier();
            }
            lds_barrier();                                          // commits before the next footprint reads
        }
        cq = cq1;
        ly = nly;
        lx = nlx;
    }
    row_end();
    if (threadIdx.x == 0) atomicAdd(&S.accepts[chain], n_acc);
    series_store_rows(f, S, base, ry0, rx0, RW, ly_cur, s, ring);
    count_work5(S.counters, nterms, nevals, ndirect, nanch, aterms);
}

template <int NQ>
__global__ void __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(3))) k_block_series(Frame f, State S, int burn_in, int B,
                                                     int py, int px, int k0, int k1, float* dbg_delta,
                                                     uint8_t* dbg_acc, int nblk) {
    extern __shared__ double lds_d[];
    int bi, chain;
    if (!xcd_block(nblk, f.C, bi, chain)) return;
    block_series_block<NQ>(f, S, burn_in, B, py, px, bi, chain, *S.t, k0, k1, dbg_delta, dbg_acc, lds_d);
}

// ---------------------------------------------------------------------------
// Block-series pass of the nine-phase scan: one wavefront per block.
//
// Blocks of side B in [(s - 1)/2, s] keep the ring of s region rows at
// s (B + s - 1) pixels, small enough for four workgroups per CU, and one
// wavefront holds a whole footprint (up to 16 entries per lane, entry
// e = lane + 64 q in descending PSF weight), so an update needs no workgroup
// barrier: a wave-wide reduction and in-order LDS suffice.  The footprint
// terms that leave their series' radius (a few dozen per update, spread over
// the PSF's heaviest few hundred entries) are queued in LDS and evaluated in
// one pass, one per lane, whatever lanes own them; the owner, which fetched
// every entry's (c, 2a) one update ahead, queues them with the term, and the
// evaluating lane derives the window constants L0 and iB from them (the
// window bracket holds for whatever (c, a) the summands use).  Terms,
// decisions (by bounds) and commits are those of the block-series pass; here the
// queue holds every term outside its radius, the bounds are taken one per lane
// from it, and four lanes re-anchor each pixel of an accepted move.  701 x 1003,
// Gaussian 15 x 15, 2 chains: 27.9 to 22.0 ms for six sweeps.
// ---------------------------------------------------------------------------
constexpr int WS_NQ = 16;                       // footprint entries per lane (F <= 1024)
// queued terms per update (beyond, the owner lanes): one per lane for the ring of
// a 31 x 31 PSF, which fills a quarter of a CU's LDS; two for the smaller ones
constexpr int ws_cap(int nq) { return nq > 8 ? 64 : 128; }
constexpr int WS_MOVE = 48;                     // these re-anchor over the window of their move, further ones
                                                // over that of the new mean

__device__ inline PixConst pc_from(float c, float a2) {
    PixConst pc;
    pc.c = c;
    pc.a2 = a2;
    pc.ks = fmaxf(c, 0.0f);
    const float ik = __builtin_amdgcn_rcpf(pc.ks + 1.0f);
    pc.L0 = a2 * (c - pc.ks) - fast_ln(pc.ks + 1.0f);
    pc.iB = __builtin_amdgcn_rcpf(a2 + ik);
    pc.inv2a = __builtin_amdgcn_rcpf(a2);
    pc.h0 = __builtin_amdgcn_sqrtf(2.0f * TAIL_T * pc.inv2a);
    return pc;
}

template <int NQ>
__device__ void wave_series_block(const Frame& f, const State& S, int burn_in, int B, int py, int px, int bi,
                                  int chain, int64_t t, int k0, int k1, float* dbg_delta, uint8_t* dbg_acc,
                                  double* lds_d) {
    constexpr int QCAP = ws_cap(NQ);
    const int s = f.s, r = f.r, F = s * s;
    const int RW = B + 2 * r, NR = s * RW;
    // queue slot QCAP and ring cell NR are write sinks: lanes with nothing
    // to queue or commit write there, so the per-entry steps need no branches
    float4* jobs = reinterpret_cast<float4*>(lds_d);                // [QCAP + 1]: (mu, d, c, 2a)
    int* job_ri = reinterpret_cast<int*>(jobs + QCAP + 1);       // [QCAP + 1]: ring index
    Ring ring;
    ring.A = reinterpret_cast<float4*>(job_ri + QCAP + 4);       // [NR + 1], 16-byte aligned
    ring.B = reinterpret_cast<float2*>(ring.A + NR + 1);            // [NR + 1]
    ring.ma = reinterpret_cast<float*>(ring.B + NR + 1);            // [NR + 1]

    const int nbx = (f.W + B - 1) / B;
    const int nbx_p = (nbx - px + 2) / 3;
    const int by = py + 3 * (bi / nbx_p), bx = px + 3 * (bi % nbx_p);
    const int by0 = by * B, bx0 = bx * B;
    const int bh = min(B, f.H - by0), bw = min(B, f.W - bx0);
    const int64_t base = (int64_t)chain * f.N;
    const int ry0 = by0 - r, rx0 = bx0 - r;
    const int lane = threadIdx.x;
    if (lane == 0) {
        ring.A[NR] = make_float4(0.0f, -1.0f, 0.0f, 0.0f);          // never inside a radius
        ring.B[NR] = make_float2(0.0f, 0.0f);
        ring.ma[NR] = 0.0f;
    }

    int off[NQ];
    float pw[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int e = lane + 64 * q;
        const int j = e < F ? (int)f.psf_order[e] : -1;
        off[q] = j >= 0 ? ((j / s) | ((j % s) << 8)) : -1;
        pw[q] = j >= 0 ? f.psf[j] : 0.0f;
    }
    int nterms = 0, nevals = 0, ndirect = 0, nanch = 0, aterms = 0;
    auto lx_lo = [&](int y) { return max(0, k0 - y * s); };
    auto lx_hi = [&](int y) { return min(bw, k1 - y * s); };
    int ly = k0 / s, lx = lx_lo(ly);
    while (ly < bh && lx >= lx_hi(ly)) { ++ly; lx = lx_lo(ly); }
    if (ly >= bh) {
        count_work5(S.counters, 0, 0, 0, 0, 0);
        return;
    }
    int ly_cur = ly;
    // ring index of each entry at column 0 of the current block row (padding
    // entries: the sink cell, whatever the column)
    int rb[NQ];
    auto row_bases = [&](int y) {
        const int slot0 = y % s;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int oy = off[q] & 0xFF, ox = (off[q] >> 8) & 0xFF;
            int slot = slot0 + oy;
            slot = slot >= s ? slot - s : slot;
            rb[q] = off[q] >= 0 ? slot * RW + ox : NR;
        }
    };
    auto ring_index = [&](int q) { return off[q] >= 0 ? rb[q] + lx : NR; };
    row_bases(ly_cur);
    series_load_rows<64>(f, S, base, ry0, rx0, RW, ly_cur, s, ring, aterms, nanch);
    wave_fence();
    // inputs of the next update, fetched one update ahead: the decision inputs
    // and every entry's (c, 2a), through a buffer resource whose range check
    // turns the reads of entries outside the frame into zeros (such entries
    // have invalid ring records and are never queued)
    float4 n_pr;
    float2 pcq[NQ];
    const __amdgpu_buffer_rsrc_t pc_rsrc =
        __builtin_amdgcn_make_buffer_rsrc((void*)f.pc, 0, (int)(f.N * (int64_t)sizeof(float4)), 0x00020000);
    const int row_stride = f.W - s;                                 // so that (oy, ox) -> oy W + ox - r (W + 1)
    (void)row_stride;
    auto prefetch = [&](int y, int x) {
        const int64_t m = (int64_t)(by0 + y) * f.W + (bx0 + x);
        n_pr = S.prop[base + m];
        const int m0 = (int)m - r * (f.W + 1);                      // the footprint's top-left pixel
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int oy = off[q] & 0xFF, ox = (off[q] >> 8) & 0xFF;
            const unsigned byte_off = (unsigned)(m0 + oy * f.W + ox) * (unsigned)sizeof(float4);
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(pc_rsrc, byte_off, 0, 0);
            pcq[q] = __builtin_bit_cast(float2, v);
        }
    };
    prefetch(ly, lx);
    const float gain = t < burn_in ? exp2f(-0.6f * log2f((float)t + 1.0f)) : 0.0f;
    const bool row_owner = lane < bw;
    float row_rho = 0.0f, row_ls = 0.0f;
    bool row_acc = false;
    int row_y = -1;
    unsigned long long n_acc = 0;
    auto row_begin = [&](int y) {
        row_y = y;
        row_acc = false;
        if (row_owner && t < burn_in) row_ls = S.log_step[base + (int64_t)(by0 + y) * f.W + (bx0 + lane)];
    };
    auto row_end = [&]() {
        if (row_y < 0 || !row_owner) return;
        const int64_t i = base + (int64_t)(by0 + row_y) * f.W + (bx0 + lane);
        if (row_acc) S.rho[i] = row_rho;
        if (t < burn_in) S.log_step[i] = row_ls;
    };
    row_begin(ly);
    while (ly < bh) {
        const float rp = n_pr.x, hast = n_pr.y, logu = n_pr.z, d0 = n_pr.w;
        int nly = ly, nlx = lx + 1;
        while (nly < bh && nlx >= lx_hi(nly)) { ++nly; nlx = lx_lo(nly); }
        if (ly != row_y) {
            row_end();
            row_begin(ly);
        }
        if (ly != ly_cur) {
            const int nr = min(ly - ly_cur, s);
            series_store_rows<64>(f, S, base, ry0, rx0, RW, ly_cur, nr, ring);
            wave_fence();
            series_load_rows<64>(f, S, base, ry0, rx0, RW, ly - nr + s, nr, ring, aterms, nanch);
            ly_cur = ly;
            row_bases(ly);
            wave_fence();
        }
        const int64_t m = (int64_t)(by0 + ly) * f.W + (bx0 + lx);
        // 1. every entry's record (four entries' loads issued together); its
        //    series term, or its place in the queue of terms outside their
        //    radius, with the (c, 2a) fetched for it
        unsigned fast = 0, over = 0;
        int nq = 0;
        float fpart = 0.0f;
        float Dq[NQ];
#pragma unroll
        for (int g = 0; g < NQ; g += 4) {
            float4 Aq[4];
            float2 Bq[4];
            float maq[4];
#pragma unroll
            for (int u = 0; u < 4 && g + u < NQ; ++u) {
                const int ri = ring_index(g + u);
                Aq[u] = ring.A[ri];
                Bq[u] = ring.B[ri];
                maq[u] = ring.ma[ri];
            }
#pragma unroll
            for (int u = 0; u < 4 && g + u < NQ; ++u) {
                const int q = g + u;
                const float dq = mul_rn(d0, pw[q]), y = fmaf(pw[q], d0, Aq[u].x);
                Dq[q] = Aq[u].x;
                const bool valid = Aq[u].y >= 0.0f;                 // inside the frame (sink: R < 0)
                const bool in_r = fabsf(y) <= Aq[u].y;
                const float sd = mul_rn(dq, series_slope(make_float4(Aq[u].z, Aq[u].w, Bq[u].x, Bq[u].y), Aq[u].x, y));
                fpart = add_rn(fpart, in_r ? sd : 0.0f);
                fast |= in_r ? 1u << q : 0u;
                const bool dir = valid && !in_r;
                nevals += valid ? 1 : 0;
                const uint64_t bal = __ballot(dir);
                if (bal) {
                    const int slot = nq + lanes_below(bal);
                    const bool queued = dir && slot < QCAP;
                    over |= (dir && !queued) ? 1u << q : 0u;
                    const int ws = queued ? slot : QCAP;
                    jobs[ws] = make_float4(add_rn(maq[u], Aq[u].x), dq, pcq[q].x, pcq[q].y);
                    job_ri[ws] = ring_index(q);
                    nq += __popcll(bal);
                }
            }
        }
        // the commit reads the masks from these lane words (keeps the
        // compiler from holding one lane mask per entry in scalar registers)
        asm volatile("" : "+v"(fast), "+v"(over));
        // the next update's inputs (another pixel: its proposal does not
        // depend on this commit; the footprint records are per frame)
        if (nly < bh) prefetch(nly, nlx);
        wave_fence();
        // terms beyond the queue (rare): their owners, one entry at a time,
        // each rebuilt from the PSF order and the ring
        auto over_entry = [&](int q, int& ri, float& dq, int64_t& pix) {
            const int j = f.psf_order[lane + 64 * q];
            const int oy = j / s, ox = j - oy * s;
            int slot = ly % s + oy;
            slot = slot >= s ? slot - s : slot;
            ri = slot * RW + ox + lx;
            dq = mul_rn(d0, f.psf[j]);
            pix = m + (int64_t)(oy - r) * f.W + (ox - r);
        };
        // 2. Delta from every term's series; too close to call within the bounds
        // of those outside their radius (or Delta asked for): the queued terms
        // evaluated directly, one per lane, then those beyond the queue
        double part = (double)fpart;
        float err = 0.0f;
        if (nq > 0) {
#pragma unroll 1
            for (int j = lane; j < min(nq, QCAP); j += 64) {
                const float4 jb = jobs[j];
                const int i = job_ri[j];
                const float4 A = ring.A[i];
                const float2 Bv = ring.B[i];
                const float4 b = make_float4(A.z, A.w, Bv.x, Bv.y);
                const TermBound tb = series_bound(ring.ma[i], b, A.x, A.x + jb.y, series_delta(b, A.x, jb.y));
                part += (double)tb.c;
                err += tb.e;
            }
            if (nq > QCAP) err = INFINITY;
            err = wave_sum_dpp_f(err);
        }
        part = wave_sum_dpp(part);
        if (nq > 0) {
            if (!decided(part + (double)hast, logu, err) || dbg_delta) {
                part = (double)fpart;
#pragma unroll 1
                for (int j = lane; j < min(nq, QCAP); j += 64) {
                    const float4 jb = jobs[j];
                    const DirectValue dv = direct_value(jb.x, jb.y, pc_from(jb.z, jb.w));
                    part += dv.v;
                    nterms += dv.terms;
                    ++ndirect;
                }
                if (nq > QCAP) {
#pragma unroll 1
                    for (int q = 0; q < NQ; ++q) {
                        if ((over >> q) & 1) {
                            int ri;
                            float dq;
                            int64_t pix;
                            over_entry(q, ri, dq, pix);
                            const DirectValue dv = notab_value(ring.ma[ri] + ring.A[ri].x, dq, load_pc(f.pc, pix));
                            part += dv.v;
                            nterms += dv.terms;
                            ++ndirect;
                        }
                    }
                }
                part = wave_sum_dpp(part);
            }
        }
        // the decision (identical in every lane)
        const double delta = part + (double)hast;
        const bool acc = isfinite(delta) && ((double)logu < delta);
        if (lane == lx) {
            row_rho = acc ? rp : row_rho;
            row_acc = row_acc || acc;
            row_ls = fmaf(gain, (acc ? 1.0f : 0.0f) - 0.44f, row_ls);
        }
        n_acc += acc ? 1 : 0;
        if (lane == 0) {
            if (dbg_delta) dbg_delta[base + m] = (float)delta;
            if (dbg_acc) dbg_acc[base + m] = acc ? 1 : 0;
        }
        if (acc) {
            // series entries move their displacement; the others write theirs
            // back unchanged (queued ones are re-anchored just after, in order)
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                ring.A[ring_index(q)].x = ((fast >> q) & 1) ? fmaf(pw[q], d0, Dq[q]) : Dq[q];
            // queued terms left their series' radius: re-anchor at the new mean
#pragma unroll 1
            for (int j = lane >> 2; j < min(nq, QCAP); j += 16) {
                const float4 jb = jobs[j];
                const bool move = j < WS_MOVE;
                const Series nx = series_after(move ? jb.x : add_rn(jb.x, jb.y), move ? jb.y : 0.0f, pc_from(jb.z, jb.w),
                                               lane & 3, aterms);
                if ((lane & 3) == 0) {
                    const int i = job_ri[j];
                    ring.A[i] = make_float4(0.0f, nx.R, nx.b.x, nx.b.y);
                    ring.B[i] = make_float2(nx.b.z, nx.b.w);
                    ring.ma[i] = add_rn(jb.x, jb.y);
                    ++nanch;
                }
            }
            if (nq > QCAP) {
#pragma unroll 1
                for (int q = 0; q < NQ; ++q) {
                    if ((over >> q) & 1) {
                        int ri;
                        float dq;
                        int64_t pix;
                        over_entry(q, ri, dq, pix);
                        if (dq != 0.0f) {
                            const float mu1 = add_rn(add_rn(ring.ma[ri], ring.A[ri].x), dq);
                            const Series sr = series_at(mu1, load_pc(f.pc, pix), aterms);
                            ring.A[ri] = make_float4(0.0f, sr.R, sr.b.x, sr.b.y);
                            ring.B[ri] = make_float2(sr.b.z, sr.b.w);
                            ring.ma[ri] = mu1;
                            ++nanch;
                        }
                    }
                }
            }
        }
        wave_fence();                                               // commits before the next footprint reads
        ly = nly;
        lx = nlx;
    }
    row_end();
    if (lane == 0) atomicAdd(&S.accepts[chain], n_acc);
    series_store_rows<64>(f, S, base, ry0, rx0, RW, ly_cur, s, ring);
    count_work5(S.counters, nterms, nevals, ndirect, nanch, aterms);
}

// (waves per SIMD: what the registers of the instantiations leave; four entries sit at the edge of three)
constexpr int wave_occupancy(int nq) { return nq <= 4 ? 3 : nq <= 7 ? 2 : 1; }

template <int NQ>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(wave_occupancy(NQ)))) k_wave_series(Frame f, State S, int burn_in, int B, int py, int px, int k0,
                                                    int k1, float* dbg_delta, uint8_t* dbg_acc, int nblk) {
    extern __shared__ double lds_d[];
    int bi, chain;
    if (!xcd_block(nblk, f.C, bi, chain)) return;
    wave_series_block<NQ>(f, S, burn_in, B, py, px, bi, chain, *S.t, k0, k1, dbg_delta, dbg_acc, lds_d);
}

// ---------------------------------------------------------------------------
// Block-phase pass decided by bounds: the direct scan of the EMCCD reading, of
// the chunk prior and of a finer object lattice, for blocks with one active
// cell per colour (B <= s).  LDS holds, beside the region's means, a local
// series of every region pixel, which serves to bound Delta only: when log u
// lies outside the bound the decision is known; else (and when Delta itself is
// asked for) every footprint term is evaluated directly, as in k_block_phase.
// Means, states and decisions are those of the all-direct pass.
//
// The series need not give a value, so its anchor may stay behind, up to BND_R
// radii and half the mean away; the truncation there, for each of a term's two
// points at most (p_4 / 5) |v|^5 / (1 - |v|) (p_4, v as at series_bound; |v| <= 1/2),
// is charged term by term.  Beyond, series_bound gives the term's interval, and
// an accepted move re-anchors the pixel.
//
// EMCCD pixels: the reading's factor is A + B f(mu), f = sqrt(mu / c) I_1(2
// sqrt(mu c)), whose zeros in mu are real and not positive, so that log f is a
// sum of log(1 + beta v) and has the bounds of the sCMOS log-likelihood.  With
// w = B f / (A + B f) at the anchor and g the change of log f from there, that
// of log(A + B f) is log(1 + w (e^g - 1)), whose slope in g lies in [0, 1]
// (bdc_bounds.h).
//
// Chunk prior: F_-k = conj F_k for a real object, so a thread holds one frequency
// of each such pair, its sums in FP32 with their rounding in the bound; the
// modulus sum's FP64 change is formed when a move is accepted.
//
// What bounds it: the chain of one block's updates (reduce, decide, commit), one
// workgroup per CU where the region takes the LDS (28 bytes a pixel: 104 KB at
// 31 x 31), so a workgroup has eight wavefronts there, and an update touches no
// global memory: a row's proposals are loaded a row ahead, one per lane, and its
// outcomes stored at its end.  Measured, two sweeps of two chains against the
// all-direct pass: EMCCD 384 x 500, PSF 21 x 21: 54.5 -> 5.0 ms (1.4 us per update
// of a block; four wavefronts of two terms a lane: 5.8 ms); chunk prior 512^2, 31 x 31:
// 68.5 -> 12.9 ms; 512^2 at k = 2, PSF 63 x 63: 285 -> 58 ms.
// ---------------------------------------------------------------------------
constexpr float BND_FLAT = 1e-7f;             // of a term: the direct evaluation's absolute rounding
constexpr size_t BND_LDS_MAX = 160 * 1024;
constexpr int BND_MAX_F = 3 * 512;            // footprint entries (three per thread of eight waves)

struct BoundedLds {
    double *red, *red2;                          // [waves]: direct sums; the prior's exact S' - S
    float4* bnd;                                 // [2][waves]: centre, half-width, S' - S
    int* cnt;                                    // [4]: queued pixels of three updates in turn
    float4* A;                                   // [RW * RW + 1]: anchor mean, reach of its series, b1, b2
    float2* B;                                   // b3, b4
    float* mu;                                   // current mean, -1 outside the frame
    float* w;                                    // EMCCD: share of B f, or log(B f / A)
    uint16_t* job;                               // [F]: queued pixels, region index
    float* job_mu;                               // [F]: their means after the move
    double2 *th, *tw;                            // chunk prior: (cos, sin)(2 pi j / n), j < th, j < tw
};

__host__ __device__ inline size_t bounded_layout(int B, int s, bool em, bool dir, char* base, BoundedLds* out) {
    const int RW = B + 2 * (s / 2), NR = RW * RW + 1, F = s * s, NW = 8;
    size_t at = 0;
    BoundedLds l;
    auto take = [&](size_t n) {
        char* p = base + at;
        at += (n + 15) / 16 * 16;
        return p;
    };
    l.red = (double*)take(NW * sizeof(double));
    l.red2 = (double*)take(NW * sizeof(double));
    l.bnd = (float4*)take(2 * NW * sizeof(float4));
    l.cnt = (int*)take(4 * sizeof(int));
    l.A = (float4*)take(NR * sizeof(float4));
    l.B = (float2*)take(NR * sizeof(float2));
    l.mu = (float*)take(NR * sizeof(float));
    l.w = (float*)take(em ? NR * sizeof(float) : 0);
    l.job = (uint16_t*)take(F * sizeof(uint16_t));
    l.job_mu = (float*)take(F * sizeof(float));
    l.th = (double2*)take(dir ? B * sizeof(double2) : 0);
    l.tw = (double2*)take(dir ? B * sizeof(double2) : 0);
    if (out) *out = l;
    return at;
}

// A thread's frequency of the chunk prior (and its conjugate's, weight n = 2).
struct DirFreq {
    double re, im;                               // spectrum
    float amA, amB;                              // alpha - 1 of the two (amB = 0 where they are one)
    float n;                                     // 0: no frequency
    int jy, jx;
};

// Exact change of the log prior under d at the cell of row ly, column lx, but
// for the modulus sum's logarithm: terms tsum, S' - S dsum; w the twiddle.
struct DirDelta { double tsum, dsum, wr, wi; };

__device__ inline DirDelta dir_delta(const DirFreq& z, double2 cy, double2 cx, float d0) {
    DirDelta o;
    const double wr = cy.x * cx.x - cy.y * cx.y, wi = -(cy.y * cx.x + cy.x * cx.y);
    const double re = z.re, im = z.im, dd = (double)d0;
    const double n2 = re * re + im * im;
    const double re1 = fma(dd, wr, re), im1 = fma(dd, wi, im);
    const double n21 = re1 * re1 + im1 * im1;
    // |F'|^2 - |F|^2 without cancellation for small moves; the ratio itself when
    // the component shrinks a lot
    const double num = dd * (2.0 * (re * wr + im * wi) + dd);
    const float lr = num > -0.5 * n2 ? log1p_k((float)(num / n2)) : fast_ln((float)(n21 / n2));
    o.tsum = (double)(z.amA * 0.5f * lr) + (double)(z.amB * 0.5f * lr);
    o.dsum = (double)z.n * (num / (double)(__builtin_amdgcn_sqrtf((float)n21) + __builtin_amdgcn_sqrtf((float)n2)));
    o.wr = wr;
    o.wi = wi;
    return o;
}

// One block (index bi among the blocks of phase (py, px)) of one chain: NT
// threads, NQ footprint entries each (NT NQ >= F).
template <bool EM, bool DIR, bool SUB, int NT, int NQ>
__device__ void bounded_block(const Frame& f, const State& S, int burn_in, const double* inv_tab, int B, int py,
                              int px, int bi, int chain, int64_t t, int k0, int k1, float* dbg_delta,
                              uint8_t* dbg_acc, char* lds) {
    constexpr int NW = NT / 64;
    const int s = f.s, r = f.r, F = s * s, k = SUB ? f.sub : 1;
    const int RW = B + 2 * r, NR = RW * RW;
    BoundedLds l;
    bounded_layout(B, s, EM, DIR, lds, &l);
    const int nbx = (f.Wp + B - 1) / B;
    const int nbx_p = (nbx - px + 1) / 2;
    const int by = py + 2 * (bi / nbx_p), bx = px + 2 * (bi % nbx_p);
    const int by0 = by * B, bx0 = bx * B;
    const int bh = min(B, f.Hp - by0), bw = min(B, f.Wp - bx0);
    const int64_t base = (int64_t)chain * f.N, pbase = (int64_t)chain * f.Np;
    const int ry0 = by0 - r, rx0 = bx0 - r;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63);
    const bool want_delta = dbg_delta || dbg_acc;
    int nterms = 0, nevals = 0, ndirect = 0, nanch = 0, aterms = 0;

    // this thread's footprint entries: region offset (padding: none), weight
    int off[NQ];
    float pw[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int e = threadIdx.x + q * NT;
        off[q] = e < F ? (e / s) * RW + e % s : -1;
        pw[q] = e < F && !SUB ? f.psf[e] : 0.0f;
    }
    auto region_pc = [&](int i) {
        const int y = i / RW;
        return load_pc(f.pc, (int64_t)(ry0 + y) * f.Wp + (rx0 + i - y * RW));
    };
    auto set_series = [&](int i, float m, const Series& sr) {
        // (counts so large that the direct window may be refused: left to series_bound)
        const float reach = m * (fabsf(sr.b.x) + 1.0f) < 1e5f ? fminf(BND_R * sr.R, 0.5f * m) : 0.0f;
        l.A[i] = make_float4(m, reach, sr.b.x, sr.b.y);
        l.B[i] = make_float2(sr.b.z, sr.b.w);
        ++nanch;
    };
    auto anchor_em = [&](int i, float m) {
        const PixConst pc = region_pc(i);
        const EmSeries es = emccd_series(m, pc.c, pc.L0, pc.iB);
        set_series(i, m, es.s);
        l.w[i] = es.w;
    };
    for (int i = threadIdx.x; i <= NR; i += NT) {
        const int y = i / RW, yy = ry0 + y, xx = rx0 + i - y * RW;
        float mu = -1.0f;
        l.A[i] = make_float4(0.0f, -1.0f, 0.0f, 0.0f);
        l.B[i] = make_float2(0.0f, 0.0f);
        if (EM) l.w[i] = INFINITY;
        if (i < NR && yy >= 0 && yy < f.Hp && xx >= 0 && xx < f.Wp) {
            mu = S.mu[pbase + (int64_t)yy * f.Wp + xx];
            if (!want_delta) {
                if constexpr (EM) anchor_em(i, mu);
                else set_series(i, mu, series_at(mu, region_pc(i), aterms));
            }
        }
        l.mu[i] = mu;
    }
    if (threadIdx.x < 4) l.cnt[threadIdx.x] = 0;
    // chunk prior: the block's spectrum (computed from rho before the pass), one
    // frequency of each conjugate pair per thread (rows 0 .. th / 2, of rows 0 and
    // th / 2 the columns 0 .. tw / 2), the modulus sum S, twiddles
    double dS_tot = 0.0;
    const int dK = bh * bw;
    const float inv_bh = 1.0f / (float)bh, inv_bw = 1.0f / (float)bw;
    DirFreq fr = {1.0, 0.0, 0.0f, 0.0f, 0.0f, 0, 0};
    float fre = 1.0f, fim = 0.0f, fabs_F = 1.0f, finv = 1.0f;        // FP32: spectrum, modulus, 1 / modulus
    auto dir_round = [&]() {
        fre = (float)fr.re;
        fim = (float)fr.im;
        const float n2 = (float)(fr.re * fr.re + fr.im * fr.im);
        fabs_F = __builtin_amdgcn_sqrtf(n2);
        finv = fast_rcp(fabs_F);
    };
    if (DIR) {
        const int shape = (bh < B ? 2 : 0) + (bw < B ? 1 : 0);
        const float* am = f.dir_am1 + (size_t)shape * B * B;
        const int half = bw / 2 + 1, e = threadIdx.x, mid = half + (bh - 1) / 2 * bw;
        const int jy = e < half ? 0 : e < mid ? 1 + (e - half) / bw : bh / 2;
        const int jx = e < half ? e : e < mid ? (e - half) % bw : e - mid;
        if (e < mid || ((bh & 1) == 0 && e < mid + half)) {
            const int cy = jy ? bh - jy : 0, cx = jx ? bw - jx : 0;  // the conjugate's
            const bool self = cy == jy && cx == jx;
            const double2 Fk = f.dir_F[base + (int64_t)(by0 + jy) * f.W + (bx0 + jx)];
            fr = {Fk.x, Fk.y, am[jy * bw + jx], self ? 0.0f : am[cy * bw + cx], self ? 1.0f : 2.0f, jy, jx};
            dS_tot = (double)fr.n * sqrt(Fk.x * Fk.x + Fk.y * Fk.y);
            dir_round();
        }
        for (int j = threadIdx.x; j < bh; j += NT) {
            double sn, cs;
            sincospi(2.0 * j / bh, &sn, &cs);
            l.th[j] = make_double2(cs, sn);
        }
        for (int j = threadIdx.x; j < bw; j += NT) {
            double sn, cs;
            sincospi(2.0 * j / bw, &sn, &cs);
            l.tw[j] = make_double2(cs, sn);
        }
        dS_tot = wave_sum(dS_tot);
        if (lane == 0) l.red2[wave] = dS_tot;
        __syncthreads();
        dS_tot = 0.0;
        for (int w = 0; w < NW; ++w) dS_tot += l.red2[w];
    }
    __syncthreads();

    const float gain = t < burn_in ? exp2f(-0.6f * log2f((float)t + 1.0f)) : 0.0f;
    const float flat = BND_FLAT * (float)F;
    // the visited colours, cell phase major: phase, block row, column
    auto settle = [&](int& p, int& y, int& x) {                     // from (p, y, x) to the next one with a cell here
        while ((p * s + y) * s + x < k1) {
            if (y >= bh) {
                ++p;
                y = 0;
                x = 0;
            } else if (x >= bw) {
                ++y;
                x = 0;
            } else {
                return true;
            }
        }
        return false;
    };
    auto cell = [&](int p, int y, int x) {
        return SUB ? base + (int64_t)((by0 + y) * k + p / k) * f.W + ((bx0 + x) * k + p % k)
                   : base + (int64_t)(by0 + y) * f.W + (bx0 + x);
    };
    float4 n_pr = make_float4(0.0f, 0.0f, 0.0f, 0.0f);              // the next row's inputs, column x in lane x
    float n_ls = 0.0f;
    auto prefetch = [&](int p, int y) {
        if (lane >= bw) return;
        const int64_t i = cell(p, y, lane);
        n_pr = S.prop[i];
        if (t < burn_in) n_ls = S.log_step[i];
    };
    int ph = k0 / F, ly = (k0 - ph * F) / s, lx0 = k0 % s, ph_w = -1;
    bool more = settle(ph, ly, lx0);
    if (more) prefetch(ph, ly);
    unsigned n_acc = 0;
    int par = 0, cq = 0;
    while (more) {
        const float4 pr = n_pr;
        const float ls = n_ls;
        int nph = ph, nly = ly, nlx = s;
        more = settle(nph, nly, nlx);
        if (more) prefetch(nph, nly);
        if (SUB && ph != ph_w) {
            ph_w = ph;
#pragma unroll
            for (int q = 0; q < NQ; ++q) pw[q] = off[q] >= 0 ? f.psf[ph * F + threadIdx.x + q * NT] : 0.0f;
        }
        const int lx1 = min(bw, k1 - (ph * s + ly) * s);
        bool my_acc = false;
        const double2 cy = DIR ? l.th[small_mod(fr.jy * ly, bh, inv_bh)] : make_double2(0.0, 0.0);
        const float cyr = (float)cy.x, cyi = (float)cy.y;
#pragma unroll 1
        for (int lx = lx0; lx < lx1; ++lx) {
            const float hast = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pr.y), lx));
            const float logu = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pr.z), lx));
            const float d0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pr.w), lx));
            const int origin = ly * RW + lx;
            // 1. centre and half-width of every term; pixels that an accepted move
            // takes out of their series' reach are queued
            float mq[NQ], cen = 0.0f, err = 0.0f, dsum = 0.0f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                mq[q] = -1.0f;
                if (q > 1 && wave0 + q * NT >= F) continue;         // none of this wave's entries
                const int i = off[q] >= 0 ? origin + off[q] : NR;
                mq[q] = l.mu[i];
                const float4 A = l.A[i];
                const float2 Bv = l.B[i];
                const float share = EM ? l.w[i] : 0.0f;
                const bool valid = mq[q] >= 0.0f;
                nevals += valid ? 1 : 0;
                const float d = mul_rn(d0, pw[q]);
                const bool out = valid && !want_delta && !(fabsf((mq[q] - A.x) + d) <= A.y);
                const TermBound tb = bounded_term<EM>(A, Bv, share, mq[q], d, out);
                // (and the rounding of the sums of centres)
                if (valid) {
                    cen += tb.c;
                    err += fmaf(1.3e-6f, fabsf(tb.c), tb.e);
                }
                const uint64_t bal = __ballot(out);
                if (bal) {
                    int slot = 0;
                    if (lane == 0) slot = atomicAdd(&l.cnt[cq], __popcll(bal));
                    slot = __builtin_amdgcn_readfirstlane(slot) + lanes_below(bal);
                    if (out) {
                        l.job[slot] = (uint16_t)i;
                        l.job_mu[slot] = fmaf(d0, pw[q], mq[q]);
                    }
                }
            }
            const int cq1 = cq == 2 ? 0 : cq + 1;
            if (threadIdx.x == 0) l.cnt[cq1] = 0;                   // read last before the previous update's barrier
            // 2. the chunk prior: with h = d / |F| and x = F conj(w) / |F|, u = h (2 Re x + h)
            // to 5e-7 h (2 + h); its logarithm and |F'| - |F| = |F| u / (1 + sqrt(1 + u))
            double2 cx = make_double2(0.0, 0.0);
            if (DIR) {
                cx = l.tw[small_mod(fr.jx * lx, bw, inv_bw)];
                const float cxr = (float)cx.x, cxi = (float)cx.y;
                const float wr = cyr * cxr - cyi * cxi, wi = -(cyi * cxr + cyr * cxi);
                const float h = d0 * finv, u = h * fmaf(2.0f, (fre * wr + fim * wi) * finv, h), u1 = 1.0f + u;
                const float du = 1e-6f * fabsf(h) * (2.0f + fabsf(h)) + 1e-7f;
                const float am = 0.5f * (fr.amA + fr.amB), rt = __builtin_amdgcn_sqrtf(u1), ir = fast_rcp(u1);
                const float lr = fast_ln(u1), ds = fr.n * fabs_F * u * fast_rcp(1.0f + rt);
                const float scale = (float)(dK - 1) * fast_rcp((float)dS_tot);
                float e = 1.5f * fabsf(am) * fmaf(du, ir, 5e-7f * fabsf(lr)) +
                          scale * fmaf(2e-6f, fabsf(ds), fr.n * fabs_F * du * rt * ir);
                if (!(du < 0.2f * u1)) e = INFINITY;
                if (fr.n > 0.0f) {
                    const bool known = e < INFINITY;
                    cen += known ? am * lr : 0.0f;
                    dsum = known ? ds : 0.0f;
                    err += known ? fmaf(1.3e-6f, fabsf(am * lr), e) : INFINITY;
                }
                dsum = wave_sum_dpp_f(dsum);
            }
            // 3. sums
            cen = wave_sum_dpp_f(cen);
            err = wave_sum_dpp_f(err);
            if (lane == 0) l.bnd[par * NW + wave] = make_float4(cen, err, dsum, 0.0f);
            lds_barrier();
            float tot_c = 0.0f, tot_e = want_delta ? INFINITY : flat, tot_s = 0.0f;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float4 v = l.bnd[par * NW + w];
                tot_c += v.x;
                tot_e += v.y;
                tot_s += v.z;
            }
            par ^= 1;
            if (DIR) {
                // - sum_k (alpha_k - 1) log(S' / S) with sum_k (alpha_k - 1) = 1 - K
                const float x = tot_s * fast_rcp((float)dS_tot), lg = (float)(dK - 1) * log1p_k(x);
                tot_e = x > -0.5f ? fmaf(2e-6f, fabsf(lg), 2.0f * tot_e) : INFINITY;
                tot_c += lg;
            }
            // 4. the decision (identical in every thread): from the bound, or, too close
            // to call (or Delta asked for), from every term's direct evaluation
            double delta = (double)tot_c + (double)hast;
            double dS = 0.0;
            bool have_dS = false;
            if (!decided(delta, logu, fmaf(1e-6f, fabsf(tot_c), tot_e))) {
                double part = 0.0;
                if (DIR) {
                    const DirDelta dd = dir_delta(fr, cy, cx, d0);
                    if (fr.n > 0.0f) {
                        part = dd.tsum;
                        dS = dd.dsum;
                    }
                    dS = wave_sum_dpp(dS);
                    if (lane == 0) l.red2[wave] = dS;
                }
#pragma unroll 1
                for (int e = threadIdx.x; e < F; e += NT) {
                    const int i = origin + (e / s) * RW + e % s;
                    const float m = l.mu[i];
                    if (m < 0.0f) continue;
                    part += delta_pix<EM>(m, mul_rn(d0, f.psf[SUB ? ph * F + e : e]), region_pc(i), inv_tab, nterms);
                    ++ndirect;
                }
                part = wave_sum_dpp(part);
                if (lane == 0) l.red[wave] = part;
                lds_barrier();
                delta = 0.0;
                dS = 0.0;
#pragma unroll 1
                for (int w = 0; w < NW; ++w) {
                    delta += l.red[w];
                    if (DIR) dS += l.red2[w];
                }
                if (DIR) delta += (double)(dK - 1) * log1p(dS / dS_tot);
                delta += (double)hast;
                have_dS = true;
            }
            const bool acc = isfinite(delta) && ((double)logu < delta);
            if (lane == lx) my_acc = acc;
            if (want_delta && threadIdx.x == 0) {
                const int64_t i = cell(ph, ly, lx);
                if (dbg_delta) dbg_delta[i] = (float)delta;
                if (dbg_acc) dbg_acc[i] = acc ? 1 : 0;
            }
            if (acc) {
                ++n_acc;
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    if (mq[q] >= 0.0f) l.mu[origin + off[q]] = fmaf(d0, pw[q], mq[q]);
                if (DIR) {
                    const DirDelta dd = dir_delta(fr, cy, cx, d0);
                    if (!have_dS) {
                        dS = wave_sum_dpp(fr.n > 0.0f ? dd.dsum : 0.0);
                        if (lane == 0) l.red2[wave] = dS;
                    }
                    fr.re = fma((double)d0, dd.wr, fr.re);
                    fr.im = fma((double)d0, dd.wi, fr.im);
                    if (fr.n > 0.0f) dir_round();
                }
                // re-anchor the queued pixels at their new means
                const int n = l.cnt[cq], id = threadIdx.x ^ (NT - 64);
                if constexpr (EM) {
                    for (int j = id; j < n; j += NT) anchor_em(l.job[j], l.job_mu[j]);
                } else {
                    for (int j = id >> 2; j < n; j += NT / 4) {
                        const int i = l.job[j];
                        const float m = l.job_mu[j];
                        const Series sr = series_after(m, 0.0f, region_pc(i), id & 3, aterms);
                        if ((id & 3) == 0) set_series(i, m, sr);
                    }
                }
                lds_barrier();                                      // commits before the next footprint reads
                if (DIR) {
                    if (!have_dS) {
                        dS = 0.0;
#pragma unroll 1
                        for (int w = 0; w < NW; ++w) dS += l.red2[w];
                    }
                    dS_tot += dS;
                }
            }
            cq = cq1;
        }
        if (wave == 0 && lane >= lx0 && lane < lx1) {
            const int64_t i = cell(ph, ly, lane);
            if (my_acc) S.rho[i] = pr.x;
            if (t < burn_in) S.log_step[i] = fmaf(gain, (my_acc ? 1.0f : 0.0f) - 0.44f, ls);
        }
        ph = nph;
        ly = nly;
        lx0 = nlx;
    }
    if (threadIdx.x == 0) atomicAdd(&S.accepts[chain], (unsigned long long)n_acc);
    for (int i = threadIdx.x; i < NR; i += NT) {
        const int y = i / RW, yy = ry0 + y, xx = rx0 + i - y * RW;
        if (yy >= 0 && yy < f.Hp && xx >= 0 && xx < f.Wp) S.mu[pbase + (int64_t)yy * f.Wp + xx] = l.mu[i];
    }
    count_work5(S.counters, nterms, nevals, ndirect, nanch, aterms);
}

template <bool EM, bool DIR, bool SUB, int NT, int NQ>
__global__ void __launch_bounds__(NT) k_block_bounded(Frame f, State S, int burn_in, const double* inv_tab, int B,
                                                      int py, int px, int k0, int k1, float* dbg_delta,
                                                      uint8_t* dbg_acc, int nblk) {
    extern __shared__ double lds_d[];
    int bi, chain;
    if (!xcd_block(nblk, f.C, bi, chain)) return;
    bounded_block<EM, DIR, SUB, NT, NQ>(f, S, burn_in, inv_tab, B, py, px, bi, chain, *S.t, k0, k1, dbg_delta,
                                        dbg_acc, reinterpret_cast<char*>(lds_d));
}

// ---------------------------------------------------------------------------
// Moments after a sweep: Welford over post-burn-in sweeps, per-batch
// statistics (mean rho, mean and M2 of log rho) for R-hat and MCSE, and
// per-workgroup partials of the log-posterior at the current mu.
// ---------------------------------------------------------------------------
// One chunk of WG pixels of one chain.
template <bool EM>
__device__ void moments_chunk(const Frame& f, const State& S, const Prior& pr, const MomentBufs& M, int burn_in,
                              int chunk, int chain, int64_t t) {
    __shared__ double s_redm[WG / 64];
    const int64_t n = (int64_t)chunk * WG + threadIdx.x;
    double lp = 0.0;
    if (n < f.N) {
        const int64_t i = (int64_t)chain * f.N + n;
        const float x = S.rho[i];
        if (t >= burn_in) {
            const float k = (float)(t - burn_in + 1);
            const float mo = M.mean[i];
            const float dlt = x - mo;
            const float mn = mo + dlt / k;
            M.mean[i] = mn;
            M.m2[i] = (t == burn_in ? 0.0f : M.m2[i]) + dlt * (x - mn);
        }
        const int64_t b = t / M.rhat_block;
        if (b < M.max_batches) {
            const int64_t CN = (int64_t)f.C * f.N;
            float* bp = M.batch + b * 3 * CN + i;
            const float lx = logf(x);
            const int j = (int)(t - b * M.rhat_block);
            if (j == 0) {
                bp[0] = x; bp[CN] = lx; bp[2 * CN] = 0.0f;
            } else {
                const float kk = (float)(j + 1);
                bp[0] += (x - bp[0]) / kk;
                const float ml = bp[CN];
                const float dl = lx - ml;
                const float ml2 = ml + dl / kk;
                bp[CN] = ml2;
                bp[2 * CN] += dl * (lx - ml2);
            }
        }
        if (n < f.Np) lp = ell_abs_cam<EM>(f, S.mu[(int64_t)chain * f.Np + n], n);   // pixels: Np <= N
        if (pr.kind == 1) lp += (double)(pr.a - 1.0f) * log((double)x) - (double)pr.b * (double)x;
    }
    lp = wave_sum(lp);
    if ((threadIdx.x & 63) == 0) s_redm[threadIdx.x >> 6] = lp;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int w = 0; w < WG / 64; ++w) tot += s_redm[w];
        M.lp_partial[(int64_t)chunk * f.C + chain] = tot;
    }
    __syncthreads();
}

template <bool EM>
__global__ void __launch_bounds__(WG) k_moments(Frame f, State S, Prior pr, MomentBufs M, int burn_in) {
    moments_chunk<EM>(f, S, pr, M, burn_in, blockIdx.x, blockIdx.y, *S.t);
}

// Fixed-order reduction of one chain's partials -> trace[t][chain].
__device__ void finalize_chain(int C, int nblk, const MomentBufs& M, int chain, int64_t t) {
    __shared__ double s_redf[WG];
    double v = 0.0;
    for (int b = threadIdx.x; b < nblk; b += WG) v += M.lp_partial[(int64_t)b * C + chain];
    s_redf[threadIdx.x] = v;
    __syncthreads();
    for (int off = WG / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) s_redf[threadIdx.x] += s_redf[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0 && t < M.max_sweeps) {
        double lp = s_redf[0];
        if (M.dir_part)
            for (int b = 0; b < M.n_chunks; ++b) lp += M.dir_part[(int64_t)b * C + chain];
        M.trace[t * C + chain] = lp;
    }
    __syncthreads();
}

// All chains' trace entries; then t += 1.
__global__ void __launch_bounds__(WG) k_finalize(int C, int nblk, MomentBufs M, int64_t* tp, int advance) {
    const int64_t t = *tp;
    for (int c = 0; c < C; ++c) finalize_chain(C, nblk, M, c, t);
    if (threadIdx.x == 0 && advance) *tp = t + 1;
}

template <bool EM>
__global__ void k_loglik(Frame f, const float* mu, double* out) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= f.Np) return;
    out[n] = ell_abs_cam<EM>(f, mu[n], n);
}

// Split R-hat per pixel on log rho from batch statistics (Chan et al.'s
// pairwise combination of means and M2).  Sequences: each chain's batches
// [b_lo, b_lo + half) and [b_lo + half, b_lo + 2 half).
__global__ void k_rhat_map(Frame f, MomentBufs M, int b_lo, int half, float* rhat) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= f.N) return;
    const int64_t CN = (int64_t)f.C * f.N;
    const double nb = (double)M.rhat_block;
    const int m = 2 * f.C;
    double sum_mean = 0.0, sum_var = 0.0, sum_mean2 = 0.0;
    double L = 0.0;
    for (int c = 0; c < f.C; ++c)
        for (int h = 0; h < 2; ++h) {
            double cnt = 0.0, mean = 0.0, m2 = 0.0;
            for (int b = b_lo + h * half; b < b_lo + (h + 1) * half; ++b) {
                const float* bp = M.batch + (int64_t)b * 3 * CN + (int64_t)c * f.N + n;
                const double bm = (double)bp[CN], bq = (double)bp[2 * CN];
                const double tot = cnt + nb;
                const double dl = bm - mean;
                mean += dl * nb / tot;
                m2 += bq + dl * dl * cnt * nb / tot;
                cnt = tot;
            }
            L = cnt;
            const double var = m2 / (cnt - 1.0);
            sum_mean += mean;
            sum_mean2 += mean * mean;
            sum_var += var;
        }
    const double gm = sum_mean / m;
    const double Bv = L * (sum_mean2 - m * gm * gm) / (m - 1);
    const double Wv = sum_var / m;
    const double vplus = (L - 1.0) / L * Wv + Bv / L;
    rhat[n] = (float)sqrt(vplus / Wv);
}

// Histogram of R-hat values: n_fine bins of width w_fine from lo, then n_coarse
// bins of width w_coarse, then one overflow bin (NaN counts as overflow).
__global__ void k_hist(const float* v, int64_t n, float lo, float w_fine, int n_fine, float w_coarse, int n_coarse,
                       unsigned int* hist) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = v[i];
    int b;
    const float top_fine = lo + w_fine * n_fine;
    if (!(x == x)) b = n_fine + n_coarse;
    else if (x < top_fine) b = x < lo ? 0 : min((int)((x - lo) / w_fine), n_fine - 1);
    else b = n_fine + min((int)((x - top_fine) / w_coarse), n_coarse);
    atomicAdd(&hist[b], 1u);
}

// Batch-means MCSE of the posterior mean per pixel, pooled over chains.
__global__ void k_mcse(Frame f, MomentBufs M, int b0, int nb, float* out) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= f.N) return;
    const int64_t CN = (int64_t)f.C * f.N;
    double acc = 0.0;
    for (int c = 0; c < f.C; ++c) {
        double s1 = 0.0, s2 = 0.0;
        for (int b = b0; b < b0 + nb; ++b) {
            const double v = (double)M.batch[(int64_t)b * 3 * CN + (int64_t)c * f.N + n];
            s1 += v;
            s2 += v * v;
        }
        const double mean = s1 / nb;
        const double var = (s2 - nb * mean * mean) / (nb - 1);
        acc += fmax(var, 0.0) / nb;
    }
    out[n] = (float)sqrt(acc / ((double)f.C * f.C));
}

__global__ void k_pooled(Frame f, MomentBufs M, int64_t ns, int chain, float* mean, float* var) {
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= f.N) return;
    if (chain >= 0) {
        const int64_t i = (int64_t)chain * f.N + n;
        if (mean) mean[n] = M.mean[i];
        if (var) var[n] = M.m2[i] / (float)(ns - 1);
        return;
    }
    double m = 0.0;
    for (int c = 0; c < f.C; ++c) m += (double)M.mean[(int64_t)c * f.N + n];
    m /= f.C;
    double ss = 0.0;
    for (int c = 0; c < f.C; ++c) {
        const double dd = (double)M.mean[(int64_t)c * f.N + n] - m;
        ss += (double)M.m2[(int64_t)c * f.N + n] + (double)ns * dd * dd;
    }
    if (mean) mean[n] = (float)m;
    if (var) var[n] = (float)(ss / ((double)f.C * ns - 1.0));
}

__global__ void k_philox(const uint4* ctr, int64_t n, uint2 key, uint4* out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = philox4x32_10(ctr[i], key);
}

__global__ void k_fill(float* p, int64_t n, float v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}


// ---------------------------------------------------------------------------
// Learned part: the frame's photon scale, the network input, the learned warm
// start, and the block independence move.
// ---------------------------------------------------------------------------
// Per-workgroup partial sums of c = (w - o)/G -> part[wg] (double).
__global__ void k_sum_c(Frame f, double* part) {
    __shared__ double s_r[WG / 64];
    const int64_t n = (int64_t)blockIdx.x * WG + threadIdx.x;
    double v = n < f.N ? (double)f.pc[n].x : 0.0;
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) s_r[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < WG / 64; ++w) t += s_r[w];
        part[blockIdx.x] = t;
    }
}

// scale = mean c if that exceeds 1e-3 photons, else 1.  One workgroup.
__global__ void k_scale(const double* part, int nw, int64_t N, float* scale) {
    __shared__ double s_r[WG];
    double v = 0.0;
    for (int i = threadIdx.x; i < nw; i += WG) v += part[i];
    s_r[threadIdx.x] = v;
    __syncthreads();
    for (int off = WG / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) s_r[threadIdx.x] += s_r[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double m = s_r[0] / (double)N;
        *scale = m > 1e-3 ? (float)m : 1.0f;
    }
}

// Network input on a zero-padded Hp x Wp grid: c / scale inside the frame.
__global__ void k_learned_input(Frame f, const float* scale, int Hp, int Wp, float* x) {
    const int64_t i = (int64_t)blockIdx.x * WG + threadIdx.x;
    if (i >= (int64_t)Hp * Wp) return;
    const int y = (int)(i / Wp), xx = (int)(i - (int64_t)y * Wp);
    x[i] = (y < f.H && xx < f.W) ? f.pc[(int64_t)y * f.W + xx].x / *scale : 0.0f;
}

// Proposal maps from the network output (m, s) and the warm start of every chain:
//   mean_log = m + log scale, sd_log = clamp(exp(s), 0.02, 3),
//   rho = exp(mean_log + sd_log xi), xi from the init stream at t = 0.
__global__ void k_learned_init(Frame f, State S, const float* out, int Wp, const float* scale, float log_step0,
                               float* pm, float* ps) {
    const int64_t n = (int64_t)blockIdx.x * WG + threadIdx.x;
    const int chain = blockIdx.y;
    if (n >= f.N) return;
    const int y = (int)(n / f.W), x = (int)(n - (int64_t)y * f.W);
    const int64_t q = (int64_t)y * Wp + x;
    float m = out[2 * q] + logf(*scale);
    float sd = expf(out[2 * q + 1]);
    if (!isfinite(m)) m = logf(fmaxf(f.pc[n].x, 0.5f));
    sd = isfinite(sd) ? fminf(fmaxf(sd, 0.02f), 3.0f) : 1.0f;
    if (chain == 0) {
        pm[n] = m;
        ps[n] = sd;
    }
    // chains start overdispersed against the network's approximation (twice
    // its spread, at most 3 in log rho), as a between-chain R-hat requires
    const float xi = box_muller(draw(f.key, (uint32_t)n, 0u, (uint32_t)chain, STREAM_INIT));
    float v = expf(m + fminf(2.0f * sd, 3.0f) * xi);
    if (!(v > 0.0f) || !isfinite(v)) v = fmaxf(f.pc[n].x, 0.5f);
    const int64_t i = (int64_t)chain * f.N + n;
    S.rho[i] = v;
    S.log_step[i] = log_step0;
}

// One colour of the block independence move.  16 x 16 blocks; colour (cy, cx)
// of the period x period block colouring; one workgroup (one thread per block
// pixel) per (block, chain).  LDS: 1/k table, PSF, mu and d-mu of the
// (16 + 2r)^2 region.
constexpr int BS = 16;

template <bool EM>
__global__ void __launch_bounds__(WG) k_block_colour(Frame f, State S, Prior pr, const float* pm, const float* ps,
                                                     const double* inv_tab, int period, int cy, int cx,
                                                     uint32_t pass, float beta, float walk, unsigned long long* bacc,
                                                     float* dbg_delta, uint8_t* dbg_acc) {
    extern __shared__ double lds_b[];
    const int s = f.s, r = f.r, RW = BS + 2 * r;
    double* s_inv = lds_b;                              // [INV_TABLE]
    double* s_red = s_inv + INV_TABLE;                  // [WG / 64]
    float* s_psf = (float*)(s_red + WG / 64);           // [s*s]
    float* s_mu = s_psf + s * s;                        // [RW*RW], -1 outside the frame
    float* s_dmu = s_mu + RW * RW;                      // [RW*RW]
    float* s_d = s_dmu + RW * RW;                       // [BS*BS]
    __shared__ int s_flag;

    const int chain = blockIdx.y;
    const int nbx = (f.W + BS - 1) / BS;
    const int nbx_c = (nbx - cx + period - 1) / period;
    const int bi = blockIdx.x;
    const int by = cy + period * (bi / nbx_c), bx = cx + period * (bi % nbx_c);
    const int by0 = by * BS, bx0 = bx * BS;
    const int ry0 = by0 - r, rx0 = bx0 - r;
    const int64_t base = (int64_t)chain * f.N;

    for (int i = threadIdx.x; i < INV_TABLE; i += WG) s_inv[i] = inv_tab[i];
    for (int j = threadIdx.x; j < s * s; j += WG) s_psf[j] = f.psf[j];
    for (int i = threadIdx.x; i < RW * RW; i += WG) {
        const int yy = ry0 + i / RW, xx = rx0 + i % RW;
        s_mu[i] = (yy >= 0 && yy < f.H && xx >= 0 && xx < f.W) ? S.mu[base + (int64_t)yy * f.W + xx] : -1.0f;
    }
    // this thread's block pixel: proposal, log q(rho) - log q(rho'), prior ratio
    const int ty = threadIdx.x / BS, tx = threadIdx.x % BS;
    const int y = by0 + ty, x = bx0 + tx;
    double term = 0.0;
    float rp = 0.0f;
    float d = 0.0f;
    const bool inside = y < f.H && x < f.W;
    if (walk > 0.0f) {
        // Walk along what the blur removes: u' = u + walk h, h = xi - P (x)_B xi,
        // the blur of the block's white noise restricted to the block's pixels
        // in the frame; symmetric in u = log rho, so the log acceptance ratio
        // carries the Jacobian sum_m (u'_m - u_m).
        const int64_t m = (int64_t)y * f.W + x;
        const float xi = inside ? box_muller(draw(f.key, (uint32_t)m, pass, (uint32_t)chain, STREAM_BLOCK)) : 0.0f;
        s_d[threadIdx.x] = xi;
        __syncthreads();
        float h = 0.0f;
        if (inside) {
            float b = 0.0f;
            const int a0 = max(0, ty - r), a1 = min(BS - 1, ty + r);
            const int c0 = max(0, tx - r), c1 = min(BS - 1, tx + r);
            for (int a = a0; a <= a1; ++a) {
                const float* prow = s_psf + (ty - a + r) * s + (tx + r);
                const float* xrow = s_d + a * BS;
                for (int c = c0; c <= c1; ++c) b = fmaf(prow[-c], xrow[c], b);
            }
            h = xi - b;
        }
        __syncthreads();
        if (inside) {
            const float r0 = S.rho[base + m];
            const float hs = walk * h;
            rp = r0 * expf(hs);
            term = (double)hs;
            if (pr.kind == 1) term += (double)(pr.a - 1.0f) * (double)hs - (double)pr.b * ((double)rp - (double)r0);
            if (!(rp > 0.0f) || !isfinite(rp)) term = -INFINITY;
            d = rp - r0;
        }
    } else if (inside) {
        const int64_t m = (int64_t)y * f.W + x;
        const float r0 = S.rho[base + m];
        const float xi = box_muller(draw(f.key, (uint32_t)m, pass, (uint32_t)chain, STREAM_BLOCK));
        const float lm = pm[m], sd = ps[m];
        const float lr0 = logf(r0);
        const float z = (lr0 - lm) / sd;
        // autoregressive step around the reference N(lm, sd^2) in log rho;
        // beta = 1 draws independently of the current value
        const float zp = beta < 1.0f ? fmaf(sqrtf(1.0f - beta * beta), z, beta * xi) : xi;
        const float lrp = fmaf(sd, zp, lm);
        rp = expf(lrp);
        term = (double)(-lr0 - 0.5f * z * z) - (double)(-lrp - 0.5f * zp * zp);
        if (pr.kind == 1) term += (double)(pr.a - 1.0f) * ((double)lrp - (double)lr0) - (double)pr.b * ((double)rp - (double)r0);
        if (!(rp > 0.0f) || !isfinite(rp)) term = -INFINITY;
        d = rp - r0;
    }
    s_d[threadIdx.x] = d;
    __syncthreads();
    // d-mu over the region and the likelihood change
    int nterms = 0;
    double part = term;
    for (int j = threadIdx.x; j < RW * RW; j += WG) {
        const int ny = j / RW, nx = j % RW;
        float acc = 0.0f;
        const int t0 = max(0, ny - 2 * r), t1 = min(BS - 1, ny);
        const int u0 = max(0, nx - 2 * r), u1 = min(BS - 1, nx);
        for (int a = t0; a <= t1; ++a) {
            const float* prow = s_psf + (ny - a) * s + nx;
            const float* drow = s_d + a * BS;
            for (int b = u0; b <= u1; ++b) acc = fmaf(drow[b], prow[-b], acc);
        }
        s_dmu[j] = acc;
        const float muv = s_mu[j];
        if (muv < 0.0f || acc == 0.0f) continue;
        const int64_t n = (int64_t)(ry0 + ny) * f.W + (rx0 + nx);
        part += delta_pix<EM>(muv, acc, load_pc(f.pc, n), s_inv, nterms);
    }
    part = wave_sum(part);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = 0.0;
        for (int w = 0; w < WG / 64; ++w) tot += s_red[w];
        const int64_t m0 = (int64_t)by0 * f.W + bx0;
        const float logu = logf(u01(draw(f.key, (uint32_t)m0, pass, (uint32_t)chain, STREAM_BLOCK_ACCEPT).x));
        const bool acc = isfinite(tot) && ((double)logu < tot);
        s_flag = acc ? 1 : 0;
        if (acc) atomicAdd(bacc, 1ull);
        const int64_t nblk = (int64_t)gridDim.x;
        if (dbg_delta) dbg_delta[(int64_t)chain * nblk + bi] = (float)tot;
        if (dbg_acc) dbg_acc[(int64_t)chain * nblk + bi] = acc ? 1 : 0;
    }
    __syncthreads();
    if (!s_flag) return;
    if (y < f.H && x < f.W) S.rho[base + (int64_t)y * f.W + x] = rp;
    for (int j = threadIdx.x; j < RW * RW; j += WG) {
        if (s_mu[j] < 0.0f) continue;
        const int yy = ry0 + j / RW, xx = rx0 + j % RW;
        S.mu[base + (int64_t)yy * f.W + xx] = s_mu[j] + s_dmu[j];
    }
}

// Training pair of one frame: the network input x = c / scale and the targets
// (mean of log(rho/scale), log std of log rho) of the log-normal with the
// posterior's mean and variance of rho.
__global__ void k_training_targets(Frame f, const float* mean, const float* var, const float* scale, float* x,
                                   float* tgt) {
    const int64_t n = (int64_t)blockIdx.x * WG + threadIdx.x;
    if (n >= f.N) return;
    const float sc = *scale;
    x[n] = f.pc[n].x / sc;
    const float m = fmaxf(mean[n], 1e-12f);
    const float s2 = log1pf(fmaxf(var[n], 0.0f) / (m * m));
    tgt[2 * n] = logf(m / sc) - 0.5f * s2;
    tgt[2 * n + 1] = 0.5f * logf(fmaxf(s2, 1e-8f));
}

// Mean of rho over batches [b0, b0 + nb) of every chain (the R-hat window).
__global__ void k_window_mean(Frame f, MomentBufs M, int b0, int nb, float* out) {
    const int64_t n = (int64_t)blockIdx.x * WG + threadIdx.x;
    if (n >= f.N) return;
    const int64_t CN = (int64_t)f.C * f.N;
    double s = 0.0;
    for (int c = 0; c < f.C; ++c)
        for (int b = b0; b < b0 + nb; ++b) s += (double)M.batch[(int64_t)b * 3 * CN + (int64_t)c * f.N + n];
    out[n] = (float)(s / ((double)f.C * nb));
}

inline unsigned grid1(int64_t n) { return (unsigned)((n + WG - 1) / WG); }

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_pixel_consts(const Frame& f, float4* pc, int* bad, hipStream_t st) {
    hipLaunchKernelGGL(k_pixel_consts, dim3(grid1(f.Np)), dim3(WG), 0, st, f, pc, bad);
    return hipGetLastError();
}

hipError_t launch_init_state(const Frame& f, const State& S, const float* rho0, float log_step0, int* bad,
                             hipStream_t st) {
    hipLaunchKernelGGL(k_init_state, dim3(grid1(f.N), f.C), dim3(WG), 0, st, f, S, rho0, log_step0, bad);
    return hipGetLastError();
}

hipError_t launch_forward_propose(const Frame& f, const State& S, const Prior& pr, int propose, hipStream_t st) {
    if (f.sub > 1) {
        hipLaunchKernelGGL(k_forward_sub, dim3(grid1(f.Np), f.C), dim3(WG), 0, st, f, S);
        if (propose) hipLaunchKernelGGL(k_propose_sub, dim3(grid1(f.N), f.C), dim3(WG), 0, st, f, S, pr);
        return hipGetLastError();
    }
    return conv_dispatch_chains(f.N * f.C, [&](auto t) {
        using T = decltype(t);
        hipLaunchKernelGGL(k_forward_propose<T>, dim3(T::tiles(f.H, f.W), f.C), dim3(WG), T::lds(f.r), st, f, S, pr,
                           propose);
        return hipGetLastError();
    });
}

hipError_t launch_colour_pass(const Frame& f, const State& S, int burn_in, const double* inv_tab, int colour,
                              float* dbg_delta, uint8_t* dbg_acc, hipStream_t st) {
    if (f.sub > 1) {
        // colours: phase-major, then the pixel position mod s
        const int phase = colour / (f.s * f.s), cy = (colour % (f.s * f.s)) / f.s, cx = colour % f.s;
        if (phase >= f.sub * f.sub) return hipErrorInvalidValue;
        if (cy >= f.Hp || cx >= f.Wp) return hipSuccess;
        const int nrow = (f.Hp - cy + f.s - 1) / f.s, ncol = (f.Wp - cx + f.s - 1) / f.s;
        hipLaunchKernelGGL(f.camera ? k_colour_pass_sub<true> : k_colour_pass_sub<false>, dim3(nrow * ncol, f.C),
                           dim3(WG), 0, st, f, S, burn_in, inv_tab, phase, cy, cx, dbg_delta, dbg_acc);
        return hipGetLastError();
    }
    const int cy = colour / f.s, cx = colour % f.s;
    if (cy >= f.H || cx >= f.W) return hipSuccess;
    const int nrow = (f.H - cy + f.s - 1) / f.s, ncol = (f.W - cx + f.s - 1) / f.s;
    hipLaunchKernelGGL(f.camera ? k_colour_pass<true> : k_colour_pass<false>, dim3(nrow * ncol, f.C), dim3(WG), 0,
                       st, f, S, burn_in, inv_tab, cy, cx, dbg_delta, dbg_acc);
    return hipGetLastError();
}

size_t block_phase_lds(int B, int s) {
    const int RW = B + 2 * (s / 2);
    return (size_t)(INV_TABLE + MAX_ACT * (WG / 64)) * sizeof(double) + (size_t)(s * s + RW * RW) * sizeof(float) +
           (size_t)(s * s) * sizeof(uint16_t) + (size_t)RW * RW;
}

size_t block_phase_sub_lds(int B, int s, int k) {
    const int RW = B + 2 * (s / 2);
    return (size_t)(INV_TABLE + MAX_ACT * WAVES) * sizeof(double) + (size_t)(k * k * s * s + RW * RW) * sizeof(float) +
           (size_t)(s * s) * sizeof(uint16_t);
}

// Grid of a block scan over nblk blocks and C chains (xcd_block): ids
// 0 .. XCDS * C * ceil(nblk / XCDS) - 1 in dispatch order (x fastest), rows of
// up to 65536 groups of XCDS * C workgroups.
static dim3 xcd_grid(int nblk, int C) {
    const int nq = (nblk + XCDS - 1) / XCDS;
    const int qx = std::min(nq, 65536);
    return dim3((unsigned)(XCDS * C * qx), (unsigned)((nq + qx - 1) / qx));
}

// The bounded pass takes the readings, priors and lattices that have no series
// scan, with one cell per block and colour and a region within the LDS.  Outside it are
// the blocks of B = 8 that AUTO gives to footprints below side 8 (several cells per
// colour), EMCCD sides from 37 on and the EMCCD tiles of a batch, whose items share one
// workgroup of four waves and 64 KB: these run the all-direct pass, several times slower.  It was
// the faster one at every size tried, from 100 x 134 (PSF 11, 3 chains: 1.8 against
// 9.1 ms for two sweeps of the all-direct pass) to 1536^2 (PSF 31, 4 chains: 130 against
// 1358 ms).  Larger blocks and regions keep the all-direct pass.
static bool bounded_fits(const Frame& f, int B) {
    if (!f.camera && !f.dir_am1 && f.sub == 1) return false;
    if (f.dir_am1 && (f.sub > 1 || B != f.dir_B || B > DIR_MAX_B)) return false;
    return B >= f.s - 1 && B >= 1 && B <= f.s && f.s * f.s <= BND_MAX_F &&
           bounded_layout(B, f.s, f.camera != 0, f.dir_am1 != nullptr, nullptr, nullptr) <= BND_LDS_MAX;
}

template <bool EM, bool DIR, bool SUB, int NT, int NQ>
static hipError_t launch_bounded_as(const Frame& f, const State& S, int burn_in, const double* inv_tab, int B,
                                    int phase, int k0, int k1, float* dbg_delta, uint8_t* dbg_acc, hipStream_t st) {
    const int py = phase / 2, px = phase % 2;
    const int nby = (f.Hp + B - 1) / B, nbx = (f.Wp + B - 1) / B;
    const int nblk = ((nby - py + 1) / 2) * ((nbx - px + 1) / 2);
    if (nblk <= 0) return hipSuccess;
    auto kern = k_block_bounded<EM, DIR, SUB, NT, NQ>;
    static OncePerDevice once;
    const hipError_t e = allow_lds(once, (const void*)kern, BND_LDS_MAX);
    if (e != hipSuccess) return e;
    const size_t lds = bounded_layout(B, f.s, EM, DIR, nullptr, nullptr);
    hipLaunchKernelGGL(kern, xcd_grid(nblk, f.C), dim3(NT), lds, st, f, S, burn_in, inv_tab, B, py, px, k0, k1,
                       dbg_delta, dbg_acc, nblk);
    return hipGetLastError();
}

static hipError_t launch_bounded(const Frame& f, const State& S, int burn_in, const double* inv_tab, int B, int phase,
                                 int k0, int k1, float* dbg_delta, uint8_t* dbg_acc, hipStream_t st) {
    auto sized = [&](auto em, auto dir, auto sub) {
        constexpr bool E = decltype(em)::value, D = decltype(dir)::value, U = decltype(sub)::value;
        const int F = f.s * f.s;
        auto go = [&](auto fn) { return fn(f, S, burn_in, inv_tab, B, phase, k0, k1, dbg_delta, dbg_acc, st); };
        if (F <= 256) return go(launch_bounded_as<E, D, U, 256, 1>);
        if (F <= 512) return go(launch_bounded_as<E, D, U, 512, 1>);
        if (F <= 1024) return go(launch_bounded_as<E, D, U, 512, 2>);
        if constexpr (!D) return go(launch_bounded_as<E, D, U, 512, 3>);
        return hipErrorInvalidValue;
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    if (f.sub > 1) return f.camera ? sized(yes, no, yes) : sized(no, no, yes);
    if (f.dir_am1) return f.camera ? sized(yes, yes, no) : sized(no, yes, no);
    return sized(yes, no, no);
}

hipError_t launch_block_phase(const Frame& f, const State& S, int burn_in, const double* inv_tab, int B,
                              int phase, int k0, int k1, float* dbg_delta, uint8_t* dbg_acc, hipStream_t st) {
    if (bounded_fits(f, B)) return launch_bounded(f, S, burn_in, inv_tab, B, phase, k0, k1, dbg_delta, dbg_acc, st);
    if (f.sub > 1) {
        const int py = phase / 2, px = phase % 2;
        const int nby = (f.Hp + B - 1) / B, nbx = (f.Wp + B - 1) / B;
        const int nby_p = (nby - py + 1) / 2, nbx_p = (nbx - px + 1) / 2;
        if (nby_p <= 0 || nbx_p <= 0) return hipSuccess;
        const size_t lds = block_phase_sub_lds(B, f.s, f.sub);
        if (B < f.s - 1 || B < 1 || B > 4 * f.s || lds > 64 * 1024 || f.dir_am1) return hipErrorInvalidValue;
        hipLaunchKernelGGL(f.camera ? k_block_phase_sub<true> : k_block_phase_sub<false>,
                           xcd_grid(nby_p * nbx_p, f.C), dim3(WG), lds, st, f, S, burn_in, inv_tab, B, py, px, k0, k1,
                           dbg_delta, dbg_acc, nby_p * nbx_p);
        return hipGetLastError();
    }
    const int py = phase / 2, px = phase % 2;
    const int nby = (f.H + B - 1) / B, nbx = (f.W + B - 1) / B;
    const int nby_p = (nby - py + 1) / 2, nbx_p = (nbx - px + 1) / 2;
    if (nby_p <= 0 || nbx_p <= 0) return hipSuccess;
    if (f.dir_am1) return hipErrorInvalidValue;              // one pixel per block and colour, B <= s <= 31
    hipLaunchKernelGGL(f.camera ? k_block_phase<true> : k_block_phase<false>, xcd_grid(nby_p * nbx_p, f.C),
                       dim3(WG), block_phase_lds(B, f.s), st, f, S, burn_in, inv_tab, B, py, px, k0, k1, dbg_delta,
                       dbg_acc, nby_p * nbx_p);
    return hipGetLastError();
}

int chunk_count(const Frame& f) {
    const int B = f.dir_B;
    return B > 0 ? ((f.H + B - 1) / B) * ((f.W + B - 1) / B) : 0;
}

static size_t chunk_fourier_lds(int B) { return (size_t)(3 * B * B + 4 * B + WAVES) * sizeof(double); }

hipError_t launch_chunk_spectra(const Frame& f, const State& S, hipStream_t st) {
    if (!f.dir_am1) return hipSuccess;
    MomentBufs M{};
    hipLaunchKernelGGL(k_chunk_fourier<0>, dim3(chunk_count(f), f.C), dim3(WG), chunk_fourier_lds(f.dir_B), st, f,
                       S, M);
    return hipGetLastError();
}

hipError_t launch_chunk_logprior(const Frame& f, const State& S, const MomentBufs& M, hipStream_t st) {
    if (!f.dir_am1 || !M.dir_part) return hipSuccess;
    hipLaunchKernelGGL(k_chunk_fourier<1>, dim3(chunk_count(f), f.C), dim3(WG), chunk_fourier_lds(f.dir_B), st, f,
                       S, M);
    return hipGetLastError();
}

size_t block_series_lds(int B, int s) {
    return block_series_fixed(B, s) + (size_t)block_series_jobs(B, s) * SER_JOB_BYTES;
}

bool block_series_fits(int B, int s) {
    return B <= s && B >= s - 1 && B >= 1 && s * s <= SER_Q * WG && block_series_lds(B, s) <= BLOCK_SERIES_LDS_MAX;
}

// Entries per lane of the instantiations: whole footprints up to sides 11, 15, 19, 21 and 32
// (an instantiation's every entry is evaluated).  64^2, Gaussian 11 x 11, 4 chains, 20 sweeps:
// 50.6 ms with four entries, 45.6 with two; 929 x 914, Airy 19 x 19, 3 sweeps: 11.7 with eight,
// 11.0 with six.  A batch runs its tiles with 4, 7 or 16: five kinds of pass are five
// branches of its graph, which took 77.6 ms for 64 tiles where three take 71.1.
int wave_entries(int s) {
    const int n = (s * s + 63) / 64;
    return n <= 2 ? 2 : n <= 4 ? 4 : n <= 6 ? 6 : n <= 7 ? 7 : 16;
}

size_t wave_series_lds(int B, int s) {
    const int RW = B + 2 * (s / 2);
    const int cap = ws_cap(wave_entries(s));
    return (cap + 1) * sizeof(float4) + (cap + 4) * sizeof(int) +
           ((size_t)s * RW + 1) * (sizeof(float4) + sizeof(float2) + sizeof(float));
}

bool wave_series_fits(int B, int s) {
    return B <= s && 2 * B >= s - 1 && B >= 1 && s * s <= WS_NQ * 64 && wave_series_lds(B, s) <= 64 * 1024;
}

hipError_t launch_wave_series(const Frame& f, const State& S, int burn_in, int B, int phase, int k0, int k1,
                              float* dbg_delta, uint8_t* dbg_acc, hipStream_t st) {
    if (!wave_series_fits(B, f.s)) return hipErrorInvalidValue;
    const int py = phase / 3, px = phase % 3;
    const int nby = (f.H + B - 1) / B, nbx = (f.W + B - 1) / B;
    const int nby_p = (nby - py + 2) / 3, nbx_p = (nbx - px + 2) / 3;
    if (nby_p <= 0 || nbx_p <= 0) return hipSuccess;
    const size_t lds = wave_series_lds(B, f.s);
    const dim3 grid = xcd_grid(nby_p * nbx_p, f.C);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(64), lds, st, f, S, burn_in, B, py, px, k0, k1, dbg_delta, dbg_acc,
                           nby_p * nbx_p);
    };
    switch (wave_entries(f.s)) {
        case 2: go(k_wave_series<2>); break;
        case 4: go(k_wave_series<4>); break;
        case 6: go(k_wave_series<6>); break;
        case 7: go(k_wave_series<7>); break;
        default: go(k_wave_series<16>); break;
    }
    return hipGetLastError();
}

hipError_t launch_block_series(const Frame& f, const State& S, int burn_in, const double* inv_tab, int B, int phase,
                               int k0, int k1, float* dbg_delta, uint8_t* dbg_acc, hipStream_t st) {
    if (!block_series_fits(B, f.s)) return hipErrorInvalidValue;
    const int py = phase / 2, px = phase % 2;
    const int nby = (f.H + B - 1) / B, nbx = (f.W + B - 1) / B;
    const int nby_p = (nby - py + 1) / 2, nbx_p = (nbx - px + 1) / 2;
    if (nby_p <= 0 || nbx_p <= 0) return hipSuccess;
    const size_t lds = block_series_lds(B, f.s);
    (void)inv_tab;   // the pass computes its reciprocals (no table in its LDS budget)
    const int nblk = nby_p * nbx_p;
    auto go = [&](auto entries) {
        auto kern = k_block_series<decltype(entries)::value>;
        static OncePerDevice once;
        const hipError_t e = allow_lds(once, (const void*)kern, BLOCK_SERIES_LDS_MAX);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, xcd_grid(nblk, f.C), dim3(WG), lds, st, f, S, burn_in, B, py, px, k0, k1, dbg_delta,
                           dbg_acc, nblk);
        return hipGetLastError();
    };
    // Three entries per thread hold the footprints up to side 27, four all up to 31.  The
    // fourth of the smaller ones is padding that every update reads: six sweeps of 301 x 388, 4
    // chains, scalar camera, four and three entries: side 23 25.4 and 24.3 ms, side 25
    // 30.3 and 28.8, side 27 35.9 and 34.1.  (A batch runs all its tiles with four.)
    return f.s * f.s <= 3 * WG ? go(std::integral_constant<int, 3>{}) : go(std::integral_constant<int, SER_Q>{});
}

hipError_t launch_moments(const Frame& f, const State& S, const Prior& pr, const MomentBufs& M, int burn_in,
                          int advance, hipStream_t st) {
    const unsigned nblk = grid1(f.N);
    hipLaunchKernelGGL(f.camera ? k_moments<true> : k_moments<false>, dim3(nblk, f.C), dim3(WG), 0, st, f, S, pr, M,
                       burn_in);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_chunk_logprior(f, S, M, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(WG), 0, st, f.C, (int)nblk, M, S.t, advance);
    return hipGetLastError();
}

hipError_t launch_loglik(const Frame& f, const float* mu, double* out, hipStream_t st) {
    hipLaunchKernelGGL(f.camera ? k_loglik<true> : k_loglik<false>, dim3(grid1(f.Np)), dim3(WG), 0, st, f, mu, out);
    return hipGetLastError();
}

hipError_t launch_rhat_map(const Frame& f, const MomentBufs& M, int b_lo, int half, float* rhat, hipStream_t st) {
    hipLaunchKernelGGL(k_rhat_map, dim3(grid1(f.N)), dim3(WG), 0, st, f, M, b_lo, half, rhat);
    return hipGetLastError();
}

hipError_t launch_hist(const float* v, int64_t n, float lo, float w_fine, int n_fine, float w_coarse, int n_coarse,
                       unsigned int* hist, hipStream_t st) {
    hipLaunchKernelGGL(k_hist, dim3(grid1(n)), dim3(WG), 0, st, v, n, lo, w_fine, n_fine, w_coarse, n_coarse, hist);
    return hipGetLastError();
}

hipError_t launch_mcse(const Frame& f, const MomentBufs& M, int b0, int nb, float* mcse, hipStream_t st) {
    hipLaunchKernelGGL(k_mcse, dim3(grid1(f.N)), dim3(WG), 0, st, f, M, b0, nb, mcse);
    return hipGetLastError();
}

hipError_t launch_pooled_moments(const Frame& f, const MomentBufs& M, int64_t n, int chain, float* mean,
                                 float* var, hipStream_t st) {
    hipLaunchKernelGGL(k_pooled, dim3(grid1(f.N)), dim3(WG), 0, st, f, M, n, chain, mean, var);
    return hipGetLastError();
}

hipError_t launch_philox(const uint32_t* ctr, int64_t n, uint2 key, uint32_t* out, hipStream_t st) {
    hipLaunchKernelGGL(k_philox, dim3(grid1(n)), dim3(WG), 0, st, (const uint4*)ctr, n, key, (uint4*)out);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, int64_t n, float v, hipStream_t st) {
    hipLaunchKernelGGL(k_fill, dim3(grid1(n)), dim3(WG), 0, st, p, n, v);
    return hipGetLastError();
}

int block_period(int r) { return 1 + (2 * r + BS - 1) / BS; }

int block_colour_count(const Frame& f, int colour) {
    const int P = block_period(f.r);
    const int cy = colour / P, cx = colour % P;
    const int nby = (f.H + BS - 1) / BS, nbx = (f.W + BS - 1) / BS;
    if (cy >= nby || cx >= nbx) return 0;
    return ((nby - cy + P - 1) / P) * ((nbx - cx + P - 1) / P);
}

size_t block_colour_lds(int s) {
    const int RW = BS + s - 1;
    return (size_t)(INV_TABLE + WG / 64) * sizeof(double) + (size_t)(s * s + 2 * RW * RW + BS * BS) * sizeof(float);
}

hipError_t launch_block_colour(const Frame& f, const State& S, const Prior& pr, const float* pm, const float* ps,
                               const double* inv_tab, int colour, uint32_t pass, float beta, float walk,
                               unsigned long long* bacc, float* dbg_delta, uint8_t* dbg_acc, hipStream_t st) {
    const int P = block_period(f.r);
    const int nb = block_colour_count(f, colour);
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(f.camera ? k_block_colour<true> : k_block_colour<false>, dim3(nb, f.C), dim3(WG),
                       block_colour_lds(f.s), st, f, S, pr, pm, ps, inv_tab, P, colour / P, colour % P, pass, beta,
                       walk, bacc, dbg_delta, dbg_acc);
    return hipGetLastError();
}

hipError_t launch_training_targets(const Frame& f, const float* mean, const float* var, const float* scale, float* x,
                                   float* tgt, hipStream_t st) {
    hipLaunchKernelGGL(k_training_targets, dim3(grid1(f.N)), dim3(WG), 0, st, f, mean, var, scale, x, tgt);
    return hipGetLastError();
}

hipError_t launch_window_mean(const Frame& f, const MomentBufs& M, int b0, int nb, float* out, hipStream_t st) {
    hipLaunchKernelGGL(k_window_mean, dim3(grid1(f.N)), dim3(WG), 0, st, f, M, b0, nb, out);
    return hipGetLastError();
}

hipError_t launch_frame_scale(const Frame& f, double* part, float* scale, hipStream_t st) {
    const unsigned nw = grid1(f.N);
    hipLaunchKernelGGL(k_sum_c, dim3(nw), dim3(WG), 0, st, f, part);
    hipLaunchKernelGGL(k_scale, dim3(1), dim3(WG), 0, st, part, (int)nw, f.N, scale);
    return hipGetLastError();
}

hipError_t launch_learned_input(const Frame& f, const float* scale, int Hp, int Wp, float* x, hipStream_t st) {
    hipLaunchKernelGGL(k_learned_input, dim3(grid1((int64_t)Hp * Wp)), dim3(WG), 0, st, f, scale, Hp, Wp, x);
    return hipGetLastError();
}

hipError_t launch_learned_init(const Frame& f, const State& S, const float* out, int Wp, const float* scale,
                               float log_step0, float* pm, float* ps, hipStream_t st) {
    hipLaunchKernelGGL(k_learned_init, dim3(grid1(f.N), f.C), dim3(WG), 0, st, f, S, out, Wp, scale, log_step0, pm,
                       ps);
    return hipGetLastError();
}

}  // namespace bdc

namespace bdc {
namespace {

using BatchConv = ConvTile<8, 4>;

__global__ void k_batch_advance(int64_t* const* tps, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) *tps[i] += 1;
}

// One item per workgroup: every item of one segment (one level, one kind of
// work, all tiles and chains).  Items of a segment are independent; the
// segment before finished with the previous launch, so no workgroup ever
// waits for another.
// Three waves per SIMD, as for the single-frame block-series kernel: the
// tile descriptor's indirection would otherwise take the series body just past
// the register count at which three fit.
template <int KIND>
__global__ void __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(3)))
k_batch(const TileDesc* tiles, const Item* items, const double* inv_tab) {
    extern __shared__ double lds_b[];
    const Item I = items[blockIdx.x];
    const TileDesc& T = tiles[I.tile];
    const int64_t t = *T.S.t;
    const int ph = I.level - 1;
    if constexpr (KIND == BK_FORWARD) {
        forward_tile<BatchConv>(T.f, T.S, T.pr, 1, I.index, I.chain, t, (float*)lds_b);
    } else if constexpr (KIND == BK_SERIES) {
        // (copies: through the descriptor every update would load their fields again; with
        // those of the nine-phase items 64 tiles, three sweeps: 72.8 to 67.8 ms)
        const Frame f = T.f;
        const State S = T.S;
        block_series_block<SER_Q>(f, S, T.burn_in, T.B, ph / 2, ph % 2, I.index, I.chain, t, 0, f.s * f.s, nullptr, nullptr,
                                  lds_b);
    } else if constexpr (KIND == BK_PHASE || KIND == BK_PHASE_EM) {
        block_phase_block<KIND == BK_PHASE_EM>(T.f, T.S, T.burn_in, inv_tab, T.B, ph / 2, ph % 2, I.index,
                                                      I.chain, t, 0, T.f.s * T.f.s, nullptr, nullptr, lds_b);
    } else if constexpr (KIND == BK_MOMENTS || KIND == BK_MOMENTS_EM) {
        moments_chunk<KIND == BK_MOMENTS_EM>(T.f, T.S, T.pr, T.M, T.burn_in, I.index, I.chain, t);
    } else {
        finalize_chain(T.f.C, T.count[LEV_MOMENTS], T.M, I.chain, t);
    }
}

// Nine-phase block-series items: one wavefront each.
template <int NQ>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(wave_occupancy(NQ)))) k_batch_wave(const TileDesc* tiles, const Item* items) {
    extern __shared__ double lds_b[];
    const Item I = items[blockIdx.x];
    const TileDesc& T = tiles[I.tile];
    const int ph = I.level - 1;
    const Frame f = T.f;
    const State S = T.S;
    wave_series_block<NQ>(f, S, T.burn_in, T.B, ph / 3, ph % 3, I.index, I.chain, *T.S.t, 0, f.s * f.s,
                          nullptr, nullptr, lds_b);
}

}  // namespace

size_t forward_lds(int s) { return BatchConv::lds(s / 2); }
int forward_items(int h, int w) { return BatchConv::tiles(h, w); }

hipError_t launch_batch_level(int kind, const TileDesc* tiles, const Item* items, int n_items,
                              const double* inv_tab, size_t lds, hipStream_t st) {
    if (n_items <= 0) return hipSuccess;
    const dim3 g(n_items), blk(WG);
    switch (kind) {
        case BK_FORWARD: hipLaunchKernelGGL(k_batch<BK_FORWARD>, g, blk, lds, st, tiles, items, inv_tab); break;
        case BK_SERIES: hipLaunchKernelGGL(k_batch<BK_SERIES>, g, blk, lds, st, tiles, items, inv_tab); break;
        case BK_PHASE: hipLaunchKernelGGL(k_batch<BK_PHASE>, g, blk, lds, st, tiles, items, inv_tab); break;
        case BK_MOMENTS: hipLaunchKernelGGL(k_batch<BK_MOMENTS>, g, blk, lds, st, tiles, items, inv_tab); break;
        case BK_FINALIZE: hipLaunchKernelGGL(k_batch<BK_FINALIZE>, g, blk, lds, st, tiles, items, inv_tab); break;
        case BK_WAVE4: hipLaunchKernelGGL(k_batch_wave<4>, g, dim3(64), lds, st, tiles, items); break;
        case BK_WAVE7: hipLaunchKernelGGL(k_batch_wave<7>, g, dim3(64), lds, st, tiles, items); break;
        case BK_WAVE16: hipLaunchKernelGGL(k_batch_wave<16>, g, dim3(64), lds, st, tiles, items); break;
        case BK_PHASE_EM: hipLaunchKernelGGL(k_batch<BK_PHASE_EM>, g, blk, lds, st, tiles, items, inv_tab); break;
        case BK_MOMENTS_EM:
            hipLaunchKernelGGL(k_batch<BK_MOMENTS_EM>, g, blk, lds, st, tiles, items, inv_tab);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_batch_advance(int64_t* const* tps, int n, hipStream_t st) {
    hipLaunchKernelGGL(k_batch_advance, dim3((n + WG - 1) / WG), dim3(WG), 0, st, tps, n);
    return hipGetLastError();
}

}  // namespace bdc
