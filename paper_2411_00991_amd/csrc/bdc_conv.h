// bdc_conv.h -- same-size convolution with the PSF in FP64 (zero outside the
// image), shared by the sampler's mean refresh and Richardson-Lucy.
//
// A wave holds 64 adjacent columns x R rows of outputs, one column per lane, so
// its LDS reads are consecutive; per PSF column the R outputs of a lane slide
// down one column of the staged image, so a value is read and converted once
// for R multiply-adds, and the PSF entry, the same for every lane, comes from
// scalar memory.  What bounds it: FP64 multiply-add issue, R per (R + 1) slots
// and a read.  SPLIT waves share a block of outputs, each with a part of the PSF
// columns, and their sums are added in LDS: small images have too few outputs to
// give every SIMD a wave of its own.
#pragma once

#include "bdc_device.h"
#include "bdc_kernels.h"

namespace bdc {

template <int R, int SPLIT>
struct ConvTile {
    static constexpr int W = 64, H = R * (WG / 64 / SPLIT);

    // Row pitch of the staged image: fixed, so that the rows of a block are reached
    // by immediate offsets (W + 2 r <= PITCH, r <= 31).
    static constexpr int PITCH = 128;

    // bytes of LDS: the staged image (spare rows: a wave reads blocks ahead), or the
    // partial sums that take its place
    __host__ __device__ static size_t lds(int r) {
        const size_t tile = (size_t)(H + 2 * r + 2 * R) * PITCH * sizeof(float);
        const size_t part = SPLIT > 1 ? (size_t)(WG / 64) * R * 64 * sizeof(double) : 0;
        return tile > part ? tile : part;
    }
    static int tiles(int h, int w) { return ((h + H - 1) / H) * ((w + W - 1) / W); }

    // Output tile `tile` (row-major) of an h x w image: out(y, x, sum) for every
    // pixel of it, sum = sum over the footprint of q[c][t] in(y - r + t, x - r + c).
    // q: [2r + 1][2r + 1], column by column.
    template <class In, class Out>
    __device__ static void run(int h, int w, int r, const double* q, int tile, float* lds, In in, Out out) {
        const int s = 2 * r + 1, TW = W + 2 * r, TH = H + 2 * r;
        const int ntx = (w + W - 1) / W;
        const int y0 = (tile / ntx) * H, x0 = (tile % ntx) * W;
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        for (int y = wave; y < TH; y += WG / 64) {
            const int yy = y0 - r + y;
            for (int x = lane; x < TW; x += 64) {
                const int xx = x0 - r + x;
                lds[y * PITCH + x] = (yy >= 0 && yy < h && xx >= 0 && xx < w) ? in(yy, xx) : 0.0f;
            }
        }
        __syncthreads();
        const int row0 = (wave / SPLIT) * R, part = wave % SPLIT;
        const int per = (s + SPLIT - 1) / SPLIT, c0 = part * per, c1 = min(s, c0 + per);
        double acc[R];
#pragma unroll
        for (int i = 0; i < R; ++i) acc[i] = 0.0;
#pragma unroll 1
        for (int c = c0; c < c1; ++c) {
            const float* col = lds + row0 * PITCH + lane + c;
            const __attribute__((address_space(4))) double* qc =
                (const __attribute__((address_space(4))) double*)(q + c * s);
            double a[R], b[R];
            float n[R];
            // rows t .. t + 2R - 2 of the column in lo, hi: taps t .. t + K - 1
            auto taps = [&](const double(&lo)[R], const double(&hi)[R], int t, int K) {
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    if (k < K) {
                        const double p = qc[t + k];
#pragma unroll
                        for (int i = 0; i < R; ++i) acc[i] = fma(p, k + i < R ? lo[(k + i) % R] : hi[(k + i) % R], acc[i]);
                    }
                }
            };
            auto fetch = [&](int t) {                       // rows t .. t + R - 1
                const float* rows = col + t * PITCH;
#pragma unroll
                for (int i = 0; i < R; ++i) n[i] = rows[i * PITCH];
            };
            auto take = [&](double(&v)[R]) {
#pragma unroll
                for (int i = 0; i < R; ++i) v[i] = (double)n[i];
            };
            fetch(0);
            take(a);
            fetch(R);
            take(b);
            int t = 0;
            for (; t + 2 * R <= s; t += 2 * R) {
                fetch(t + 2 * R);
                taps(a, b, t, R);
                take(a);
                fetch(t + 3 * R);
                taps(b, a, t + R, R);
                take(b);
            }
            if (s - t >= R) {
                fetch(t + 2 * R);
                taps(a, b, t, R);
                take(a);
                taps(b, a, t + R, s - t - R);
            } else {
                taps(a, b, t, s - t);
            }
        }
        if constexpr (SPLIT == 1) {
            const int x = x0 + lane;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const int y = y0 + row0 + i;
                if (y < h && x < w) out(y, x, acc[i]);
            }
        } else {
            double* ps = reinterpret_cast<double*>(lds);    // [wave][R][64]
            __syncthreads();
#pragma unroll
            for (int i = 0; i < R; ++i) ps[(wave * R + i) * 64 + lane] = acc[i];
            __syncthreads();
            for (int o = wave; o < H; o += WG / 64) {
                const int y = y0 + o, x = x0 + lane;
                double v = 0.0;
#pragma unroll
                for (int k = 0; k < SPLIT; ++k) v += ps[((o / R * SPLIT + k) * R + o % R) * 64 + lane];
                if (y < h && x < w) out(y, x, v);
            }
        }
    }
};

// The tile for n outputs, by measurement (us for one image, PSF 31 x 31):
//   n        <2,4>   <4,4>   <8,4>   <8,2>   multiply-adds alone
//   2^14      10.7    11.4    14.2    23.6     0.4
//   2^16      11.2    11.5    14.4    23.8     1.6
//   2^17      15.9    15.0    17.1    24.1     3.2
//   2^18      21.6    17.6    17.7    24.2     6.4
//   2^20      66.3    49.9    44.7    44.9    25.6
//   2^24     982     713     627     587     410
// (the lines lie at the same n for PSFs of 11 x 11 and 63 x 63): few outputs
// need more waves and shorter chains, many need fewer reads and conversions.
//
// The mean refresh keeps to four parts of the PSF columns at any size: a split is an
// order of the FP64 sum, and a chain's means must not depend on how many chains share
// the launch or on whether its tile runs in a batch (whose items take <8, 4>).  That
// costs a refresh of 2^24 means 7 % (a sweep of 2048 x 2048, four chains, 0.1 %).
template <class F>
hipError_t conv_dispatch_chains(int64_t n, F&& launch) {
    if (n >= 1 << 18) return launch(ConvTile<8, 4>{});
    if (n >= 1 << 16) return launch(ConvTile<4, 4>{});
    return launch(ConvTile<2, 4>{});
}

// Richardson-Lucy, one image per launch: also two parts.
template <class F>
hipError_t conv_dispatch(int64_t n, F&& launch) {
    if (n >= 1 << 20) return launch(ConvTile<8, 2>{});
    return conv_dispatch_chains(n, launch);
}

}  // namespace bdc
