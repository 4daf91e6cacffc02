// The resampler's tables on the host: interpolation taps by phase, and their matrix form (see
// resample_bands_kernel in audio.hip).  Plain C++, so that the tests can look at them without a GPU.
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace prep {

constexpr int kZeroCrossings = 6;
constexpr double kRolloff = 0.99;
constexpr int kBandQuadsMost = 6;                     // S / 4: a band of 96 samples, p / q up to about 3.4

struct BandPlan {
    int32_t P, Q;          // the period
    int32_t blocks;        // of sixteen phases
    int32_t quads;         // S / 4; 0 = the rates are not for this kernel
};
// A rate pair p : q (reduced) is accepted up to this size of either term; its tap table has q
// rows of at most 2 * 6 / 0.99 * max(p / q, 1) + 2 taps, fewer than 14 * max(p, q) + 2 q entries.
constexpr int kMaxRateTerm = 4096;
constexpr size_t kMaxTapEntries = 16 * (size_t)kMaxRateTerm;
// Entry of `bands` for sample n of block b's band and phase 16 b + j
constexpr size_t band_entry(int quads, int b, int n, int j)
{
    return ((size_t)(b * quads + n / 16) * 4 + (size_t)(n % 4)) * 64 + (size_t)(n % 16 / 4) * 16 + (size_t)j;
}

inline double sinc(double u) { return u == 0.0 ? 1.0 : sin(M_PI * u) / (M_PI * u); }

inline uint64_t resampled_length(uint64_t len, int p, int q) { return (len * (uint64_t)q + (uint64_t)p - 1) / (uint64_t)p; }

// taps[j][r] = h((first[r] + j) / p - r / q) for phase r of p : q (input : output rate, reduced)
inline void make_taps(int p, int q, std::vector<double> *taps, std::vector<int32_t> *first, int *n_taps)
{
    const double base = kRolloff * std::min(p, q);
    const double reach = kZeroCrossings / base * p;  // in input samples
    int width = 0;
    first->resize((size_t)q);
    std::vector<int> last((size_t)q);
    for (int r = 0; r < q; r++) {
        const double centre = (double)r * p / q;
        (*first)[(size_t)r] = (int32_t)ceil(centre - reach);
        last[(size_t)r] = (int)floor(centre + reach);
        width = std::max(width, last[(size_t)r] - (*first)[(size_t)r] + 1);
    }
    *n_taps = width;
    taps->assign((size_t)q * width, 0.0);
    for (int r = 0; r < q; r++)
        for (int j = 0; j < width; j++) {
            const int n = (*first)[(size_t)r] + j;
            const double uarg = base * ((double)n / p - (double)r / q);
            if (fabs(uarg) < kZeroCrossings && n <= last[(size_t)r]) {
                const double c = cos(M_PI * uarg / (2.0 * kZeroCrossings));
                (*taps)[(size_t)j * q + r] = (base / p) * sinc(uarg) * c * c;
            }
        }
}

// The matrix form of these taps, in place of them, if the rates are for it: the shortest period
// that fills its blocks of sixteen phases to 98 %, or the one of at most sixteen times p : q, with
// room for its table, that fills them best.
inline void make_bands(int p, int q, int n_taps, std::vector<double> *taps, std::vector<int32_t> *first, BandPlan *plan)
{
    *plan = BandPlan{};
    const int most = (n_taps + (15 * p + q - 1) / q + 1 + 15) / 16;  // quads of a band
    int m = 0;
    double best = 0.0;
    for (int k = 1; k <= 16 && best < 0.98; k++) {
        if ((size_t)((q * k + 15) / 16) * (size_t)std::max(2, most) * 256 > kMaxTapEntries) break;
        const double used = (double)q * k / (16.0 * ((q * k + 15) / 16));
        if (used > best + 1e-9) { best = used; m = k; }
    }
    if (m == 0) return;
    BandPlan t;
    t.P = p * m;
    t.Q = q * m;
    t.blocks = (t.Q + 15) / 16;
    auto start = [&](int r) { return (*first)[(size_t)(r % q)] + r / q * p; };
    int width = 0;
    for (int b = 0; b < t.blocks; b++)
        width = std::max(width, start(std::min(16 * b + 15, t.Q - 1)) + n_taps - start(16 * b));
    t.quads = std::max(2, (width + 15) / 16);
    if (t.quads > kBandQuadsMost) return;
    std::vector<double> bands((size_t)t.blocks * (size_t)t.quads * 256, 0.0);
    std::vector<int32_t> starts((size_t)t.blocks);
    for (int b = 0; b < t.blocks; b++) starts[(size_t)b] = start(16 * b);
    for (int r = 0; r < t.Q; r++)
        for (int k = 0; k < n_taps; k++)
            bands[band_entry(t.quads, r / 16, start(r) + k - starts[(size_t)(r / 16)], r % 16)] = (*taps)[(size_t)k * q + r % q];
    taps->swap(bands);
    first->swap(starts);
    *plan = t;
}

}  // namespace prep
