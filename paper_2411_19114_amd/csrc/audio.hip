// Audio preprocessing for gfx950: resample -> log-Mel spectrogram -> per-feature normalize.
//
// The audio compute units of PREBA's DPU (section 2.3 item b; section 4.2, Fig. 11(b), Table 1:
// Resample, Mel spectrogram, Normalize).  The paper names the operations only; the definitions
// are: band-limited interpolation with a Hann-windowed sinc (six zero crossings, cut-off at
// 0.99 of the lower Nyquist rate); frames of n_fft samples every hop samples, centred by
// reflecting the signal at both ends, a periodic Hann window of win_length samples centred in
// the frame, squared magnitude of the DFT; n_mels unit-peak triangles with corners equally
// spaced on m(f) = 2595 log10(1 + f/700) from 0 to half the rate; ln(x + 2^-24); per Mel
// channel and utterance mean, variance (mean squared deviation) and
// (x - mean) / (sqrt(variance) + 1e-5).
//
// Tables (interpolation taps per phase, window, twiddle factors, Mel weights) are computed on
// the host in double precision.  From the input samples to the logarithm everything is double:
// fp64 runs at the rate of unpacked fp32 on this chip, and in float the transform's rounding
// noise (a few 1e-7 of the strongest bin) would be a visible fraction of the weak high bands
// whose logarithm is taken.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <numeric>
#include <type_traits>
#include <vector>

#include "../../include/prep.h"
#include "audio_plan.h"

using namespace prep;

namespace {

constexpr float kLogGuard = 5.9604644775390625e-08f;  // 2^-24
constexpr float kStdGuard = 1e-5f;
constexpr int kFft = 512;                             // the transform the kernel is built for
constexpr int kFrameThreads = 256;                    // one wave per pair of frames
constexpr int kMaxMels = 128;

struct Utterance {
    uint64_t in_off;    // first input sample
    uint64_t mid_off;   // first resampled sample in the workspace
    uint64_t out_off;   // first output element
    uint32_t in_len, mid_len, frames, pad_;
};
constexpr size_t kRecordBytes = sizeof(Utterance) + 3 * sizeof(uint64_t);  // of one utterance and its starts
static_assert(sizeof(Utterance) % sizeof(uint64_t) == 0, "the starts behind the records are aligned");

// ---- resample -----------------------------------------------------------------------------
// Output m = a q + r of an utterance (r < q) is sum_j x[a p + first[r] + j] taps[j][r]: the
// taps depend on the phase r only.  Neighbouring lanes have neighbouring phases, so tap j of
// all phases is contiguous.
__global__ __launch_bounds__(256) void resample_kernel(const float *__restrict__ in, const Utterance *__restrict__ utt,
                                                       const uint64_t *__restrict__ mid_start, int n_utt,
                                                       const double *__restrict__ taps, const int32_t *__restrict__ first,
                                                       int p, int q, int n_taps, double *__restrict__ mid,
                                                       uint64_t total)
{
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= total) return;
    // the utterance that holds output g: the last one whose first output does not exceed g
    int lo = 0, hi = n_utt - 1;
    while (lo < hi) {
        const int m = (lo + hi + 1) >> 1;
        if (mid_start[m] <= g) lo = m; else hi = m - 1;
    }
    const Utterance u = utt[lo];
    const uint32_t m = (uint32_t)(g - u.mid_off);
    const uint32_t a = m / (uint32_t)q, r = m - a * (uint32_t)q;
    const int64_t n0 = (int64_t)a * p + first[r];
    const float *x = in + u.in_off;
    const double *t = taps + r;
    double acc = 0.0;
    if (n0 >= 0 && n0 + n_taps <= (int64_t)u.in_len) {
        // every tap lies inside the utterance
        const float *xs = x + n0;
#pragma unroll 4
        for (int j = 0; j < n_taps; j++) acc = fma((double)xs[j], t[(size_t)j * q], acc);
    } else {
        for (int j = 0; j < n_taps; j++) {
            const int64_t n = n0 + j;
            if (n >= 0 && n < (int64_t)u.in_len) acc = fma((double)x[n], t[(size_t)j * q], acc);
        }
    }
    mid[g] = acc;
}

// The same sum as a matrix product.  A period is P input and Q output samples, a multiple of p
// and q.  Sixteen neighbouring phases of a period read one band of 4 S input samples, so
//   y[a Q + 16 b + j] = sum_n x[a P + first_b + n] T_b[n][j],   n < 4 S, j < 16,
// is a product of sixteen periods' bands (rows a) with a matrix T_b that holds each phase's taps
// where they fall in the band, and zeros.  S steps of V_MFMA_F64_16X16X4_F64 make a tile of 256
// outputs.  The order of the band's samples in the sum is free: step 4 i + e takes sample
// 16 i + 4 g + e from lane group g = lane / 16, so a lane loads sixteen bytes at a time and
// four lanes of a row 64 neighbouring bytes.  A wave keeps its T_b, S doubles a lane, for all its
// tiles, and loads the next tile's samples while it multiplies.  Neighbouring waves of an XCD take the
// blocks of the same periods, so that most find the samples in its cache.
//
// 64 recordings of 1.5 to 35 s (1168 s), 44.1 to 16 kHz: 275 -> 100 us, of which the matrix
// cores are busy 40.  With a lane per output and its taps in registers 33 samples were loaded and
// converted per output, here five.  (The same with chunks staged in LDS for all phases, with
// two barriers each, took 130.)
typedef double Acc4 __attribute__((ext_vector_type(4)));
typedef float Quad __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kBandWaves = 8;                         // of a workgroup
constexpr uint32_t kXcds = 8;                         // (workgroups go to them in turn)

// Samples that a handle may be asked to hold: more than any device's memory takes (8 bytes each), and few enough
// that their sizes fit 64 bits and the tiles of resample_bands_kernel (at least 128 samples each) 30.
constexpr uint64_t kMaxSamples = 1ull << 36;

// One output by itself, its own taps only.  Out of line: inlined, it cost the kernel that calls
// it (almost never) its registers.
__device__ __attribute__((noinline)) double resample_one(const float *x, int64_t from, int64_t in_len, const double *bands,
                                                         int quads, int b, int j)
{
    double y = 0.0;
    for (int n = 0; n < 16 * quads; n++) {
        const double w = bands[band_entry(quads, b, n, j)];
        if (w != 0.0 && from + n >= 0 && from + n < in_len) y = fma((double)x[from + n], w, y);
    }
    return y;
}

// first[b] = first sample of band b, counted from the period's start; tile_start[u] = first tile of
// utterance u
template <int kQuads>
__global__ __launch_bounds__(64 * kBandWaves, 4) void resample_bands_kernel(
    const float *__restrict__ in, const Utterance *__restrict__ utt, const uint64_t *__restrict__ tile_start,
    int n_utt, uint32_t n_tiles, const double *__restrict__ bands, const int32_t *__restrict__ first, BandPlan plan,
    double *__restrict__ mid)
{
    const int lane = threadIdx.x & 63, j = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // waves that run on one XCD have neighbouring numbers (the grid is a multiple of kXcds)
    const uint32_t id = ((blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds) * kBandWaves + (uint32_t)wave;
    const uint32_t turns = gridDim.x * kBandWaves / (uint32_t)plan.blocks;  // tiles that are worked on side by side
    const int b = (int)(id % (uint32_t)plan.blocks);
    uint32_t t = id / (uint32_t)plan.blocks;
    if (t >= turns || t >= n_tiles) return;
    double tap[4 * kQuads];
#pragma unroll
    for (int s = 0; s < 4 * kQuads; s++) tap[s] = bands[((size_t)b * kQuads * 4 + s) * 64 + lane];
    const int32_t band = first[b];
    int u = 0;
    {
        int hi = n_utt - 1;
        while (u < hi) {
            const int m = (u + hi + 1) >> 1;
            if (tile_start[m] <= t) u = m; else hi = m - 1;
        }
    }
    uint32_t period = 0;  // the tile's first
    Quad v[kQuads];
    // the lane's samples of tile t (of utterance u); zeros where the utterance has none
    auto load = [&]() {
        const int64_t len = utt[u].in_len;
        const float *x = in + utt[u].in_off;
        period = (t - (uint32_t)tile_start[u]) * 16u;
        const int64_t at = (int64_t)(period + (uint32_t)j) * plan.P + band + 4 * g;
        if (at >= 0 && at + 16 * (kQuads - 1) + 4 <= len) {
#pragma unroll
            for (int i = 0; i < kQuads; i++) v[i] = *reinterpret_cast<const Quad *>(x + at + 16 * i);
        } else {
#pragma unroll
            for (int i = 0; i < kQuads; i++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const int64_t n = at + 16 * i + e;
                    v[i][e] = n >= 0 && n < len ? x[n] : 0.0f;
                }
        }
    };
    load();
    for (;;) {
        double x[4 * kQuads];
#pragma unroll
        for (int s = 0; s < 4 * kQuads; s++) x[s] = (double)v[s / 4][s % 4];
        const uint32_t here = period;
        const int uh = u;
        t += turns;
        const bool more = t < n_tiles;
        if (more) {
            while (u + 1 < n_utt && tile_start[u + 1] <= t) u++;
            load();
        }
        Acc4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4 * kQuads; s++) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[s], tap[s], acc, 0, 0, 0);
        // acc[i] is output (row g + 4 i, phase j) of the tile
        const uint32_t len = utt[uh].mid_len;
        double *y = mid + utt[uh].mid_off;
        const int phase = 16 * b + j;
        if (phase < plan.Q) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint64_t a = here + (uint32_t)(g + 4 * i), m = a * (uint32_t)plan.Q + (uint32_t)phase;
                // a sample that is no finite number makes all sixteen phases of its band one too: those
                // whose taps do not reach it are summed without it
                if (m < len) {
                    double r = acc[i];
                    if (!(fabs(r) <= 1.7976931348623157e308))
                        r = resample_one(in + utt[uh].in_off, (int64_t)a * plan.P + band, utt[uh].in_len, bands, kQuads, b, j);
                    y[m] = r;
                }
            }
        }
        if (!more) break;
    }
}

// ---- frames -> log-Mel --------------------------------------------------------------------
// The corners of the triangles cut the bins into n_mels + 1 ranges.  In range i lie the rising side of
// triangle i and the falling one of triangle i - 1 (those that do not exist, at both ends, are summed all the
// same and not used), so that every bin is read once.  Both sides are linear in the bin: a range needs
// no table of weights.
struct MelRange {
    double rising, falling, step;  // weights of the range's first bin; growth of the former from bin to bin
    int32_t start, count;          // bins
};

// ln(x) for x >= 2^-24 from x = 2^e (1 + f), 1 + f in [sqrt 1/2, sqrt 2): ln(1 + f) = 2 artanh(s), s = f / (2 + f),
// by its series up to s^19 (|s| <= 0.172: what is left out is 1e-16 of the sum).  The quotient is within
// a few units of 2^-52.  (For the device library's general logarithm the compiler takes twice
// the instructions.)
__device__ __forceinline__ double log_of(double x)
{
    double m = __builtin_amdgcn_frexp_mant(x);
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool low = m < 0.70710678118654752440;
    m = low ? 2.0 * m : m;
    e = low ? e - 1 : e;
    const double f = m - 1.0, d = 2.0 + f;
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    const double s = f * r, z = s * s;
    double q = 1.0 / 19.0;
#pragma unroll
    for (int k = 17; k >= 3; k -= 2) {
        double c = 1.0 / k;
        asm volatile("" : "+s"(c));  // a scalar register pair: the vector registers are needed
        q = fma(q, z, c);
    }
    const double y = fma((double)e, 0.69314718055994530942, fma(2.0 * s * z, q, 2.0 * s));
    return x <= 1.7976931348623157e308 ? y : x;  // infinity, and no number, as they are
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 times_minus_i(double2 a) { return make_double2(a.y, -a.x); }

// Forward DFT of four values: Y[k] = sum_n y[n] (-i)^(n k)
__device__ __forceinline__ void dft4(const double2 y[4], double2 *Y0, double2 *Y1, double2 *Y2, double2 *Y3)
{
    const double2 s02 = cadd(y[0], y[2]), d02 = csub(y[0], y[2]);
    const double2 s13 = cadd(y[1], y[3]), d13 = times_minus_i(csub(y[1], y[3]));
    *Y0 = cadd(s02, s13);
    *Y2 = csub(s02, s13);
    *Y1 = cadd(d02, d13);
    *Y3 = csub(d02, d13);
}

// Forward DFT of eight values in place, natural order: even outputs from x[n] + x[n+4], odd
// ones from (x[n] - x[n+4]) W^n, W = exp(-2 pi i / 8).
__device__ __forceinline__ void dft8(double2 v[8])
{
    constexpr double h = 0.70710678118654752440;
    double2 e[4], o[4];
#pragma unroll
    for (int n = 0; n < 4; n++) {
        e[n] = cadd(v[n], v[n + 4]);
        o[n] = csub(v[n], v[n + 4]);
    }
    o[1] = make_double2(h * (o[1].x + o[1].y), h * (o[1].y - o[1].x));     // * (1 - i) / sqrt 2
    o[2] = times_minus_i(o[2]);
    o[3] = make_double2(h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y));    // * (-1 - i) / sqrt 2
    dft4(e, &v[0], &v[2], &v[4], &v[6]);
    dft4(o, &v[1], &v[3], &v[5], &v[7]);
}

// LDS index of element i of a frame: one spare element after every eight keeps the eight lanes
// that a 16-byte access serves per cycle on different banks in every pass.
__device__ __forceinline__ int padded(int i) { return i + (i >> 3); }
constexpr int kFramePadded = kFft + kFft / 8;

// One wave per two adjacent frames a, b of an utterance, transformed together as a + i b: a
// 512-point transform in three radix-8 passes (self-sorting: pass s reads element j + 64 r,
// multiplies by W512^(r k 512 / (8 Ns)), k = j mod Ns, Ns = 8^s, transforms the eight values and
// writes them Ns apart from (j / Ns) 8 Ns + k), each lane holding eight values in registers; the
// first pass reads the signal itself.  Its outputs Z hold both spectra of the real frames,
// A[k] = (Z[k] + conj Z[512 - k]) / 2 and i B[k] = (Z[k] - conj Z[512 - k]) / 2.  A wave takes several
// pairs one after the other (per_wave; one each where there are few): it keeps the last pass's
// factors, loads the next pair's samples while it sums one's powers, and reads every power
// once (see MelRange).  117 000 frames 256 -> 140 us, 394 with one frame a transform.  Bound by the
// latency of its passes through LDS at three waves a SIMD (registers, LDS); the fp64 units are
// busy a third of the time.
// The rounding error of a quiet frame's spectrum is relative to its louder neighbour: silence beside a
// full tone comes out 7e-10 off in the logarithm with samples of up to 2^24, 7e-7 with up to
// 2^31, where a transform by itself gives the guard exactly.  (The features are rounded to fp32.)
// A pair never spans two utterances (a NaN would cross over); the last of an odd number of
// frames is transformed alone.  pair_start[u] = first pair of utterance u among
// all pairs.  Sample is double for a resampled signal, float where the input is framed as it is.
constexpr uint32_t kPairsPerWave = 4;  // (140 us for the 117 000 frames; 154 with eight, 171 with sixteen: a last round of waves)
template <typename Sample>
__global__ __launch_bounds__(kFrameThreads, 3) void log_mel_kernel(
    const Sample *__restrict__ mid, const Utterance *__restrict__ utt, const uint64_t *__restrict__ pair_start,
    int n_utt, uint64_t n_pairs, uint32_t per_wave, int hop, const double *__restrict__ window,
    const double2 *__restrict__ twiddle, const MelRange *__restrict__ ranges, int n_mels, float *__restrict__ out)
{
    __shared__ double2 s_x[kFrameThreads / 64][kFramePadded];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    uint64_t f = ((uint64_t)blockIdx.x * (kFrameThreads / 64) + (uint64_t)wave) * per_wave;
    const uint64_t f_end = min(f + per_wave, n_pairs);
    // the factors of the last two passes (there are 64 of the first of them), the window and the ranges
    __shared__ double2 s_factor[8 * 8];
    __shared__ double s_window[kFft];
    __shared__ MelRange s_range[kMaxMels + 1];
    static_assert(kFft == 2 * kFrameThreads && kMaxMels < kFrameThreads, "a lane copies two window values, and a range");
    double2 factor[8];
#pragma unroll
    for (int r = 1; r < 8; r++) factor[r] = twiddle[r * lane];
    // (asked for here, put into LDS when the samples have been asked for too)
    const double2 some_factor = twiddle[(lane >> 3) * (lane & 7) * (kFft / 64)];
    const double some_window[2] = {window[threadIdx.x], window[threadIdx.x + kFrameThreads]};
    const MelRange some_range = ranges[min((int)threadIdx.x, n_mels)];
    int lo = 0;
    if (f < f_end) {
        int hi = n_utt - 1;
        while (lo < hi) {
            const int m = (lo + hi + 1) >> 1;
            if (pair_start[m] <= f) lo = m; else hi = m - 1;
        }
    }
    double2 *x = s_x[wave];
    // The ranges widen with their number, so where there are more than 64 a lane takes a narrow one, `lane`,
    // and the wide one that mirrors it: every busy lane sums about the same number of bins.  (One range is
    // left over where there are more than 128.)  Up to 64 have a lane each, or, a power of two of them, several: one
    // channel, two ranges, 8 utterances of 5 s 60 -> 11 us.
    const int n_ranges = n_mels + 1, mirrored = n_ranges - 1 - lane;
    int log_parts = 0;
    while ((n_ranges << (log_parts + 1)) <= 64) log_parts++;
    // the samples of both frames of pair f: loaded while the pair before is summed, where both frames
    // lie inside the signal
    uint32_t t = 0, frames = 0;
    int64_t from = 0;
    bool inside = false;
    double ab[2][8];
    auto load = [&]() {
        while (lo + 1 < n_utt && pair_start[lo + 1] <= f) lo++;
        t = 2 * (uint32_t)(f - pair_start[lo]);
        frames = utt[lo].frames;
        from = (int64_t)t * hop - kFft / 2;
        inside = t + 1 < frames && from >= 0 && from + hop + kFft <= (int64_t)utt[lo].mid_len;
        if (inside) {
            const Sample *a = mid + utt[lo].mid_off + from, *b = a + hop;
#pragma unroll
            for (int r = 0; r < 8; r++) {
                ab[0][r] = (double)a[lane + 64 * r];
                ab[1][r] = (double)b[lane + 64 * r];
            }
        }
    };
    if (f < f_end) load();
    if (threadIdx.x < 64) s_factor[threadIdx.x] = some_factor;
    s_window[threadIdx.x] = some_window[0];
    s_window[threadIdx.x + kFrameThreads] = some_window[1];
    if ((int)threadIdx.x <= n_mels) s_range[threadIdx.x] = some_range;
    __syncthreads();
    if (f >= f_end) return;    // no workgroup-wide barrier below: a wave works on its own pairs
    for (;;) {
        const bool two = t + 1 < frames;
        if (!inside) {
            const Sample *sig = mid + utt[lo].mid_off;
            const int64_t len = (int64_t)utt[lo].mid_len;
            double *staged = reinterpret_cast<double *>(x);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll 1
            for (int k = lane; k < 2 * kFft; k += 64) {
                int64_t s = from + (k >= kFft && two ? hop : 0) + (k & (kFft - 1));
                if (s < 0) s = -s;                       // reflection about the first sample
                if (s >= len) s = 2 * (len - 1) - s;     // and about the last (len > n_fft / 2)
                staged[k] = (double)sig[s];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int r = 0; r < 8; r++) {
                ab[0][r] = staged[lane + 64 * r];
                ab[1][r] = staged[kFft + lane + 64 * r];
            }
        }
        double2 v[8];
#pragma unroll
        for (int r = 0; r < 8; r++) {
            const double win = s_window[lane + 64 * r];
            v[r] = make_double2(ab[0][r] * win, two ? ab[1][r] * win : 0.0);
        }
        dft8(v);
        // (the accesses of one wave to LDS complete in order; the fences keep the compiler from
        // moving loads over the stores)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int r = 0; r < 8; r++) x[padded(lane * 8 + r)] = v[r];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int pass = 1; pass < 3; pass++) {
            const int ns = pass == 1 ? 8 : 64;
            const int k = lane & (ns - 1);
#pragma unroll
            for (int r = 0; r < 8; r++) v[r] = x[padded(lane + 64 * r)];
#pragma unroll
            for (int r = 1; r < 8; r++) v[r] = cmul(v[r], pass == 1 ? s_factor[r * 8 + k] : factor[r]);
            dft8(v);
            if (pass == 1) {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                const int j0 = (lane >> 3) * 64 + k;
#pragma unroll
                for (int r = 0; r < 8; r++) x[padded(j0 + 8 * r)] = v[r];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
        }
        // After the last pass value r of lane j is Z[j + 64 r].  Z[512 - k] is value 7 - r of lane
        // 64 - j, in lane 0 its own value 8 - r.  The powers of both frames, bins 0 .. 256, replace
        // the values of the last pass in LDS (all lanes have read theirs: the fence).
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int r = 0; r < 4; r++) {
            double2 w = make_double2(__shfl(v[7 - r].x, (64 - lane) & 63), __shfl(v[7 - r].y, (64 - lane) & 63));
            if (lane == 0) w = v[(8 - r) & 7];
            const double ax = v[r].x + w.x, ay = v[r].y - w.y, bx = v[r].x - w.x, by = v[r].y + w.y;
            x[lane + 64 * r] = make_double2(0.25 * (ax * ax + ay * ay), 0.25 * (bx * bx + by * by));
        }
        // bin 256 is its own partner: both spectra are real there
        if (lane == 0) x[kFft / 2] = make_double2(v[4].x * v[4].x, v[4].y * v[4].y);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const bool more = f + 1 < f_end;
        const uint32_t stride = frames;
        float *o = out + utt[lo].out_off + t;
        f++;
        if (more) load();
        // the sums of the ranges, behind the powers, of both frames
        double2 *rising = x + kFft / 2 + 1, *falling = rising + kMaxMels + 1;
        static_assert(kFft / 2 + 1 + 2 * (kMaxMels + 1) <= kFramePadded, "the sums fit behind the powers");
        // part = [first, last) of range m's bins; a part's weights are not those that the host has looked at
        auto sum = [&](int m, auto part, int first, int last) {
            const MelRange range = s_range[m];
            double2 up = make_double2(0.0, 0.0), down = up;
            double wu = range.rising, wd = range.falling;
            if constexpr (part) {
                wu += first * range.step;
                wd -= first * range.step;
            } else {
                first = 0;
                last = range.count;
            }
            const double2 *pw = x + range.start;
            // four bins at a time, so that their loads are under way together
            for (int k = first; k < last; k += 4) {
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const double2 power = pw[min(k + e, last - 1)];
                    const double u = k + e < last ? wu : 0.0, d = k + e < last ? (part ? fmax(wd, 0.0) : wd) : 0.0;
                    up = make_double2(fma(u, power.x, up.x), fma(u, power.y, up.y));
                    down = make_double2(fma(d, power.x, down.x), fma(d, power.y, down.y));
                    wu += range.step;
                    wd -= range.step;
                }
            }
            if constexpr (part) {
                for (int i = 1; i < 1 << log_parts; i *= 2) {
                    up = cadd(up, make_double2(__shfl_xor(up.x, i), __shfl_xor(up.y, i)));
                    down = cadd(down, make_double2(__shfl_xor(down.x, i), __shfl_xor(down.y, i)));
                }
                if (lane & ((1 << log_parts) - 1)) return;
            }
            rising[m] = up;
            falling[m] = down;
        };
        if (n_ranges > 64) {
            if (lane <= mirrored) sum(lane, std::false_type(), 0, 0);
            if (lane < mirrored) sum(mirrored, std::false_type(), 0, 0);
            if (n_ranges > 128 && lane == 0) sum(64, std::false_type(), 0, 0);
        } else if (lane >> log_parts < n_ranges) {
            const int m = lane >> log_parts, count = s_range[m].count;
            const int each = (count + (1 << log_parts) - 1) >> log_parts, first = (lane & ((1 << log_parts) - 1)) * each;
            sum(m, std::true_type(), min(first, count), min(first + each, count));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const double *up = reinterpret_cast<const double *>(rising), *down = reinterpret_cast<const double *>(falling + 1);
        for (int i = lane; i < 2 * n_mels; i += 64) {   // i = 2 m + frame
            const float y = (float)log_of(up[i] + down[i] + (double)kLogGuard);
            if ((i & 1) == 0 || two) o[(uint64_t)(i >> 1) * stride + (i & 1)] = y;
        }
        if (!more) break;
    }
}

// ---- normalize ----------------------------------------------------------------------------
// One workgroup per (utterance, Mel channel) row: mean, then the mean squared deviation, then
// the normalised values, the row held in registers (up to kRowPerThread * 256 frames) or
// re-read from memory when longer.
constexpr int kRowPerThread = 16;

__device__ __forceinline__ double block_sum_256(double v, double *s)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    return s[0] + s[1] + s[2] + s[3];
}

__global__ __launch_bounds__(256) void normalize_kernel(const Utterance *__restrict__ utt, int n_mels, float *__restrict__ out)
{
    __shared__ double s[4];
    const Utterance u = utt[blockIdx.x / n_mels];
    float *row = out + u.out_off + (uint64_t)(blockIdx.x % n_mels) * u.frames;
    const uint32_t n = u.frames;
    const bool cached = n <= (uint32_t)kRowPerThread * 256u;
    float v[kRowPerThread];
    double sum = 0.0;
    if (cached) {
#pragma unroll
        for (int i = 0; i < kRowPerThread; i++) {
            const uint32_t k = threadIdx.x + 256u * i;
            v[i] = k < n ? row[k] : 0.0f;
            sum += v[i];
        }
    } else {
        for (uint32_t k = threadIdx.x; k < n; k += 256) sum += row[k];
    }
    const double mean = block_sum_256(sum, s) / (double)n;
    double dev = 0.0;
    if (cached) {
#pragma unroll
        for (int i = 0; i < kRowPerThread; i++) {
            const uint32_t k = threadIdx.x + 256u * i;
            const double d = (double)v[i] - mean;
            dev += k < n ? d * d : 0.0;
        }
    } else {
        for (uint32_t k = threadIdx.x; k < n; k += 256) { const double d = (double)row[k] - mean; dev += d * d; }
    }
    const double var = block_sum_256(dev, s) / (double)n;
    const double scale = 1.0 / (sqrt(var) + (double)kStdGuard);
    if (cached) {
#pragma unroll
        for (int i = 0; i < kRowPerThread; i++) {
            const uint32_t k = threadIdx.x + 256u * i;
            if (k < n) row[k] = (float)(((double)v[i] - mean) * scale);
        }
    } else {
        for (uint32_t k = threadIdx.x; k < n; k += 256) row[k] = (float)(((double)row[k] - mean) * scale);
    }
}

}  // namespace

struct prep_audio {
    prep_audio_config cfg;
    // tables on the device
    double *d_window = nullptr;
    double2 *d_twiddle = nullptr;
    MelRange *d_ranges = nullptr;
    // interpolation taps of the two rate pairs seen last, in buffers of the largest size a rate
    // pair can need (reserved in prep_audio_create: a call never allocates or frees): bands where the
    // plan has steps, else taps by phase
    struct TapSlot {
        int p = 0, q = 0, n_taps = 0;
        BandPlan plan = {};
        double *d_taps = nullptr;
        int32_t *d_first = nullptr;
        uint64_t used = 0;       // call counter when the slot served last
    } slot[2];
    double *h_taps_pinned = nullptr;   // staging of an upload, free again once `done` has passed
    int32_t *h_first_pinned = nullptr;
    uint64_t calls = 0;
    // per call
    // a call's n records, and behind them [mid_start n][pair_start n][tile_start n]: they go up in
    // one copy
    Utterance *h_utt = nullptr, *d_utt = nullptr;
    double *d_mid = nullptr;
    hipEvent_t done = nullptr;
    bool pending = false;
    std::vector<double> h_taps;
    std::vector<int32_t> h_first;
};

namespace {

#define AUDIO_TRY(expr)                                   \
    do {                                                  \
        if ((expr) != hipSuccess) {                       \
            (void)hipGetLastError();                      \
            return PREP_E_HIP;                            \
        }                                                 \
    } while (0)

}  // namespace

extern "C" {

int64_t prep_audio_frames(const prep_audio_config *cfg, uint64_t samples_in, int32_t rate_in)
{
    if (!cfg || rate_in < 1 || cfg->rate < 1 || cfg->hop < 1) return PREP_E_INVALID_ARG;
    const int g = std::gcd(rate_in, cfg->rate);
    const uint64_t len = resampled_length(samples_in, rate_in / g, cfg->rate / g);
    return (int64_t)(1 + len / (uint64_t)cfg->hop);
}

int prep_audio_create(prep_audio **out, const prep_audio_config *cfg)
{
    if (!out) return PREP_E_INVALID_ARG;
    *out = nullptr;
    if (!cfg || cfg->max_batch < 1 || cfg->rate < 1 || cfg->n_fft != kFft || cfg->win_length < 1 ||
        cfg->win_length > cfg->n_fft || cfg->hop < 1 || cfg->n_mels < 1 || cfg->n_mels > kMaxMels ||
        cfg->max_total_samples < 1)
        return PREP_E_INVALID_ARG;
    if (cfg->max_total_samples > kMaxSamples) return PREP_E_NOMEM;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || cfg->device < 0 || cfg->device >= ndev) {
        (void)hipGetLastError();
        return PREP_E_HIP;
    }
    prep_audio *h = new (std::nothrow) prep_audio;
    if (!h) return PREP_E_NOMEM;
    h->cfg = *cfg;
    // window, twiddle factors, Mel triangles: double precision, rounded once
    std::vector<double> window((size_t)kFft, 0.0);
    const int left = (kFft - cfg->win_length) / 2;
    for (int i = 0; i < cfg->win_length; i++)
        window[(size_t)(left + i)] = 0.5 - 0.5 * cos(2.0 * M_PI * i / cfg->win_length);
    std::vector<double2> tw((size_t)kFft);  // W^k = exp(-2 pi i k / 512), k = 0 .. 511 (r k reaches 7 * 63)
    for (int k = 0; k < kFft; k++)
        tw[(size_t)k] = make_double2(cos(2.0 * M_PI * k / kFft), -sin(2.0 * M_PI * k / kFft));
    std::vector<MelRange> ranges((size_t)cfg->n_mels + 1);
    {
        auto mel_of = [](double f) { return 2595.0 * log10(1.0 + f / 700.0); };
        auto hz_of = [](double m) { return 700.0 * (pow(10.0, m / 2595.0) - 1.0); };
        const double top = mel_of(cfg->rate / 2.0);
        std::vector<double> corner((size_t)cfg->n_mels + 2);
        for (int i = 0; i < cfg->n_mels + 2; i++) corner[(size_t)i] = hz_of(top * i / (cfg->n_mels + 1));
        // range i = the bins from corner i up to corner i + 1 (bin 0 lies on a corner, with no weight)
        int k = 1;
        for (int i = 0; i <= cfg->n_mels; i++) {
            const double lo = corner[(size_t)i], hi = corner[(size_t)i + 1], width = (double)cfg->rate / kFft;
            MelRange &range = ranges[(size_t)i];
            range.start = k;
            range.rising = (k * width - lo) / (hi - lo);
            range.falling = (hi - k * width) / (hi - lo);
            range.step = width / (hi - lo);
            while (k <= kFft / 2 && k * width < hi) k++;
            range.count = k - range.start;
            // the falling weights, one after the other as the kernel forms them, stay above zero
            auto last = [&]() {
                double w = range.falling;
                for (int b = 1; b < range.count; b++) w -= range.step;
                return w;
            };
            while (range.count > 0 && last() < 0.0) range.falling = nextafter(range.falling, 2.0);
        }
    }
    const size_t n = (size_t)cfg->max_batch;
    bool ok = hipSetDevice(cfg->device) == hipSuccess;
    ok = ok && hipMalloc((void **)&h->d_window, sizeof(double) * kFft) == hipSuccess;
    ok = ok && hipMalloc((void **)&h->d_twiddle, sizeof(double2) * kFft) == hipSuccess;
    ok = ok && hipMalloc((void **)&h->d_ranges, sizeof(MelRange) * ranges.size()) == hipSuccess;
    ok = ok && hipMalloc((void **)&h->d_utt, kRecordBytes * n) == hipSuccess;
    ok = ok && hipHostMalloc((void **)&h->h_utt, kRecordBytes * n, hipHostMallocDefault) == hipSuccess;
    // the resampled signal is never longer than max_total_samples scaled by the largest ratio accepted
    ok = ok && hipMalloc((void **)&h->d_mid, sizeof(double) * (cfg->max_total_samples + n)) == hipSuccess;
    for (auto &ts : h->slot) {
        ok = ok && hipMalloc((void **)&ts.d_taps, sizeof(double) * kMaxTapEntries) == hipSuccess;
        ok = ok && hipMalloc((void **)&ts.d_first, sizeof(int32_t) * kMaxRateTerm) == hipSuccess;
    }
    ok = ok && hipHostMalloc((void **)&h->h_taps_pinned, sizeof(double) * kMaxTapEntries, hipHostMallocDefault) == hipSuccess;
    ok = ok && hipHostMalloc((void **)&h->h_first_pinned, sizeof(int32_t) * kMaxRateTerm, hipHostMallocDefault) == hipSuccess;
    ok = ok && hipEventCreateWithFlags(&h->done, hipEventDisableTiming) == hipSuccess;
    ok = ok && hipMemcpy(h->d_window, window.data(), sizeof(double) * kFft, hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipMemcpy(h->d_twiddle, tw.data(), sizeof(double2) * kFft, hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipMemcpy(h->d_ranges, ranges.data(), sizeof(MelRange) * ranges.size(), hipMemcpyHostToDevice) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        prep_audio_destroy(h);
        return PREP_E_NOMEM;
    }
    *out = h;
    return PREP_OK;
}

int prep_audio_destroy(prep_audio *h)
{
    if (!h) return PREP_E_INVALID_ARG;
    (void)hipSetDevice(h->cfg.device);
    if (h->pending) (void)hipEventSynchronize(h->done);
    (void)hipFree(h->d_window);
    (void)hipFree(h->d_twiddle);
    (void)hipFree(h->d_ranges);
    (void)hipFree(h->d_utt);
    (void)hipFree(h->d_mid);
    for (auto &ts : h->slot) {
        (void)hipFree(ts.d_taps);
        (void)hipFree(ts.d_first);
    }
    if (h->h_taps_pinned) (void)hipHostFree(h->h_taps_pinned);
    if (h->h_first_pinned) (void)hipHostFree(h->h_first_pinned);
    if (h->h_utt) (void)hipHostFree(h->h_utt);
    if (h->done) (void)hipEventDestroy(h->done);
    delete h;
    return PREP_OK;
}

int prep_audio_features(prep_audio *h, const float *waveforms, const uint64_t *offsets, int32_t n, int32_t rate_in,
                        float *out, uint64_t *out_offsets, void *stream_ptr)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    if (!h || !waveforms || !offsets || !out || !out_offsets || n < 0 || rate_in < 1) return PREP_E_INVALID_ARG;
    if (n > h->cfg.max_batch) return PREP_E_TOO_LARGE;
    out_offsets[0] = 0;
    if (n == 0) return PREP_OK;
    const int g = std::gcd(rate_in, h->cfg.rate);
    const int p = rate_in / g, q = h->cfg.rate / g;
    if (p > kMaxRateTerm || q > kMaxRateTerm) return PREP_E_INVALID_ARG;  // the tap table has q rows
    AUDIO_TRY(hipSetDevice(h->cfg.device));
    if (h->pending) {  // the pinned records of the call before are still being read
        AUDIO_TRY(hipEventSynchronize(h->done));
        h->pending = false;
    }
    uint64_t *h_starts = reinterpret_cast<uint64_t *>(h->h_utt + n);
    const uint64_t *d_starts = reinterpret_cast<const uint64_t *>(h->d_utt + n);
    uint64_t mid_total = 0, pairs_total = 0, out_total = 0, tiles_total = 0;
    for (int32_t i = 0; i < n; i++) {
        if (offsets[i + 1] < offsets[i] || offsets[i + 1] - offsets[i] > 0xFFFFFFFFull) return PREP_E_INVALID_ARG;
        Utterance &u = h->h_utt[i];
        u.in_off = offsets[i];
        u.in_len = (uint32_t)(offsets[i + 1] - offsets[i]);
        const uint64_t len = resampled_length(u.in_len, p, q);
        // centring reflects n_fft / 2 samples at both ends
        if (len <= (uint64_t)kFft / 2 || len > 0x7FFFFFFFull) return PREP_E_INVALID_ARG;
        u.mid_len = (uint32_t)len;
        u.frames = (uint32_t)(1 + len / (uint64_t)h->cfg.hop);
        u.mid_off = mid_total;
        u.out_off = out_total;
        u.pad_ = 0;
        h_starts[i] = mid_total;
        h_starts[(size_t)n + i] = pairs_total;
        mid_total += len;
        pairs_total += (u.frames + 1) / 2;
        out_total += (uint64_t)u.frames * (uint64_t)h->cfg.n_mels;
        out_offsets[i + 1] = out_total;
    }
    if (offsets[n] - offsets[0] > h->cfg.max_total_samples || mid_total > h->cfg.max_total_samples + (uint64_t)n)
        return PREP_E_TOO_LARGE;
    prep_audio::TapSlot *taps = &h->slot[0];
    if (p != q) {
        h->calls++;
        if (!(taps->p == p && taps->q == q)) {
            if (h->slot[1].p == p && h->slot[1].q == q) {
                taps = &h->slot[1];
            } else {
                // a new rate pair: build its taps into the slot that served longest ago and upload
                // them on the caller's stream, ahead of the kernels that read them (the pinned
                // staging is free: the call before has been waited for above; so is the slot)
                if (h->slot[1].used < taps->used) taps = &h->slot[1];
                taps->p = taps->q = 0;
                make_taps(p, q, &h->h_taps, &h->h_first, &taps->n_taps);
                make_bands(p, q, taps->n_taps, &h->h_taps, &h->h_first, &taps->plan);
                if (h->h_taps.size() > kMaxTapEntries) return PREP_E_TOO_LARGE;
                memcpy(h->h_taps_pinned, h->h_taps.data(), sizeof(double) * h->h_taps.size());
                memcpy(h->h_first_pinned, h->h_first.data(), sizeof(int32_t) * h->h_first.size());
                AUDIO_TRY(hipMemcpyAsync(taps->d_taps, h->h_taps_pinned, sizeof(double) * h->h_taps.size(),
                                         hipMemcpyHostToDevice, stream));
                AUDIO_TRY(hipMemcpyAsync(taps->d_first, h->h_first_pinned, sizeof(int32_t) * h->h_first.size(),
                                         hipMemcpyHostToDevice, stream));
                taps->p = p;
                taps->q = q;
            }
        }
        taps->used = h->calls;
    }
    if (p != q && taps->plan.quads) {
        const uint64_t per_tile = 16ull * (uint64_t)taps->plan.Q;
        for (int32_t i = 0; i < n; i++) {
            h_starts[2 * (size_t)n + i] = tiles_total;
            tiles_total += (h->h_utt[i].mid_len + per_tile - 1) / per_tile;
        }
    }
    if (p == q) {
        // same rate: the frames read the input itself; utterance offsets are the input's
        for (int32_t i = 0; i < n; i++) h->h_utt[i].mid_off = h->h_utt[i].in_off;
    }
    AUDIO_TRY(hipMemcpyAsync(h->d_utt, h->h_utt, kRecordBytes * (size_t)n, hipMemcpyHostToDevice, stream));
    if (p != q && taps->plan.quads) {
        // (a slot with a plan holds its taps in that form only, so there is no other way for it)
        const BandPlan &plan = taps->plan;
        // as many waves as the chip holds, or as there are tiles' blocks, but one for each block at least
        const uint64_t unit = kXcds * kBandWaves, wanted = (tiles_total * (uint64_t)plan.blocks + unit - 1) / unit * unit;
        const uint64_t waves = std::max(std::min<uint64_t>(wanted, 256 * 16), ((uint64_t)plan.blocks + unit - 1) / unit * unit);
        const dim3 grid((unsigned)(waves / kBandWaves));
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(64 * kBandWaves), 0, stream, waveforms, h->d_utt, d_starts + 2 * n, n,
                               (uint32_t)tiles_total, taps->d_taps, taps->d_first, plan, h->d_mid);
        };
        switch (plan.quads) {
        case 2: launch(resample_bands_kernel<2>); break;
        case 3: launch(resample_bands_kernel<3>); break;
        case 4: launch(resample_bands_kernel<4>); break;
        case 5: launch(resample_bands_kernel<5>); break;
        default: launch(resample_bands_kernel<kBandQuadsMost>); break;
        }
    } else if (p != q) {
        hipLaunchKernelGGL(resample_kernel, dim3((unsigned)((mid_total + 255) / 256)), dim3(256), 0, stream, waveforms,
                           h->d_utt, d_starts, n, taps->d_taps, taps->d_first, p, q, taps->n_taps, h->d_mid, mid_total);
    }
    // (from sixteen waves a compute unit on, a wave takes more pairs than one)
    const uint32_t per_wave = (uint32_t)std::min<uint64_t>(kPairsPerWave, std::max<uint64_t>(1, pairs_total / (256 * 16)));
    const uint64_t per_wg = (uint64_t)per_wave * (kFrameThreads / 64);
    const dim3 pair_grid((unsigned)((pairs_total + per_wg - 1) / per_wg));
    if (p == q)
        hipLaunchKernelGGL(log_mel_kernel<float>, pair_grid, dim3(kFrameThreads), 0, stream, waveforms, h->d_utt,
                           d_starts + n, n, pairs_total, per_wave, h->cfg.hop, h->d_window, h->d_twiddle,
                           h->d_ranges, h->cfg.n_mels, out);
    else
        hipLaunchKernelGGL(log_mel_kernel<double>, pair_grid, dim3(kFrameThreads), 0, stream, (const double *)h->d_mid,
                           h->d_utt, d_starts + n, n, pairs_total, per_wave, h->cfg.hop, h->d_window, h->d_twiddle,
                           h->d_ranges, h->cfg.n_mels, out);
    hipLaunchKernelGGL(normalize_kernel, dim3((unsigned)n * (unsigned)h->cfg.n_mels), dim3(256), 0, stream, h->d_utt,
                       h->cfg.n_mels, out);
    AUDIO_TRY(hipGetLastError());
    AUDIO_TRY(hipEventRecord(h->done, stream));
    h->pending = true;
    return PREP_OK;
}

}  // extern "C"
