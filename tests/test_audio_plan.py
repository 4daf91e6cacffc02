"""The resampler's host tables without a GPU: which rate pairs take the matrix form, and that its bands hold
every tap of every phase where the product finds it, and zeros elsewhere."""
import math
import os
import subprocess

import pytest

import test_gpu_audio

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_19114_amd", "csrc")

SOURCE = r'''
#include "audio_plan.h"
#include <stdio.h>
#include <stdlib.h>
using namespace prep;
// 0: no plan; 1: a plan whose bands are the taps; 2: one whose are not
static int check(int p, int q)
{
    std::vector<double> taps, bands;
    std::vector<int32_t> first, starts;
    int n_taps = 0;
    make_taps(p, q, &taps, &first, &n_taps);
    if (taps.size() > kMaxTapEntries || first.size() > (size_t)kMaxRateTerm) return 2;
    bands = taps;
    starts = first;
    BandPlan t;
    make_bands(p, q, n_taps, &bands, &starts, &t);
    if (t.quads == 0) return bands == taps && starts == first ? 0 : 2;
    if (t.quads < 2 || t.quads > kBandQuadsMost || t.P % p != 0 || t.Q != t.P / p * q || t.blocks != (t.Q + 15) / 16) return 2;
    if (bands.size() != (size_t)t.blocks * t.quads * 256 || bands.size() > kMaxTapEntries) return 2;
    if (starts.size() != (size_t)t.blocks || starts.size() > (size_t)kMaxRateTerm) return 2;
    for (int b = 0; b < t.blocks; b++)
        for (int j = 0; j < 16; j++) {
            const int r = 16 * b + j;                       // phase of the period
            for (int n = 0; n < 16 * t.quads; n++) {        // sample of the band
                const int k = starts[b] + n - (r < t.Q ? first[r % q] + r / q * p : 0);
                const double want = r < t.Q && k >= 0 && k < n_taps ? taps[(size_t)k * q + r % q] : 0.0;
                if (bands[band_entry(t.quads, b, n, j)] != want) return 2;
            }
            // no tap lies before the band or behind it
            if (r < t.Q && (first[r % q] + r / q * p < starts[b] || first[r % q] + r / q * p + n_taps > starts[b] + 16 * t.quads)) return 2;
        }
    return 1;
}
int main(int argc, char **argv)
{
    for (int i = 1; i + 1 < argc; i += 2) printf("%d\n", check(atoi(argv[i]), atoi(argv[i + 1])));
}
'''


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "check.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-I", CSRC,
                    str(d / "check.cpp"), "-o", str(d / "check")], check=True)

    def run(pairs):
        args = [str(x) for pair in pairs for x in pair]
        return [int(x) for x in subprocess.run([str(d / "check")] + args, check=True, capture_output=True, text=True).stdout.split()]
    return run


def _pair(rate_in, rate=16000):
    g = math.gcd(rate_in, rate)
    return rate_in // g, rate // g


def test_rates_of_the_gpu_tests_take_the_form_they_name(forms):
    assert set(forms([_pair(r) for r in test_gpu_audio.MATRIX_RATES])) == {1}
    assert set(forms([_pair(r) for r in test_gpu_audio.PHASE_RATES])) == {0}


def test_bands_hold_the_taps(forms):
    pairs = [(p, q) for p in range(1, 49) for q in range(1, 49) if p != q and math.gcd(p, q) == 1]
    pairs += [(441, 160), (160, 441), (441, 320), (147, 80), (4096, 4095), (4095, 4096), (1, 4096), (4096, 1), (2049, 2048),
              (2047, 2048), (2001, 4000), (3201, 3200), (4000, 1201), (1601, 1600), (4096, 1205)]
    got = forms(pairs)
    assert 2 not in got
    assert {p > 4 * q for (p, q), f in zip(pairs, got) if f} == {False}    # a band of 96 samples at most
    assert {f for (p, q), f in zip(pairs, got) if p <= 3 * q and q <= 1600} == {1}
