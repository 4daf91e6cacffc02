"""Parity of the GPU audio path (prep_audio_*, through the C ABI) with the numpy oracle:
normalised log-Mel features within FEATURE_TOL.  The kernels compute in double from the float32
samples to the logarithm and store float32 features: what remains is the rounding of a
log-Mel value of magnitude up to about 20 to float32 (1e-6) divided by a standard deviation
of order one, and the order of summation."""
import numpy as np
import pytest

from oracle import audio

pytestmark = pytest.mark.gpu

FEATURE_TOL = 2e-5


def speech_like(seed, rate, seconds):
    """Seeded stand-in for an utterance: a few drifting harmonics under a slow envelope plus
    low-pass noise, peak about 0.5."""
    rng = np.random.default_rng(seed)
    n = int(rate * seconds)
    t = np.arange(n) / rate
    f0 = 110.0 + 60.0 * rng.random() + 20.0 * np.sin(2 * np.pi * (0.7 + rng.random()) * t)
    phase = 2 * np.pi * np.cumsum(f0) / rate
    x = sum(rng.random() / (h ** 0.8) * np.sin(h * phase + rng.random() * 6.28) for h in range(1, 24))
    envelope = 0.55 + 0.45 * np.sin(2 * np.pi * 3.1 * t + rng.random() * 6.28)
    noise = np.convolve(rng.standard_normal(n + 15), np.hanning(16) / 8.0, mode="valid")
    x = x * envelope + 0.6 * noise
    return (0.5 * x / np.abs(x).max()).astype(np.float32)


@pytest.fixture(scope="module")
def prep():
    import paper_2411_19114_amd as p
    return p


def run(ap, waves, rate_in):
    import torch
    offsets = np.zeros(len(waves) + 1, dtype=np.uint64)
    np.cumsum([len(w) for w in waves], out=offsets[1:])
    dev = torch.from_numpy(np.concatenate(waves)).to("cuda:0")
    total = sum(ap.cfg.n_mels * ap.frames(len(w), rate_in) for w in waves)
    out = torch.full((total,), 777.0, dtype=torch.float32, device="cuda:0")
    oo = ap.features(dev.data_ptr(), offsets, rate_in, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    flat = out.cpu().numpy()
    assert int(oo[-1]) == total
    return [flat[int(oo[i]):int(oo[i + 1])].reshape(ap.cfg.n_mels, -1) for i in range(len(waves))]


@pytest.mark.parametrize("rate_in", [44100, 48000, 22050, 16000, 8000])
def test_features_match_the_oracle(prep, rate_in):
    waves = [speech_like(10 * rate_in % 997 + k, rate_in, sec) for k, sec in enumerate((0.9, 2.3, 1.0, 0.35, 3.1))]
    ap = prep.AudioPreprocessor(max_batch=8, max_total_samples=sum(len(w) for w in waves) * 3)
    try:
        got = run(ap, waves, rate_in)
        for w, g in zip(waves, got):
            ref = audio.preprocess(w.astype(np.float64), rate_in)
            assert g.shape == ref.shape
            assert np.isfinite(g).all()
            assert np.abs(g - ref).max() <= FEATURE_TOL
        # a second call on the same handle, other lengths, same rate pair
        again = run(ap, waves[::-1][:3], rate_in)
        for g, h in zip(again, got[::-1][:3]):
            assert np.array_equal(g, h)
    finally:
        ap.close()


def test_other_frame_parameters_and_many_short_utterances(prep):
    rate_in = 32000
    waves = [speech_like(300 + k, rate_in, 0.05 + 0.03 * k) for k in range(24)]
    ap = prep.AudioPreprocessor(max_batch=32, max_total_samples=400000, rate=16000, win_length=512, hop=128, n_mels=64)
    try:
        for w, g in zip(waves, run(ap, waves, rate_in)):
            ref = audio.preprocess(w.astype(np.float64), rate_in, rate=16000, win_length=512, hop=128, n_mels=64)
            assert g.shape == ref.shape and np.abs(g - ref).max() <= FEATURE_TOL
    finally:
        ap.close()


def test_long_utterance_rows_longer_than_the_register_cache(prep):
    rate = 16000
    w = speech_like(7, rate, 45.0)               # 4501 frames > 4096
    ap = prep.AudioPreprocessor(max_batch=1, max_total_samples=len(w))
    try:
        g, = run(ap, [w], rate)
        ref = audio.preprocess(w.astype(np.float64), rate)
        assert g.shape == ref.shape == (80, 4501)
        assert np.abs(g - ref).max() <= FEATURE_TOL
    finally:
        ap.close()


def test_argument_errors(prep):
    import torch
    ap = prep.AudioPreprocessor(max_batch=2, max_total_samples=20000)
    try:
        x = torch.zeros(20000, device="cuda:0")
        out = torch.zeros(80 * 200, device="cuda:0")
        ok = np.array([0, 4000, 8000], dtype=np.uint64)
        ap.features(x.data_ptr(), ok, 16000, out.data_ptr())
        torch.cuda.synchronize()
        with pytest.raises(prep.PrepError):      # an utterance of 200 samples cannot be centred
            ap.features(x.data_ptr(), np.array([0, 200], dtype=np.uint64), 16000, out.data_ptr())
        with pytest.raises(prep.PrepError):      # three utterances, max_batch two
            ap.features(x.data_ptr(), np.array([0, 3000, 6000, 9000], dtype=np.uint64), 16000, out.data_ptr())
        with pytest.raises(prep.PrepError):      # more samples than reserved
            ap.features(x.data_ptr(), np.array([0, 30000], dtype=np.uint64), 16000, out.data_ptr())
    finally:
        ap.close()
    with pytest.raises(prep.PrepError):
        prep.AudioPreprocessor(max_batch=1, max_total_samples=1000, n_fft=1024)
    # more than the device holds, and more than the sizes in bytes hold
    for samples in (1 << 37, 1 << 61, (1 << 64) - 1):
        with pytest.raises(prep.PrepError) as e:
            prep.AudioPreprocessor(max_batch=1, max_total_samples=samples)
        assert e.value.code == prep.E_NOMEM


def test_frames_in_pairs(prep):
    """Two frames share a transform: odd and even counts of frames (from two on: the shortest signal
    that can be reflected holds 257 samples), a frame of silence beside loud ones, and a NaN that
    stays in its own utterance."""
    rate = 16000
    waves = [speech_like(700 + k, rate, 1.0)[:n] for k, n in enumerate((257, 319, 320, 479, 480, 481, 4000, 4160))]
    waves.append(np.concatenate([waves[-1], np.zeros(1600, np.float32), waves[-1]]))
    bad = waves[3].copy()
    bad[100] = np.nan
    ap = prep.AudioPreprocessor(max_batch=16, max_total_samples=sum(len(w) for w in waves) * 3)
    try:
        plain = run(ap, waves, rate)
        for w, g in zip(waves, plain):
            ref = audio.preprocess(w.astype(np.float64), rate)
            assert g.shape == ref.shape and np.abs(g - ref).max() <= FEATURE_TOL
        got = run(ap, waves[:3] + [bad] + waves[4:], rate)
        assert np.isnan(got[3]).any()
        for i in range(len(waves)):
            assert i == 3 or np.array_equal(got[i], plain[i])
    finally:
        ap.close()


# rate pairs that take the matrix form: 441 : 160, 3 : 1, 441 : 640, 3 : 2, 441 : 400, 25 : 8, 4 : 5, 1601 : 1600; and those
# that take a lane per output: 6 : 1 and 441 : 80 (the band is too long), 3201 : 3200 (the table is too large)
# (tests/test_audio_plan.py holds both lists to it)
MATRIX_RATES = [44100, 48000, 11025, 24000, 17640, 50000, 12800, 16010]
PHASE_RATES = [96000, 88200, 16005]


@pytest.mark.parametrize("rate_in", MATRIX_RATES + PHASE_RATES)
def test_resampled_lengths_at_the_edges_of_chunks(prep, rate_in):
    """Utterances of one sample more or less than whole periods and tiles, one that fills none,
    and one of NaNs beside them, which must not reach its neighbours.  (No shorter ones: the bound
    above is for deviations of order one.  The two frames of an utterance of 300 samples differ by 0.02
    in some channels, which makes 1e-4 of a log-Mel value's rounding.)"""
    import math
    g = math.gcd(rate_in, 16000)
    p, q = rate_in // g, 16000 // g
    period = q if q >= 100 else math.lcm(q, 16)              # outputs of a row of a tile
    lengths = [n * p // q for n in (1500, 16 * period, 128 * period) if 1500 <= n and n * p // q < 120000]
    waves = [speech_like(900 + k, rate_in, 8.0)[:n + d] for k, n in enumerate(lengths) for d in (-1, 0, 1)]
    bad = np.full(len(waves[1]), np.nan, np.float32)
    ap = prep.AudioPreprocessor(max_batch=16, max_total_samples=sum(len(w) for w in waves) * 3)
    try:
        plain = run(ap, waves, rate_in)
        for w, f in zip(waves, plain):
            ref = audio.preprocess(w.astype(np.float64), rate_in)
            assert f.shape == ref.shape and np.abs(f - ref).max() <= FEATURE_TOL
        got = run(ap, waves[:1] + [bad] + waves[2:], rate_in)
        assert np.isnan(got[1]).any()
        for i in range(len(waves)):
            assert i == 1 or np.array_equal(got[i], plain[i])
    finally:
        ap.close()


@pytest.mark.parametrize("rate_in,bad", [(44100, np.nan), (48000, np.inf), (24000, -np.inf), (11025, np.nan)])
def test_bad_samples_between_frames(prep, rate_in, bad):
    """Samples that are no finite numbers reach the outputs whose own taps hold them, not the others of their band:
    with frames of 512 samples every 1024, those in the middle of a gap reach no frame, and all features are the
    oracle's.  One stands just so far from a frame that the taps of the nearest output inside end before it."""
    rate, hop = 16000, 1024
    good = speech_like(5, rate_in, 3.0)
    reach = int(np.ceil(6 / 0.99 * max(rate_in, rate) / rate)) + 1             # samples on either side that an output reads
    bad_at = [int(round((hop * k + 512) * rate_in / rate)) for k in (1, 7, 20)]     # the middles of gaps
    bad_at += [int(np.ceil((hop * k + 256) * rate_in / rate)) + reach for k in (3, 11)]    # just behind a frame
    bad_at += [int((hop * k - 257) * rate_in / rate) - reach for k in (5, 13)]             # just before one
    w = good.copy()
    w[bad_at] = bad
    ap = prep.AudioPreprocessor(max_batch=2, max_total_samples=4 * len(w), hop=hop)
    try:
        clean, got = run(ap, [good], rate_in)[0], run(ap, [w], rate_in)[0]
        ref = audio.preprocess(good.astype(np.float64), rate_in, hop=hop)
        assert clean.shape == ref.shape and np.abs(clean - ref).max() <= FEATURE_TOL
        assert np.isfinite(got).all() and np.abs(got - ref).max() <= FEATURE_TOL
    finally:
        ap.close()


@pytest.mark.parametrize("n_mels", [1, 2, 63, 64, 127, 128])
def test_numbers_of_triangles(prep, n_mels):
    # one range more than triangles: an even or odd number of them, and one more than two a lane
    rate = 16000
    w = speech_like(40 + n_mels, rate, 1.3)
    ap = prep.AudioPreprocessor(max_batch=1, max_total_samples=len(w), n_mels=n_mels)
    try:
        g, = run(ap, [w], rate)
        ref = audio.preprocess(w.astype(np.float64), rate, n_mels=n_mels)
        assert g.shape == ref.shape and np.abs(g - ref).max() <= FEATURE_TOL
    finally:
        ap.close()


# the last number of triangles, and the first, whose ranges have 2^k lanes each; and as many ranges as lanes
@pytest.mark.parametrize("n_mels", [3, 4, 7, 8, 15, 16, 31, 32, 62])
def test_ranges_of_several_lanes(prep, n_mels):
    """Two utterances, one of an odd number of frames; a full tone and silence in the other, where a weight
    that rounded below zero would show."""
    rate = 16000
    t = np.arange(rate) / rate
    loud = np.concatenate([np.zeros(4000), 1e9 * np.sin(2 * np.pi * 3000.0 * t), np.zeros(4000)]).astype(np.float32)
    waves = [speech_like(60 + n_mels, rate, 0.9)[:160 * 80 + 11], loud]
    ap = prep.AudioPreprocessor(max_batch=2, max_total_samples=sum(map(len, waves)), n_mels=n_mels)
    try:
        got = run(ap, waves, rate)
        ref = audio.preprocess(waves[0].astype(np.float64), rate, n_mels=n_mels)
        assert got[0].shape == ref.shape and np.abs(got[0] - ref).max() <= FEATURE_TOL
        ref = audio.preprocess(waves[1].astype(np.float64), rate, n_mels=n_mels)
        assert np.isfinite(got[1]).all() and np.abs(got[1] - ref).max() <= FEATURE_TOL
    finally:
        ap.close()


def test_waves_that_take_several_pairs(prep):
    """From 8192 pairs of frames on a wave takes more than one, across the utterances' borders: the
    features are those of the utterances by themselves, bit for bit."""
    rate = 16000
    waves = [speech_like(500 + k % 7, rate, 4.2)[:60000 + 1111 * (k % 7)] for k in range(48)]
    ap = prep.AudioPreprocessor(max_batch=48, max_total_samples=sum(map(len, waves)))
    try:
        assert sum((1 + len(w) // 160 + 1) // 2 for w in waves) >= 8192
        alone = [run(ap, [w], rate)[0] for w in waves[:7]]
        for k, g in enumerate(run(ap, waves, rate)):
            assert np.array_equal(g, alone[k % 7])
    finally:
        ap.close()
