"""Streams without restart markers, cut into windows that are decoded side by side: coefficients,
pixels and tensors against the oracle where the windows and their rows can go wrong."""
import numpy as np
import pytest

import oracle
import synth
from helpers import WINDOW_BASES, check_against_oracle, check_damaged, damaged_streams, run_gpu
from oracle import MODE_420, MODE_422, MODE_440, MODE_444, MODE_GRAY
from paper_2411_19114_amd import STREAM_UNJOINED, STREAM_WHOLE, STREAM_WINDOWS

pytestmark = pytest.mark.gpu
MODES = [MODE_444, MODE_420, MODE_GRAY, MODE_422, MODE_440]


@pytest.fixture(scope="module")
def pp():
    import paper_2411_19114_amd as prep
    h = prep.Preprocessor(device=0, max_batch=48, max_width=1024, max_height=1024, max_bitstream_bytes=24 << 20,
                          flags=prep.FLAG_FULL_RGB)
    yield h
    h.close()


def _decoded(pp, n):
    """How the last call decoded its n streams, without repetitions."""
    return {pp.debug_last_stream(i) for i in range(n)}


def _file(seed, w, h, quality, mode, sigma=12.0, table_mode=0):
    rgb = synth.gradient_noise_image(np.random.default_rng(seed), w, h, sigma)
    return oracle.encode(rgb, quality, mode, 0, table_mode=table_mode)[0]


@pytest.mark.parametrize("mode", MODES)
def test_one_window_to_many_with_short_rows(pp, mode):
    # 30 bytes to 60 KB of data each: no full row, a window's edge, an overlap that the data end in
    files = [_file(10 * mode + k, w, h, q, mode, sigma=6.0, table_mode=k % 2)
             for k, (w, h, q) in enumerate([(8, 8, 50), (33, 17, 60), (64, 64, 75), (96, 80, 85), (131, 117, 90),
                                            (200, 160, 92), (255, 199, 50), (640, 480, 90)])]
    assert sum(map(len, files)) < 1 << 20
    check_against_oracle(pp, files, 0, 1, 1, "f32")
    assert _decoded(pp, len(files)) == {STREAM_WINDOWS}


@pytest.mark.parametrize("mode", MODES)
def test_many_windows_with_long_rows(pp, mode):
    # more than 1 MiB of data in the call
    files = [_file(20 * mode + k, 1000, 900, 94, mode, sigma=7.0) for k in range(2)]
    files += [_file(20 * mode + 9 + k, 40 + 37 * k, 300 - 23 * k, 60 + 4 * k, mode) for k in range(8)]
    while sum(map(len, files)) < (1 << 20) + 4096:
        files.append(files[0])
    check_against_oracle(pp, files, 0, 1, 1, "f32")
    assert _decoded(pp, len(files)) == {STREAM_WINDOWS}


@pytest.mark.parametrize("sigma,table_mode", [(9.0, 0), (9.0, 1), (30.0, 0)])
@pytest.mark.parametrize("mode", MODES)
def test_dense_streams(pp, mode, sigma, table_mode):
    # noise near the densities up to which streams are cut, where most rows need extra nodes, and
    # far beyond, where one workgroup takes each
    files = [_file(30 * mode + k, 200 + 40 * k, 160, 95, mode, sigma, table_mode) for k in range(4)]
    check_against_oracle(pp, files, 0, 1, 1, "f32")
    assert _decoded(pp, len(files)) <= ({STREAM_WHOLE} if sigma > 20 else {STREAM_WHOLE, STREAM_WINDOWS})


def test_an_image_of_many_chain_tiles():
    # 2400 x 2000: more than 128 windows several times over, and a tile that is not full
    import paper_2411_19114_amd as prep
    f = _file(40, 2400, 2000, 92, MODE_420, sigma=7.0)
    assert len(f) > 3 * 128 * 2584
    with_one = prep.Preprocessor(device=0, max_batch=1, max_width=2400, max_height=2000, max_bitstream_bytes=len(f))
    try:
        check_against_oracle(with_one, [f], 0, 64, 64, "f32")
        assert _decoded(with_one, 1) == {STREAM_WINDOWS}
    finally:
        with_one.close()


@pytest.mark.parametrize("mode,n,w,h,quality,how", [
    (MODE_GRAY, 191, 40, 40, 80, STREAM_WINDOWS), (MODE_GRAY, 192, 40, 40, 80, STREAM_WHOLE),
    (MODE_444, 192, 40, 40, 80, STREAM_WHOLE), (MODE_422, 383, 80, 80, 80, STREAM_WINDOWS),
    (MODE_440, 384, 80, 80, 80, STREAM_WHOLE), (MODE_420, 256, 96, 80, 85, STREAM_WINDOWS),
    (MODE_420, 256, 16, 16, 60, STREAM_WHOLE), (MODE_GRAY, 192, 256, 224, 92, STREAM_WINDOWS)])
def test_batches_on_either_side_of_the_rules(mode, n, w, h, quality, how):
    # many streams of one chunk take a workgroup each; from one chunk (the last case) on they do not
    import paper_2411_19114_amd as prep
    files = [_file(50 + k, w - k % 3, h, quality, mode) for k in range(16)]
    files = (files * (n // 16 + 1))[:n]
    many = prep.Preprocessor(device=0, max_batch=n, max_width=w, max_height=h, max_bitstream_bytes=sum(map(len, files)))
    try:
        check_against_oracle(many, files, 0, 1, 1, "f16")
        assert _decoded(many, n) == {how}
    finally:
        many.close()


def test_every_length_across_a_window_edge(pp):
    # heights that move the end of the data by some tens of bytes over a window's 1260 and an overlap's 252
    files = [_file(7, 64, 16 * k, 88, MODE_420) for k in range(1, 33)]
    check_against_oracle(pp, files, 0, 1, 1, "f32")
    assert _decoded(pp, len(files)) == {STREAM_WINDOWS}


def test_streams_with_and_without_markers_in_one_batch(pp):
    rgb = synth.gradient_noise_image(np.random.default_rng(3), 300, 251, 12.0)
    files = [oracle.encode(rgb, 88, m, dri)[0] for m in MODES for dri in (0, 5, 0, 200)]
    check_against_oracle(pp, files, 0, 1, 1, "f16")
    assert [pp.debug_last_stream(i) for i in range(4)] == [STREAM_WINDOWS, STREAM_WHOLE, STREAM_WINDOWS, STREAM_WHOLE]


def test_markers_and_damage_inside_the_data(pp):
    # a restart marker in a file that declares none, a cut file, bytes left over: refused as before,
    # and the sound files around them are decoded
    good = _file(5, 256, 256, 90, MODE_420)
    mid = len(good) // 2
    while good[mid - 1] == 0xFF or good[mid] == 0xFF:
        mid += 1
    marker = good[:mid] + b"\xff\xd0" + good[mid:]
    cut = good[:mid] + b"\xff\xd9"
    left = good[:-2] + b"\x55\x55\x55" + b"\xff\xd9"
    status, tensor = run_gpu(pp, [good, marker, cut, good, left, good], 0, 64, 64, "f32")
    assert [s == 0 for s in status] == [True, False, False, True, False, True], status
    assert [pp.debug_last_stream(i) for i in range(6)] == [STREAM_WINDOWS, STREAM_UNJOINED, STREAM_UNJOINED,
                                                           STREAM_WINDOWS, STREAM_UNJOINED, STREAM_WINDOWS]
    coef = oracle.decode(good)[0]
    for i in (0, 3, 5):
        assert np.array_equal(pp.debug_last_coefficients(i, coef.shape[0]), coef)
    for i in (1, 2, 4):
        assert not np.any(tensor[i])


@pytest.mark.parametrize("seed", [31, 32])
def test_random_damage(pp, seed):
    # every stream is cut; those whose windows show the damage are decoded again, and refused or
    # decoded as the oracle decodes them
    streams = damaged_streams(seed, 8, bases=WINDOW_BASES)
    status, tensor = run_gpu(pp, streams, 0, 64, 64, "f32")
    check_damaged(streams, status, lambda i, nb: pp.debug_last_coefficients(i, nb), tensor)
    assert _decoded(pp, len(streams)) == {STREAM_WINDOWS, STREAM_UNJOINED}


# windows of 1.3 KB in these calls (at most 1 MiB of data): one image of most of the windows that such a call can have,
# which the larger tile of chain_streams holds, and one of more than the smaller tile's beside many of one window, which
# keep it small
@pytest.mark.parametrize("n_small,w,h", [(0, 1600, 1400), (8, 1100, 800)])
def test_chains_longer_than_a_tile(n_small, w, h):
    import paper_2411_19114_amd as prep
    files = [_file(77, w, h, 94, MODE_420, sigma=9.0)] + [_file(80 + k, 24, 16, 60, MODE_420) for k in range(n_small)]
    windows = len(files[0]) // ((42 - 7) * 36)  # (42 rows of 36 bytes, seven of which overlap the next window)
    assert sum(map(len, files)) < 1 << 20 and windows > (640 if n_small == 0 else 256)
    h = prep.Preprocessor(device=0, max_batch=len(files), max_width=w, max_height=h, max_bitstream_bytes=1 << 20,
                          flags=prep.FLAG_FULL_RGB)
    try:
        check_against_oracle(h, files, 0, 1, 1, "f32")
        assert _decoded(h, len(files)) == {STREAM_WINDOWS}
    finally:
        h.close()


def test_more_windows_than_the_larger_tile():
    # windows of 2.6 KB (more than 1 MiB of data): a full tile of 833 of them, and some
    import paper_2411_19114_amd as prep
    f = _file(41, 2800, 2500, 93, MODE_420, sigma=8.0)
    assert 834 < len(f) // ((42 - 4) * 68) < 2 * 833
    h = prep.Preprocessor(device=0, max_batch=1, max_width=2800, max_height=2500, max_bitstream_bytes=len(f))
    try:
        check_against_oracle(h, [f], 0, 64, 64, "f32")
        assert _decoded(h, 1) == {STREAM_WINDOWS}
    finally:
        h.close()
