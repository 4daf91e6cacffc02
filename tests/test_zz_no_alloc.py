"""The entry point that allocates nothing (prep_resize_normalize_static) against the entry
point it is a variant of (prep_resize_normalize): same kernels, so the outputs must be equal
bit for bit, on two calls in a row, the second with a smaller input (the library's device
array keeps the first call's records)."""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import oracle  # noqa: E402
import paper_2411_19114_amd as prep  # noqa: E402
from paper_2411_19114_amd.binding import make_params  # noqa: E402

pytestmark = pytest.mark.gpu

MEAN, STD = (0.485, 0.456, 0.406), (0.229, 0.224, 0.225)


def _run_both(pp, imgs, shapes, rs, ch, cw, dt, aa):
    import torch
    flat = np.concatenate([im.reshape(-1) for im in imgs])
    offs = np.cumsum([0] + [im.size for im in imgs[:-1]]).astype(np.uint64)
    dev = torch.from_numpy(flat).to("cuda:0")
    tdt = {"f16": torch.float16, "f32": torch.float32, "u8": torch.uint8}[dt]
    shape = (len(imgs), ch, cw, 3) if dt == "u8" else (len(imgs), 3, ch, cw)
    want = torch.full(shape, 77, dtype=tdt, device="cuda:0")
    got = torch.full(shape, 99, dtype=tdt, device="cuda:0")
    params = make_params(rs, ch, cw, dt, MEAN, STD, aa)
    stream = torch.cuda.current_stream().cuda_stream
    w, h, p = [s[0] for s in shapes], [s[1] for s in shapes], [s[0] * 3 for s in shapes]
    pp.resize_normalize(dev.data_ptr(), offs, w, h, p, params, want.data_ptr(), stream)
    prep.resize_normalize_static(0, dev.data_ptr(), offs, w, h, p, params, got.data_ptr(), stream)
    torch.cuda.synchronize()
    return want.cpu().numpy(), got.cpu().numpy()


def test_static_entry_point_equals_the_handle_entry_point_on_two_calls_in_a_row():
    import torch
    assert torch.cuda.is_available()
    pp = prep.Preprocessor(device=0, max_batch=80, max_width=1920, max_height=1080, max_bitstream_bytes=1 << 20)
    rng = np.random.default_rng(41)
    # first call: 70 images (three fills of the record array), second: 3 smaller ones
    first = [(int(rng.integers(40, 400)), int(rng.integers(40, 300))) for _ in range(69)] + [(1920, 1080)]
    second = [(33, 77), (256, 256), (300, 200)]
    for shapes, (rs, ch, cw, dt, aa) in ((first, (36, 32, 30, "f16", 0)), (second, (32, 30, 32, "f32", 0)),
                                         (first, (36, 32, 30, "f32", 1)), (second, (24, 24, 20, "u8", 1))):
        imgs = [rng.integers(0, 256, size=(h, w, 3), dtype=np.uint8) for w, h in shapes]
        want, got = _run_both(pp, imgs, shapes, rs, ch, cw, dt, aa)
        assert np.array_equal(want, got), (len(shapes), rs, ch, cw, dt, aa)
        if dt != "u8":
            # and both are the oracle's resize, to the stage's bar
            tol = 0.02 if dt == "f16" else 1e-4
            for i in (0, len(imgs) - 1):
                ref = oracle.preprocess(imgs[i], rs, ch, cw, MEAN, STD, bool(aa))
                assert np.abs(got[i].astype(np.float64) - ref).max() <= tol
    pp.close()


def test_static_entry_point_refuses_what_does_not_fit():
    import torch
    params = make_params(0, 4, 4, "f32", MEAN, STD)
    n = 1025
    dev = torch.zeros(8 * 8 * 3, dtype=torch.uint8, device="cuda:0")
    out = torch.zeros(4, dtype=torch.float32, device="cuda:0")
    with pytest.raises(prep.PrepError) as e:
        prep.resize_normalize_static(0, dev.data_ptr(), np.zeros(n, dtype=np.uint64), [8] * n, [8] * n, [24] * n,
                                     params, out.data_ptr(), 0)
    assert e.value.code == prep.E_TOO_LARGE
    with pytest.raises(prep.PrepError) as e:
        prep.resize_normalize_static(0, dev.data_ptr(), np.zeros(1, dtype=np.uint64), [8], [8], [24],
                                     make_params(0, 16, 16, "f32", MEAN, STD), out.data_ptr(), 0)
    assert e.value.code == prep.E_INVALID_ARG


@pytest.mark.parametrize("dt,aa,rs", [("f32", 0, 6), ("f32", 1, 6), ("f32", 0, 1), ("f32", 1, 1), ("f16", 1, 4)])
def test_rows_at_the_edges_of_wide_loads(dt, aa, rs):
    # rows of 3 to 33 bytes and one of 900, back to back and at odd addresses: loads that are moved
    # back at the end of a row, images too narrow for them, reductions with tall windows.  Bars: those of
    # the other test (fp32 sums of 8-bit samples, and half a unit of fp16 at a magnitude below 4).
    rng = np.random.default_rng(43)
    shapes = [(w, h) for w in range(1, 12) for h in (1, 2, 9)] + [(300, 17), (9, 64), (3, 5)]
    imgs = [rng.integers(0, 256, size=(h, w, 3), dtype=np.uint8) for w, h in shapes]
    pp = prep.Preprocessor(device=0, max_batch=len(imgs), max_width=320, max_height=320, max_bitstream_bytes=1 << 20)
    want, got = _run_both(pp, imgs, shapes, rs, rs, rs, dt, aa)
    pp.close()
    assert np.array_equal(want, got)
    for im, g in zip(imgs, got):
        ref = oracle.preprocess(im, rs, rs, rs, MEAN, STD, bool(aa))
        assert np.abs(g.astype(np.float64) - ref).max() <= (0.02 if dt == "f16" else 1e-4), im.shape
