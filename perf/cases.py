"""What is timed when the speed of this library is measured: batches of JPEG files (host or
device resident) to model-input tensors, decoded frames through the resize stage, and
utterances to log-Mel features, over the sizes and options that serving and evaluation use.

A JPEG case: `n` files, widths and heights drawn from [w_lo, w_hi] x [h_lo, h_hi], chroma
`mode` (420, 422, 444, gray, or mixed = 444 / 420 / gray in turn), quality drawn from
[q_lo, q_hi], `restart` (none, row = a marker per MCU row, 8 = a marker per eight MCUs).
`optimised` of every eight files carry Huffman tables of their own.  Content is smooth or soft
edged with Gaussian noise, so that the bits per pixel are those of photographs.
"""
import concurrent.futures
import functools
import math
import weakref

import numpy as np
import torch

import paper_2411_19114_amd as prep
import synth
from paper_2411_19114_amd.binding import make_params

MODES = {"444": 0, "420": 1, "gray": 2, "422": 3}
# compressed bytes per pixel at these qualities (soft-edged content, noise of 6 levels)
QUALITIES = (50, 65, 75, 85, 90, 95)
BYTES_PER_PIXEL = {"444": (0.065, 0.094, 0.133, 0.22, 0.356, 0.761), "420": (0.048, 0.071, 0.096, 0.152, 0.226, 0.383),
                   "422": (0.054, 0.078, 0.106, 0.171, 0.253, 0.489), "gray": (0.036, 0.058, 0.082, 0.133, 0.199, 0.332)}
SAMPLES_PER_PIXEL = {"444": 3.0, "420": 1.5, "422": 2.0, "gray": 1.0}


def _jpeg(name, n, w, h, mode="420", q=(90, 90), restart="none", content="shapes", optimised=1, short=256, crop=224,
          dtype="f16", filter="bilinear", smooth=False, source="host"):
    case = {"kind": "jpeg", "n": n, "w_lo": w[0], "w_hi": w[1], "h_lo": h[0], "h_hi": h[1], "mode": mode,
            "q_lo": q[0], "q_hi": q[1], "restart": restart, "content": content, "optimised": optimised,
            "short": short, "crop": crop, "dtype": dtype, "filter": filter, "smooth": smooth, "source": source}
    return dict(case, name=name) if name else case


def _frames(name, n, w, h, short, crop, dtype, filter):
    case = {"kind": "frames", "n": n, "w_lo": w[0], "w_hi": w[1], "h_lo": h[0], "h_hi": h[1], "content": "shapes",
            "short": short, "crop": crop, "dtype": dtype, "filter": filter}
    return dict(case, name=name) if name else case


def _audio(name, n, sec_lo, sec_hi, rate, mels):
    case = {"kind": "audio", "n": n, "sec_lo": sec_lo, "sec_hi": sec_hi, "rate": rate, "mels": mels}
    return dict(case, name=name) if name else case


def listed():
    small, photo_w, photo_h, hd_w, hd_h = (256, 256), (300, 640), (250, 500), (1920, 1920), (1080, 1080)
    return [
        # a request served by itself: one small image whose encoder wrote restart markers
        _jpeg("one_small_markers", 1, small, small, q=(85, 85), restart="row", content="gradient", dtype="f32"),
        # a request served by itself: one photograph as cameras and web servers write it, no markers
        _jpeg("one_photo", 1, (500, 500), (375, 375)),
        # the same for a full-HD still, resized crop kept as 8-bit RGB
        _jpeg("one_hd", 1, hd_w, hd_h, q=(95, 95), short=384, crop=384, dtype="u8"),
        # a consumer of the batching server: eight small images at a time
        _jpeg("serve_8_small", 8, small, small, q=(85, 85), restart="row", content="gradient", dtype="f32"),
        # a model's whole batch of small images, already on the GPU
        _jpeg("batch_64_small", 64, small, small, q=(85, 85), restart="row", content="gradient", dtype="f32",
              source="resident"),
        # classification in bulk: photographs of all sizes with frequent markers
        _jpeg("photos_256_markers", 256, photo_w, photo_h, restart="8", source="resident"),
        # the same from files as they are found (no markers), with the filters of image libraries:
        # antialiased reduction, interpolated chroma
        _jpeg("photos_128_library", 128, photo_w, photo_h, filter="antialias", smooth=True),
        # video frames or camera stills: 64 full-HD images
        _jpeg("hd_64_markers", 64, hd_w, hd_h, q=(95, 95), restart="row", short=384, crop=384, source="resident"),
        # thumbnails of mixed sampling and quality, no markers
        _jpeg("thumbs_512_mixed", 512, small, small, mode="mixed", q=(50, 95), content="gradient", source="resident"),
        # frames that a hardware decoder left in memory: resize, crop and normalize only
        _frames("frames_32", 32, hd_w, hd_h, 384, 384, "f16", "bilinear"),
        # one utterance for a speech model, already at the model's rate
        _audio("one_utterance", 1, 12.0, 12.0, 16000, 80),
        # transcription in bulk: 64 recordings of 1.5 to 35 s at 44.1 kHz
        _audio("utterances_64", 64, 1.5, 35.0, 44100, 80),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng):
    w = _log(rng, 64, 1920)
    return w, max(48, min(1088, int(w * rng.uniform(0.5, 1.4))))


def _output(rng):
    short = rng.randint(96, 400)
    return short, rng.randint(80, short), rng.choice(("f32", "f16", "f16", "u8")), rng.choice(("bilinear", "bilinear", "antialias"))


def draw(rng):
    what = rng.random()
    if what < 0.2:
        n = _log(rng, 1, 64)
        hi = rng.uniform(2.0, min(35.0, 700.0 / n))
        lo = hi if rng.random() < 0.3 else rng.uniform(1.0, hi)
        return _audio(None, n, round(lo, 2), round(hi, 2), rng.choice((8000, 16000, 22050, 44100, 48000)), rng.choice((40, 64, 80, 128)))
    w, h = _size(rng)
    short, crop, dtype, filter = _output(rng)
    # at most 48 Mpixel in and 24 M outputs a plane
    most = max(1, min(512, 48000000 // (w * h), 24000000 // (crop * crop)))
    n = _log(rng, 1, most)
    spread = (rng.random() < 0.5)
    ws, hs = ((max(48, int(w * 0.6)), w), (max(48, int(h * 0.6)), h)) if spread else ((w, w), (h, h))
    if what < 0.3:
        return _frames(None, min(n, 128), ws, hs, short, crop, dtype, filter)
    q = rng.randint(50, 95)
    return _jpeg(None, n, ws, hs, rng.choice(("420", "420", "420", "422", "444", "gray", "mixed")),
                 (q, q) if rng.random() < 0.5 else (50, q), rng.choice(("none", "none", "row", "8")),
                 rng.choice(("shapes", "gradient")), rng.choice((0, 1, 8)), short, crop, dtype, filter,
                 rng.random() < 0.25, rng.choice(("host", "resident")))


# ---- inputs ----------------------------------------------------------------------------------

def _picture(gen, w, h, content, rnd):
    """One RGB picture (uint8 [h, w, 3] on the GPU): a colour gradient with noise of 8 levels, or
    5 to 15 soft-edged rectangles and ellipses with noise of 6 (synth's two kinds of content)."""
    dev = gen.device
    x = torch.arange(w, device=dev, dtype=torch.float32)[None, :]
    y = torch.arange(h, device=dev, dtype=torch.float32)[:, None]
    noise = torch.randn((h, w, 3), generator=gen, device=dev)
    if content == "gradient":
        a, bx, by = (torch.tensor([rnd.uniform(*r) for _ in range(3)], dtype=torch.float32, device=dev)
                     for r in ((48.0, 208.0), (-48.0, 48.0), (-48.0, 48.0)))
        img = a + bx * (x / w)[..., None] + by * (y / h)[..., None] + 8.0 * noise
    else:
        k, blur = int(rnd.integers(5, 16)), rnd.uniform(1.0, 3.0)
        p = torch.from_numpy(np.stack([rnd.uniform(0, w, k), rnd.uniform(0, h, k), rnd.uniform(0.05, 0.35, k) * w,
                                       rnd.uniform(0.05, 0.35, k) * h, rnd.random(k)]).astype(np.float32)).to(dev)
        colour = torch.from_numpy(rnd.uniform(0.0, 255.0, (k + 1, 3)).astype(np.float32)).to(dev)
        cx, cy, rx, ry, square = (v[:, None, None] for v in p)
        dx, dy = (x - cx).abs(), (y - cy).abs()
        # distance to the edge in pixels, negative inside
        box = torch.maximum(dx - rx, dy - ry)
        oval = (torch.sqrt((dx / rx) ** 2 + (dy / ry) ** 2) - 1.0) * torch.minimum(rx, ry)
        cover = torch.sigmoid(torch.where(square < 0.5, box, oval) * (-1.7 / blur))
        img = colour[0].expand(h, w, 3)
        for i in range(k):
            img = torch.lerp(img, colour[i + 1], cover[i][..., None])
        img = img + 6.0 * noise
    return img.round_().clamp_(0, 255).to(torch.uint8)


def _pictures(case, seed):
    rnd = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    for _ in range(case["n"]):
        yield _picture(gen, int(rnd.integers(case["w_lo"], case["w_hi"] + 1)),
                       int(rnd.integers(case["h_lo"], case["h_hi"] + 1)), case["content"], rnd)


@functools.lru_cache(None)
def _encoders():
    return concurrent.futures.ThreadPoolExecutor(16)


def _files(case, seed):
    rnd = np.random.default_rng(seed + 1)
    restart = {"none": {}, "row": {"restart_rows": 1}, "8": {"restart_blocks": 8}}[case["restart"]]
    jobs = []
    for i, picture in enumerate(_pictures(case, seed)):
        mode = ("444", "420", "gray")[i % 3] if case["mode"] == "mixed" else case["mode"]
        jobs.append(_encoders().submit(synth.encode_jpeg, picture.cpu().numpy(), rnd.integers(case["q_lo"], case["q_hi"] + 1),
                                       MODES[mode], optimize=i % 8 >= 8 - case["optimised"], **restart))
    return synth.pack([j.result() for j in jobs])


def _speech(case, seed):
    """Drifting harmonics under a slow envelope plus noise, float32, peak 0.5, back to back."""
    rnd = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rate, waves = case["rate"], []
    # (the lengths belong to the case, so that the features of every seed have one shape)
    for sec in np.random.default_rng(case["n"]).uniform(case["sec_lo"], case["sec_hi"], case["n"]):
        m = int(rate * sec)
        t = torch.arange(m, device="cuda", dtype=torch.float64) / rate
        f = rnd.uniform(0.7, 1.7)
        phase = 2 * math.pi * (rnd.uniform(110.0, 170.0) * t - 20.0 / (2 * math.pi * f) * torch.cos(2 * math.pi * f * t))
        x = torch.zeros_like(t)
        for k in range(1, 12):
            x += rnd.random() / k ** 0.8 * torch.sin(k * phase + rnd.random() * 6.28)
        x *= 0.55 + 0.45 * torch.sin(2 * math.pi * 3.1 * t + rnd.random() * 6.28)
        x += 0.2 * torch.randn(m, generator=gen, device="cuda", dtype=torch.float64)
        waves.append((0.5 * x / x.abs().max()).float())
    offsets = np.zeros(case["n"] + 1, dtype=np.uint64)
    np.cumsum([w.numel() for w in waves], out=offsets[1:])
    return torch.cat(waves), offsets


# ---- what a program keeps ------------------------------------------------------------------------

_handles = weakref.WeakValueDictionary()  # a program has one handle for all its batches


def _handle(key, make):
    h = _handles.get(key)
    if h is None:
        h = make()
        _handles[key] = h
    return h


def _jpeg_handle(case):
    n, w, h = case["n"], case["w_hi"], case["h_hi"]
    flags = prep.FLAG_SMOOTH_CHROMA if case["smooth"] else 0
    return _handle(("jpeg", n, w, h, flags),
                   lambda: prep.Preprocessor(max_batch=n, max_width=w, max_height=h, flags=flags,
                                             max_bitstream_bytes=n * (w * h * 5 // 4 + 4096)))


def _params(case):
    return make_params(case["short"], case["crop"], case["crop"], case["dtype"], synth.IMAGENET_MEAN, synth.IMAGENET_STD,
                       prep.FILTER_ANTIALIAS if case["filter"] == "antialias" else prep.FILTER_BILINEAR)


def _out(case):
    n, c = case["n"], case["crop"]
    if case["dtype"] == "u8":
        return torch.zeros((n, c, c, 3), dtype=torch.uint8, device="cuda")
    return torch.zeros((n, 3, c, c), dtype=torch.float16 if case["dtype"] == "f16" else torch.float32, device="cuda")


def prepare(case, seed):
    state = {"kind": case["kind"]}
    if case["kind"] == "jpeg":
        state["blob"], state["offsets"] = _files(case, seed)
        state["device"] = torch.from_numpy(state["blob"]).cuda() if case["source"] == "resident" else None
        state.update(handle=_jpeg_handle(case), params=_params(case), out=_out(case))
    elif case["kind"] == "frames":
        frames = list(_pictures(case, seed))
        size = np.array([f.numel() for f in frames], dtype=np.uint64)
        state["offsets"] = np.concatenate([np.zeros(1, np.uint64), np.cumsum(size)[:-1]])
        state["heights"] = np.array([f.shape[0] for f in frames], dtype=np.int32)
        state["widths"] = np.array([f.shape[1] for f in frames], dtype=np.int32)
        state["device"] = torch.cat([f.reshape(-1) for f in frames])
        state.update(params=_params(case), out=_out(case))
    else:
        state["device"], state["offsets"] = _speech(case, seed)
        most = int(case["sec_hi"] * max(case["rate"], 16000) + 1) * case["n"]
        state["handle"] = _handle(("audio", case["n"], most, case["mels"]),
                                  lambda: prep.AudioPreprocessor(case["n"], most, n_mels=case["mels"]))
        frames = sum(state["handle"].frames(int(m), case["rate"]) for m in np.diff(state["offsets"].astype(np.int64)))
        state.update(rate=case["rate"], out=torch.zeros(frames * case["mels"], dtype=torch.float32, device="cuda"))
    return state


def run(state):
    stream = torch.cuda.current_stream().cuda_stream
    out = state["out"]
    if state["kind"] == "jpeg":
        if state["device"] is None:
            state["handle"].decode_resize_batch(state["blob"], state["offsets"], state["params"], out.data_ptr(), stream)
        else:
            state["handle"].decode_resize_batch_resident(state["blob"], state["device"].data_ptr(), state["offsets"],
                                                         state["params"], out.data_ptr(), stream)
        return out
    if state["kind"] == "frames":
        prep.resize_normalize_static(0, state["device"].data_ptr(), state["offsets"], state["widths"], state["heights"],
                                     state["widths"] * 3, state["params"], out.data_ptr(), stream)
        return out
    return out, state["handle"].features(state["device"].data_ptr(), state["offsets"], state["rate"], out.data_ptr(), stream)


# ---- the work ----------------------------------------------------------------------------------------

def _bytes_per_pixel(mode, q):
    if mode == "mixed":
        return sum(_bytes_per_pixel(m, q) for m in ("444", "420", "gray")) / 3
    return float(np.interp(q, QUALITIES, BYTES_PER_PIXEL[mode]))


def work(case):
    """Bytes: the files (or samples) in, the tensor out.  Operations: the inverse transform and
    the colour of the pixels under the crop window, four (or all covered) taps an output; the
    transform, the filters and the interpolation of the audio path.  Sizes that are drawn count
    with their means; entropy decoding is not counted, it has no floating-point operations."""
    if case["kind"] == "audio":
        sec = case["n"] * (case["sec_lo"] + case["sec_hi"]) / 2
        frames = sec * 100 + case["n"]
        taps = 0 if case["rate"] == 16000 else 2 * 6 / 0.99 * max(1.0, case["rate"] / 16000)
        return {"bytes": 4 * sec * case["rate"] + 4 * frames * case["mels"],
                "flops": frames * (2.5 * 512 * 9 + 3 * 257 + 4 * 257 + 8 * case["mels"]) + sec * 16000 * 2 * taps}
    w, h = (case["w_lo"] + case["w_hi"]) / 2, (case["h_lo"] + case["h_hi"]) / 2
    pixels, outputs, scale = w * h, case["crop"] ** 2, max(min(w, h) / case["short"], 1e-3)
    seen = min(1.0, (case["crop"] / case["short"]) ** 2 * min(w, h) / max(w, h))  # share under the crop window
    out = outputs * 3 * {"f32": 4, "f16": 2, "u8": 1}[case["dtype"]]
    taps = 4 * max(1.0, scale) ** 2 if case["filter"] == "antialias" else 4
    flops = outputs * 3 * (2 * taps + 2)
    if case["kind"] == "frames":
        return {"bytes": case["n"] * (min(3 * pixels * seen, 3.0 * outputs * taps) + out), "flops": case["n"] * flops}
    bpp = (_bytes_per_pixel(case["mode"], case["q_lo"]) + _bytes_per_pixel(case["mode"], case["q_hi"])) / 2
    samples = sum(SAMPLES_PER_PIXEL[m] for m in ("444", "420", "gray")) / 3 if case["mode"] == "mixed" else SAMPLES_PER_PIXEL[case["mode"]]
    return {"bytes": case["n"] * (700 + pixels * bpp + out), "flops": case["n"] * (flops + pixels * seen * (9.5 * samples + 7))}


def tolerance(case):
    """Decoded samples are rounded to 8 bits on the way: another correct decoder puts a few of
    them in 100 000 one level off (two in blue), which is 0.02 to 0.04 of the tensor's unit
    deviation in those places and nothing elsewhere; fp16 adds its own rounding, and the 8-bit
    output may round the other way within 2^-12 of a half.  Audio is 64-bit up to 32-bit features."""
    if case["kind"] == "audio":
        return {"rel": 1e-5, "max": 1e-3}
    if case["dtype"] == "u8":
        return {"differ": 1e-3}
    return {"rel": 1e-3 if case["dtype"] == "f16" else 1e-4, "max": 0.05}
