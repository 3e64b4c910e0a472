"""The work that users of the Encode-stage library have it do, as cases for timing it.

Four kinds, each one call (or one batch) of the C ABI in ``include/epd_encode.h``:

  encode      packed patch rows -> visual tokens (``epd_encode``)
  preprocess  raw uint8 pixels -> packed patch rows (``epd_preprocess``)
  cached      raw uint8 pixels -> visual tokens of items the feature store already holds
              (``epd_encode_cached``, every item a hit)
  hash        raw uint8 buffers -> store keys (``MMStore.hash``)

``model`` names a configuration of ``workloads.py``; its weights are drawn at random.  ``items``
lists patch grids "t x h x w", ``sources`` the pixel sizes "h x w" of the raw frames (one per
item), ``sizes`` the bytes of each hashed buffer.
"""

import ctypes
import math

import numpy as np
import torch

from paper_2601_11590_amd import binding as B, workloads as W

DEVICE = "cuda:0"
MEAN, STD = [0.48, 0.46, 0.41], [0.27, 0.26, 0.28]     # of the order image processors use
SALT = 7


# ------------------------------------------------------------------ text <-> sizes

def _join(rows):
    return ",".join("x".join(str(int(v)) for v in r) for r in rows)


def _rows(text):
    return [tuple(int(v) for v in r.split("x")) for r in text.split(",")]


# ------------------------------------------------------------------ the cases

def listed():
    mixed = [(448, 448), (480, 640), (1080, 1920), (224, 224), (600, 400), (448, 448), (333, 777), (900, 900)]
    return [
        # the fp32 configuration: one 224 x 224 image through one layer; launches and latency
        {"name": "encode-f32-image", "kind": "encode", "model": "C1", "items": "1x16x16", "segments": "item"},
        # one 448 x 448 image of a chat request, alone: 784 tokens against 0.6 B weights
        {"name": "encode-1-image", "kind": "encode", "model": "C2", "items": "1x28x28", "segments": "item"},
        # the same encoder on a batch of eight
        {"name": "encode-8-images", "kind": "encode", "model": "C2", "items": _join(W.grids_for(W.C2)), "segments": "item"},
        # 32 images of as many sizes packed into one ragged batch
        {"name": "encode-32-ragged", "kind": "encode", "model": "C3", "items": _join(W.grids_for(W.C3)), "segments": "item"},
        # five document / screenshot resolutions, 400 to 10 764 tokens, LayerNorm and head dim 72
        {"name": "encode-5-resolutions", "kind": "encode", "model": "T42",
         "items": _join(W.t42_grid(h, w) for h, w in W.T42_SIZES_PX[:5]), "segments": "item"},
        # one 2688 x 2688 image: attention over 28 224 tokens
        {"name": "encode-long-image", "kind": "encode", "model": "C4", "items": _join(W.grids_for(W.C4)), "segments": "item"},
        # one clip of 16 frames through the 6 B video encoder, attention inside every frame
        {"name": "encode-clip-frames", "kind": "encode", "model": "C5", "items": "8x32x32", "segments": "frame"},
        # four clips, attention over whole clips: the largest call
        {"name": "encode-4-clips", "kind": "encode", "model": "C5", "items": _join(W.grids_for(W.C5)), "segments": "item"},
        # eight uploads of different sizes resized to 448 x 448
        {"name": "preprocess-8-images", "kind": "preprocess", "model": "C2", "items": _join([(1, 28, 28)] * 8), "sources": _join(mixed)},
        # 64 decoded video frames already at the encoder's size
        {"name": "preprocess-4-clips", "kind": "preprocess", "model": "C5", "items": _join(W.grids_for(W.C5)), "sources": _join([(448, 448)] * 4)},
        # eight images that were all seen before: hash, look up, copy
        {"name": "cached-8-images", "kind": "cached", "model": "C2", "items": _join([(1, 28, 28)] * 8), "sources": _join([(448, 448)] * 8)},
        # keys of the four clips
        {"name": "hash-4-clips", "kind": "hash", "sizes": ",".join([str(3 * 16 * 448 * 448)] * 4)},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _images(rng, n, lo, hi, limit):
    """n grids of even sides in [lo, hi] patches, shrunk until at most `limit` tokens in all."""
    even = lambda v: max(lo, v // 2 * 2)
    grids = [(1, even(_log_int(rng, lo, hi)), even(_log_int(rng, lo, hi))) for _ in range(n)]
    while W.num_tokens(grids) > limit:
        grids = [(t, even(int(h * 0.9)), even(int(w * 0.9))) for t, h, w in grids]
    return grids


def _sources(rng, grids, patch):
    """Raw sizes of the items: the encoder's own size, or 0.4 to 3 times it."""
    out = []
    for _, h, w in grids:
        if rng.random() < 0.3:
            out.append((h * patch, w * patch))
        else:
            out.append((max(9, int(h * patch * math.exp(rng.uniform(-0.9, 1.1)))), max(9, int(w * patch * math.exp(rng.uniform(-0.9, 1.1))))))
    return out


def draw(rng):
    what = rng.choice(["C1", "C2", "C2", "C2", "C4", "T42", "C5", "preprocess", "preprocess", "cached", "hash"])
    if what == "C1":
        return {"kind": "encode", "model": "C1", "items": _join(_images(rng, rng.randint(1, 4), 8, 32, 2048)), "segments": "item"}
    if what == "C2":
        return {"kind": "encode", "model": "C2", "items": _join(_images(rng, _log_int(rng, 1, 32), 8, 84, 73896)), "segments": "item"}
    if what == "C4":
        return {"kind": "encode", "model": "C4", "items": _join(_images(rng, rng.randint(1, 3), 20, 168, 28224)), "segments": "item"}
    if what == "T42":
        return {"kind": "encode", "model": "T42", "items": _join(_images(rng, rng.randint(1, 6), 12, 138, 24000)), "segments": "item"}
    if what == "C5":
        clip = lambda: (rng.randint(1, 8), 2 * rng.randint(6, 16), 2 * rng.randint(6, 16))
        return {"kind": "encode", "model": "C5", "items": _join(clip() for _ in range(rng.randint(1, 4))), "segments": rng.choice(["item", "frame"])}
    if what == "preprocess":
        if rng.random() < 0.6:
            grids = _images(rng, _log_int(rng, 1, 32), 8, 84, 40000)
            return {"kind": "preprocess", "model": "C2", "items": _join(grids), "sources": _join(_sources(rng, grids, 16))}
        grids = [(rng.randint(1, 8), 2 * rng.randint(8, 16), 2 * rng.randint(8, 16)) for _ in range(rng.randint(1, 4))]
        return {"kind": "preprocess", "model": "C5", "items": _join(grids), "sources": _join(_sources(rng, grids, 14))}
    if what == "cached":
        grids = _images(rng, _log_int(rng, 1, 16), 14, 84, 32000)
        return {"kind": "cached", "model": "C2", "items": _join(grids), "sources": _join(_sources(rng, grids, 16))}
    n = _log_int(rng, 1, 40)
    return {"kind": "hash", "sizes": ",".join(str(_log_int(rng, 20000, 64000000 // n)) for _ in range(n))}


# ------------------------------------------------------------------ what a program has in hand

class _Encoder:
    """An encoder handle made from random weights that are already on the GPU, and its workspace."""

    def __init__(self, cfg, gen, max_tokens, max_segments, max_items):
        dt = B.torch_dtype(cfg.dtype)
        ccfg = B.make_cfg(cfg, max_tokens, max_segments, max_items)

        def tensor(name):
            t = torch.randn(W._tensor_shape(cfg, name), generator=gen, device=DEVICE, dtype=torch.float32).mul_(0.02)
            return (t.add_(1.0) if name.endswith("_g") else t).to(dt)

        glob = {n: tensor(n) for n in W._GLOBAL_TENSORS if W._present(cfg, n)}
        layers = [{n: tensor(n) for n in W._LAYER_TENSORS if W._present(cfg, n)} for _ in range(cfg.num_layers)]
        arr = (B.epd_layer_weights * max(1, len(layers)))()
        for slot, lw in zip(arr, layers):
            for n, t in lw.items():
                setattr(slot, n, t.data_ptr())
        w = B.epd_weights()
        for n, t in glob.items():
            setattr(w, n, t.data_ptr())
        w.layers = ctypes.cast(arr, ctypes.POINTER(B.epd_layer_weights))
        need = B.epd_encode_workspace_bytes(ccfg)
        self.workspace = torch.empty(need + 256, dtype=torch.uint8, device=DEVICE)
        ccfg.weights = ctypes.pointer(w)
        ccfg.workspace = (self.workspace.data_ptr() + 255) // 256 * 256
        ccfg.workspace_bytes = need
        torch.cuda.synchronize()
        self.handle = B.epd_encode_create(ccfg)

    def __del__(self):
        if getattr(self, "handle", None):
            torch.cuda.synchronize()
            B.epd_encode_destroy(self.handle)


def _raw_frames(gen, cfg, grids, sources):
    """Planar uint8 frames, items packed in order: smooth waves plus noise, as natural images have
    correlated neighbours and every byte value."""
    parts = []
    for (t, _, _), (hs, ws) in zip(grids, sources):
        n = cfg.in_channels * t * cfg.temporal_patch
        f = torch.rand((n, 3, 1, 1), generator=gen, device=DEVICE) * 5.5 + 0.5
        y = torch.arange(hs, device=DEVICE, dtype=torch.float32)[None, :, None] / hs
        x = torch.arange(ws, device=DEVICE, dtype=torch.float32)[None, None, :] / ws
        wave = 0.5 + 0.35 * torch.sin(6.2832 * (f[:, 0] * y + f[:, 1] * x) + f[:, 2])
        noise = torch.rand((n, hs, ws), generator=gen, device=DEVICE) * 0.3 - 0.15
        parts.append(((wave + noise) * 255.0).round_().clamp_(0, 255).to(torch.uint8).reshape(-1))
    return torch.cat(parts)


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    s = dict(case)
    if case["kind"] == "hash":
        sizes = [int(v) for v in case["sizes"].split(",")]
        s["offsets"] = np.cumsum([0] + sizes).astype(np.uint64)
        s["salts"] = np.arange(1, len(sizes) + 1, dtype=np.uint64)
        s["pixels"] = torch.randint(0, 256, (sum(sizes),), generator=gen, device=DEVICE, dtype=torch.uint8)
        s["store"] = B.MMStore(2 << 20, DEVICE)
        return s
    cfg, grids = W.CONFIGS[case["model"]], _rows(case["items"])
    dt = B.torch_dtype(cfg.dtype)
    T, Tm = W.num_tokens(grids), W.num_merged_tokens(grids, cfg.merge)
    s["cu"], s["grid"] = W.metadata(grids, case.get("segments", "item"))
    s["tm"], s["out_dim"], s["dtype"] = Tm, cfg.out_dim, dt
    if case["kind"] == "encode":
        s["encoder"] = _Encoder(cfg, gen, T, len(s["cu"]) - 1, len(grids))
        s["patches"] = torch.rand((T, cfg.patch_dim), generator=gen, device=DEVICE, dtype=torch.float32).to(dt)
        return s
    s["src"] = np.asarray(_rows(case["sources"]), dtype=np.int32)
    s["pixels"] = _raw_frames(gen, cfg, grids, s["src"].tolist())
    s["rows"] = torch.empty((T, cfg.patch_dim), dtype=dt, device=DEVICE)
    if case["kind"] == "preprocess":      # the encoder behind it does not matter here: no layers
        s["encoder"] = _Encoder(cfg.replace(num_layers=0), gen, T, len(grids), len(grids))
        return s
    s["encoder"] = _Encoder(cfg, gen, T, len(grids), len(grids))
    s["scratch"] = torch.empty((Tm, cfg.out_dim), dtype=dt, device=DEVICE)
    s["store"] = B.MMStore((1 << 20) + 2 * Tm * cfg.out_dim * 2 + 65536, DEVICE)
    _cached(s)                            # the items were seen before
    torch.cuda.synchronize()
    return s


# ------------------------------------------------------------------ one pass

def _cached(s):
    out = torch.empty((s["tm"], s["out_dim"]), dtype=s["dtype"], device=DEVICE)
    hit, keys = B.epd_encode_cached(s["encoder"].handle, s["store"].handle, SALT, s["pixels"].data_ptr(), s["src"], s["grid"], MEAN, STD,
                                    s["rows"].data_ptr(), s["scratch"].data_ptr(), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    return out, hit, keys.view(np.int64)


def run(state):
    s = state
    if s["kind"] == "hash":
        return s["store"].hash(s["pixels"], s["offsets"], s["salts"]).view(np.int64)
    if s["kind"] == "cached":
        return _cached(s)
    stream = torch.cuda.current_stream().cuda_stream
    if s["kind"] == "preprocess":
        B.epd_preprocess(s["encoder"].handle, s["pixels"].data_ptr(), s["src"], s["grid"], MEAN, STD, s["rows"].data_ptr(), stream)
        return s["rows"]
    out = torch.empty((s["tm"], s["out_dim"]), dtype=s["dtype"], device=DEVICE)
    B.epd_encode(s["encoder"].handle, s["patches"].data_ptr(), s["cu"], s["grid"], out.data_ptr(), stream)
    return out


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    if case["kind"] == "hash":
        return {"bytes": sum(int(v) for v in case["sizes"].split(",")), "flops": 0}
    cfg, grids = W.CONFIGS[case["model"]], _rows(case["items"])
    es = 4 if cfg.dtype == "f32" else 2
    T, Tm = W.num_tokens(grids), W.num_merged_tokens(grids, cfg.merge)
    rows, out = T * cfg.patch_dim * es, Tm * cfg.out_dim * es
    if case["kind"] != "encode":
        raw = sum(cfg.in_channels * t * cfg.temporal_patch * h * w for (t, _, _), (h, w) in zip(grids, _rows(case["sources"])))
        if case["kind"] == "preprocess":
            return {"bytes": raw + rows, "flops": 0}
        return {"bytes": raw + 2 * out, "flops": 0}
    D, F, L = cfg.hidden, cfg.mlp_dim, cfg.num_layers
    cu, _ = W.metadata(grids, case["segments"])
    params = D * cfg.patch_dim + L * (4 * D * D + 2 * D * F) + cfg.merge ** 2 * D * cfg.out_dim
    attn = sum(4.0 * float(b - a) ** 2 * D for a, b in zip(cu[:-1], cu[1:]))
    flops = 2.0 * T * cfg.patch_dim * D + L * (8.0 * T * D * D + 4.0 * T * D * F + attn) + 2.0 * Tm * cfg.merge ** 2 * D * cfg.out_dim
    return {"bytes": params * es + rows + out, "flops": flops}


def tolerance(case):
    if case["kind"] == "hash":
        return "exact"
    if case["kind"] == "preprocess":
        # bf16 results of fp32 arithmetic: another order moves a value by one unit in the last
        # place (2^-7 of it at most), and few values
        return {"rel": 2e-3, "max": 1e-2}
    if W.CONFIGS[case["model"]].dtype == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    # full depth in bf16: the same inputs with the sums of every layer in another order (other GEMM
    # tiles, other query tiles of the attention) differ by rel 2.9e-3 ... 4.7e-3 and max 2.8e-2
    return {"rel": 1.9e-2, "max": 0.11}
