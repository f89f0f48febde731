"""Workloads that stand for what a program does with this library on one GPU.

listed() are fixed cases over the range of real use: the smallest field, where
launches and latency count, ragged ones, the paper's grid sizes, the largest
single field and the batch of many uneven fields; both C schedules; labels,
verification, the storage of the edits in both directions, the learned warm
start and a training step of its network.  draw() gives further cases of the
same ranges.  All inputs are made on the GPU from the seed alone.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2406_09423_amd as msz
from paper_2406_09423_amd import train_net


def listed() -> list:
    return [
        # the smallest field that is corrected in earnest: 21 or so rounds over
        # 16384 vertices, so launches and latency are everything
        {"name": "fix_bumps_128", "kind": "fix", "field": "bumps", "shape": "128x128", "rel": 1e-3, "merged": False},
        # a ragged 2D field (odd sides, rows not 16-byte aligned), parallel C rounds
        {"name": "fix_2d_ragged", "kind": "fix", "field": "grf", "shape": "1153x1795", "rel": 1e-2, "merged": True},
        # an ocean-like 2D field of 8.6 million vertices with the default schedule
        {"name": "fix_2d_ocean", "kind": "fix", "field": "grf", "shape": "2400x3600", "rel": 1e-3, "merged": False},
        # a small 3D simulation block with odd sides, parallel C rounds
        {"name": "fix_3d_ragged", "kind": "fix", "field": "grf", "shape": "48x95x177", "rel": 1e-3, "merged": True},
        # the largest single field: a 512^3 turbulence-like snapshot, default schedule
        {"name": "fix_3d_512", "kind": "fix", "field": "grf", "shape": "512x512x512", "rel": 1e-3, "merged": False},
        # many uneven fields of a run corrected together (64 2D fields, 32 cubes)
        {"name": "batch_96", "kind": "batch", "n2": 64, "n3": 32, "lo2": 64, "hi2": 2048, "lo3": 32, "hi3": 192,
         "shapes_seed": 3, "merged": True},
        # the segmentation of a 3D field on its own
        {"name": "labels_256", "kind": "labels", "field": "grf", "shape": "256x256x256"},
        # the check of a decompressed field against its original (bound of 1e-3)
        {"name": "count_2d_ocean", "kind": "count", "field": "grf", "shape": "2400x3600", "rel": 1e-3},
        # the edits of a corrected field, stored ...
        {"name": "encode_2d_ocean", "kind": "encode", "field": "grf", "shape": "2400x3600", "rel": 1e-3},
        # ... and loaded again
        {"name": "decode_2d_ocean", "kind": "decode", "field": "grf", "shape": "2400x3600", "rel": 1e-3},
        # a correction started from the network's proposal (the stored weights)
        {"name": "learned_256", "kind": "learned", "field": "grf", "shape": "256x256x256", "rel": 1e-3,
         "merged": False},
        # loss and gradients of one training field of the network
        {"name": "train_128", "kind": "train", "shape": "128x128x128", "rel": 1e-3},
    ]


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shape(rng: random.Random, ndim: int, hi2: int = 3000, hi3: int = 288) -> str:
    if ndim == 2:
        return "x".join(str(_log_int(rng, 40, hi2)) for _ in range(2))
    return "x".join(str(_log_int(rng, 16, hi3)) for _ in range(3))


def draw(rng: random.Random) -> dict:
    kind = rng.choice(["fix", "fix", "fix", "batch", "labels", "count", "encode", "decode", "learned", "train"])
    rel = rng.choice([1e-4, 1e-3, 1e-2])
    if kind == "batch":
        return {"kind": kind, "n2": rng.randint(1, 40), "n3": rng.randint(0, 16), "lo2": 40,
                "hi2": _log_int(rng, 200, 1500), "lo3": 16, "hi3": _log_int(rng, 40, 160),
                "shapes_seed": rng.randint(0, 1 << 20), "merged": rng.random() < 0.5}
    if kind == "train":
        return {"kind": kind, "shape": _draw_shape(rng, 3, hi3=128), "rel": rel}
    ndim = 3 if kind == "learned" else rng.choice([2, 3])
    case = {"kind": kind, "field": "grf", "shape": _draw_shape(rng, ndim, hi3=200 if kind == "learned" else 288)}
    if kind != "labels":
        case["rel"] = rel
    if kind in ("fix", "learned"):
        case["merged"] = rng.random() < 0.5
    return case


# ------------------------------------------------------------------ inputs ---

def _shape(case) -> tuple:
    return tuple(int(s) for s in case["shape"].split("x"))


def _generator(seed: int) -> torch.Generator:
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) & 0x7FFFFFFF)
    return gen


def _normalised(a: torch.Tensor) -> torch.Tensor:
    lo, hi = a.min(), a.max()
    return ((a - lo) / (hi - lo)).float().contiguous()


def _random_field(shape, gen: torch.Generator) -> torch.Tensor:
    """A float32 field in [0, 1] with a power spectrum ~ k^-3 (2D) or k^-11/3
    (3D): the corner of a power-of-two box of filtered white noise."""
    box = [max(16, 1 << (int(s) - 1).bit_length()) for s in shape]
    spec = torch.fft.rfftn(torch.randn(box, generator=gen, device="cuda"))
    k2 = torch.zeros((), device="cuda")
    for ax, n in enumerate(box):
        k = torch.fft.rfftfreq(n, device="cuda") if ax == len(box) - 1 else torch.fft.fftfreq(n, device="cuda")
        k2 = k2 + (k * k).reshape([-1 if a == ax else 1 for a in range(len(box))])
    power = 3.0 if len(shape) == 2 else 11.0 / 3.0
    amp = torch.where(k2 > 0, k2.clamp_min(1e-30) ** (-power / 4.0), torch.zeros_like(k2))
    out = torch.fft.irfftn(spec * amp, s=box)
    return _normalised(out[tuple(slice(0, int(s)) for s in shape)])


def _bumps(shape, gen: torch.Generator) -> torch.Tensor:
    """32 Gaussian bumps of random centre, width and amplitude, with weak noise."""
    ny, nx = shape
    u = torch.rand((32, 4), generator=gen, device="cuda")
    x = torch.arange(nx, device="cuda", dtype=torch.float32)
    y = torch.arange(ny, device="cuda", dtype=torch.float32)
    s = 3.0 + 12.0 * u[:, 2:3]
    gx = torch.exp(-0.5 * ((x[None, :] - nx * u[:, 0:1]) / s) ** 2)
    gy = torch.exp(-0.5 * ((y[None, :] - ny * u[:, 1:2]) / s) ** 2)
    f = ((2.0 * u[:, 3:4] - 1.0)[:, :, None] * gy[:, :, None] * gx[:, None, :]).sum(0)
    return (f + 1e-3 * torch.randn(shape, generator=gen, device="cuda")).contiguous()


def _bound(f: torch.Tensor, rel: float) -> float:
    return float(np.float32(rel * (float(f.max()) - float(f.min()))))


def _decompressed(f: torch.Tensor, xi: float) -> torch.Tensor:
    """A uniform quantiser's output, within xi of f everywhere."""
    d = f.double()
    h = (2.0 * xi * torch.round(d / (2.0 * xi))).float()
    for _ in range(4):
        e = d - h.double()
        h = torch.where(e < -xi, torch.nextafter(h, torch.full_like(h, -math.inf)), h)
        h = torch.where(e > xi, torch.nextafter(h, torch.full_like(h, math.inf)), h)
    return h.contiguous()


def _pair(case, gen):
    shape = _shape(case)
    f = _bumps(shape, gen) if case.get("field") == "bumps" else _random_field(shape, gen)
    xi = _bound(f, case["rel"])
    return f, _decompressed(f, xi), xi


def _batch_shapes(case) -> list:
    rng = random.Random(case["shapes_seed"])
    out = []
    for _ in range(case["n2"]):
        out.append(((rng.randint(case["lo2"], case["hi2"]), rng.randint(case["lo2"], case["hi2"])),
                    rng.choice([1e-4, 1e-3, 1e-2])))
    for _ in range(case["n3"]):
        s = rng.randint(case["lo3"], case["hi3"])
        out.append(((s, s, s), rng.choice([1e-4, 1e-3, 1e-2])))
    return out


def _bytes(n: int) -> torch.Tensor:
    return torch.empty(n, dtype=torch.uint8, device="cuda")


def _train_inputs(case, seed):
    """Parameters, features and target as a training step meets them: the
    continuous channels of a quantised field, sparse flags, a target that is
    zero at most vertices."""
    gen = _generator(seed)
    f, fh, xi = _pair(case, gen)
    n = f.numel()

    def box_mean(a):
        pool = torch.nn.functional.avg_pool3d
        return pool(a[None, None], 3, 1, 1, count_include_pad=False)[0, 0]

    chans = [((fh - box_mean(fh)) / xi).clamp(-8, 8), torch.full_like(f, math.log10(case["rel"]) / 4 + 1)]
    for share in (0.002, 0.02, 0.001, 0.02):
        chans.append((torch.rand(f.shape, generator=gen, device="cuda") < share).float())
    chans += [((fh - f) / xi).clamp(-8, 8), ((f - box_mean(f)) / xi).clamp(-8, 8)]
    for share in (0.02, 0.001, 0.1, 0.1):
        chans.append((torch.rand(f.shape, generator=gen, device="cuda") < share).float())
    chans += [torch.zeros_like(f)] * 4
    feat = torch.stack([c.reshape(-1) for c in chans], 1).to(torch.bfloat16).contiguous()
    target = (torch.rand(n, generator=gen, device="cuda") < 0.05).float()
    return train_net.load_weights(), feat, target


# ------------------------------------------------------------------- cases ---

def prepare(case, seed) -> dict:
    kind = case["kind"]
    st = {"case": case, "kind": kind}
    if kind == "train":
        params, feat, target = _train_inputs(case, seed)
        st.update(params=params, feat=feat.view(torch.int16), target=target, shape=_shape(case),
                  grad=torch.empty_like(params), ws=_bytes(msz.net_workspace_bytes(_shape(case))))
        return st
    gen = _generator(seed)
    if kind == "batch":
        fields = []
        for shape, rel in _batch_shapes(case):
            f = _random_field(shape, gen)
            xi = _bound(f, rel)
            fields.append((f, _decompressed(f, xi), xi))
        # every field's edits in one array, its edited values in another (each
        # field's part starts on a 256-byte boundary)
        at = [0]
        for f, _, _ in fields:
            at.append(at[-1] + (f.numel() + 63) // 64 * 64)
        edits, g = torch.zeros(at[-1], device="cuda"), torch.zeros(at[-1], device="cuda")
        outs = [tuple(a[o:o + f.numel()].view(f.shape) for a in (edits, g)) for o, (f, _, _) in zip(at, fields)]
        st.update(fields=fields, edits=edits, g=g, outs=outs,
                  ws=_bytes(msz.batch_workspace_bytes([f.shape for f, _, _ in fields])))
        return st
    if kind == "labels":
        st["f"] = _random_field(_shape(case), gen)
        return st
    f, fh, xi = _pair(case, gen)
    st.update(f=f, fh=fh, xi=xi)
    if kind == "count":
        return st
    if kind == "learned":
        st.update(params=train_net.load_weights(), p_min=train_net.stored_p_min(),
                  ws=_bytes(msz.learned_workspace_bytes(f.shape)))
    else:
        st["ws"] = _bytes(msz.workspace_bytes(f.shape))
    st.update(edits=torch.empty_like(f), g=torch.empty_like(f))
    if kind in ("encode", "decode"):
        rc, edits, _, _ = msz.fix(f, fh, xi, workspace=st["ws"], edits_out=st["edits"], g_out=st["g"])
        if rc not in (msz.OK, msz.ESTALL):  # a stalled correction still has its edits
            raise RuntimeError(msz.strerror(rc))
        st["blob"] = _bytes(max(16, msz.edits_bound(edits.numel()))).zero_()
        if kind == "decode":
            rc, blob, _ = msz.encode_edits(edits, out=st["blob"])
            if rc != msz.OK:
                raise RuntimeError(msz.strerror(rc))
            st.update(blob=blob.clone(), shape=tuple(f.shape))
        for key in ("f", "fh", "g", "ws"):
            del st[key]
    return st


def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "fix":
        rc, edits, g, stats = msz.fix(st["f"], st["fh"], st["xi"], workspace=st["ws"], edits_out=st["edits"],
                                      g_out=st["g"], merged=case["merged"])
        return {"rc": rc, "edits": edits, "g": g, "stats": stats}
    if kind == "learned":
        rc, edits, g, stats = msz.fix_learned(st["f"], st["fh"], st["xi"], st["params"], p_min=st["p_min"],
                                              workspace=st["ws"], edits_out=st["edits"], g_out=st["g"],
                                              merged=case["merged"])
        return {"rc": rc, "edits": edits, "g": g, "stats": stats}
    if kind == "batch":
        rc, res = msz.fix_batch(st["fields"], workspace=st["ws"], outs=st["outs"], merged=case["merged"])
        stats = np.array([[*d["rounds"], *d["false_init"], d["rounds_r"], d["outer_iters"], d["n_edited"],
                           d["mislabel_init"], d["n_inexact"], d["status"]] for _, _, _, d in res], dtype=np.int64)
        return {"rc": rc, "edits": st["edits"], "g": st["g"], "stats": stats}
    if kind == "labels":
        return msz.labels(st["f"])
    if kind == "count":
        return msz.count_false(st["f"], st["fh"])
    if kind == "encode":
        rc, _, stats = msz.encode_edits(st["edits"], out=st["blob"])
        return {"rc": rc, "blob": st["blob"], "stats": stats}  # the stream fills the first stats["bytes"] bytes
    if kind == "decode":
        rc, edits = msz.decode_edits(st["blob"], st["shape"], out=st["edits"])
        return {"rc": rc, "edits": edits}
    loss, grad = msz.net_gradients(st["params"], st["feat"], st["target"], st["shape"], edit_weight=16.0,
                                   grad_out=st["grad"], workspace=st["ws"])
    return {"loss": loss, "grad": grad}


_EDITED = {1e-4: 0.01, 1e-3: 0.09, 1e-2: 0.3}  # share of vertices that a correction edits, about


def work(case) -> dict:
    kind = case["kind"]
    if kind == "batch":
        return {"bytes": 16 * sum(math.prod(s) for s, _ in _batch_shapes(case)), "flops": 0}
    n = math.prod(_shape(case))
    layers = (27 * 16 * 16, 27 * 16 * 16, 27 * 16)
    if kind == "fix":
        return {"bytes": 16 * n, "flops": 0}
    if kind == "labels":
        return {"bytes": 12 * n, "flops": 0}
    if kind == "count":
        return {"bytes": 8 * n, "flops": 0}
    if kind in ("encode", "decode"):
        return {"bytes": int(4 * n + 4 * _EDITED[case["rel"]] * n), "flops": 0}
    if kind == "learned":
        return {"bytes": 16 * n, "flops": 2 * n * sum(layers)}
    # forward, weight gradients of all layers, data gradients of all but the first
    return {"bytes": 36 * n, "flops": 2 * n * (2 * sum(layers) + layers[1] + layers[2])}


def exact(case, seed):
    """The loss and gradients in 64 bits; every other output is defined by
    float32 operations, or is a whole number or bytes."""
    if case["kind"] != "train":
        return None
    params, feat, target = _train_inputs(case, seed)
    shape, n = _shape(case), target.numel()
    p = params.double().requires_grad_(True)
    sizes = (27 * 256, 16, 27 * 256, 16, 27 * 16, 1)
    w0, b0, w1, b1, w2, b2 = torch.split(p, sizes)

    def conv(x, w, b):
        pad = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
        out = b
        for tap in range(27):
            dz, dy, dx = tap // 9, (tap // 3) % 3, tap % 3
            out = out + pad[dz:dz + shape[0], dy:dy + shape[1], dx:dx + shape[2]].reshape(n, -1) @ w[tap]
        return out.reshape(*shape, -1)

    x = feat.double().reshape(*shape, 16)
    h = torch.relu(conv(x, w0.reshape(27, 16, 16), b0))
    h = torch.relu(conv(h, w1.reshape(27, 16, 16), b1))
    y = conv(h, w2.reshape(27, 16, 1), b2).reshape(-1)
    t = target.double()
    loss = ((1.0 + 16.0 * (t > 0)) * (y - t) ** 2).mean()
    grad, = torch.autograd.grad(loss, p)
    return {"loss": float(loss.detach()), "grad": grad}
