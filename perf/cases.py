"""The work that a user has this framework do, as cases that can be timed and compared.

Six kinds of call, through the package's public entry points:

    infer         ntbc.Model.infer            one material's (or a region's) BC blocks from its network
    batch         ntbc.Batch.run              load-time decode of several materials with their mip chains
    train         ntbc.Trainer.step           one training step of a material's network
    paper_infer   ntbc.FaithfulModel.infer    blocks from the paper's own two-network layout
    paper_train   ntbc.FaithfulTrainer.step   one training step of that layout
    codec         ntbc.encode_ref, decode, block_sse and fallback: the reference encode of every texture,
                  the decode of its blocks, and the per-block judge

Formats are one letter a texture: "c" a three-channel BC1 texture, "s" a single-channel BC4 one.  A
training case is a step from the last tenth of its schedule, with warm Adam moments.
"""
import math

import torch
import torch.nn.functional as F

from paper_2407_09543_amd import ntbc

_PRECISION = {"fp32": ntbc.FP32, "bf16": ntbc.BF16, "fp16": ntbc.FP16}


def listed():
    paper = {"levels": 8, "feats": 8, "hidden": 256, "n_hidden": 3, "formats": "ccsss"}
    mid = {"levels": 6, "feats": 8, "hidden": 128, "n_hidden": 3, "formats": "ccsss"}
    small = {"levels": 4, "feats": 4, "hidden": 64, "n_hidden": 2, "formats": "cs"}
    return [
        # the decode of a whole 4096^2 five-texture material when it is loaded: the headline workload
        {"name": "infer 4096 bf16", "kind": "infer", "w": 4096, "h": 4096, "u8": True, "precision": "bf16",
         "first": 0, "count": 1024 * 1024, "heads": False, **paper},
        # the smallest material, a 256^2 pair of textures with a float grid: launches and latency
        {"name": "infer 256 bf16", "kind": "infer", "w": 256, "h": 256, "u8": False, "precision": "bf16",
         "first": 0, "count": 64 * 64, "heads": False, **small},
        # an ordinary 1024^2 material in the paper's network precision
        {"name": "infer 1024 fp16", "kind": "infer", "w": 1024, "h": 1024, "u8": True, "precision": "fp16",
         "first": 0, "count": 256 * 256, "heads": False, **mid},
        # a ragged region of a four-texture material streamed with its predicted heads
        {"name": "infer region heads", "kind": "infer", "w": 2000, "h": 1100, "u8": True, "precision": "bf16",
         "first": 12345, "count": 37001, "heads": True, **{**mid, "formats": "cssc"}},
        # the accuracy reference: FP32 inference of a 2048^2 material
        {"name": "infer 2048 fp32", "kind": "infer", "w": 2048, "h": 2048, "u8": True, "precision": "fp32",
         "first": 0, "count": 512 * 512, "heads": False, **paper},
        # a scene's materials with full mip chains, decoded at load time
        {"name": "batch 6 materials", "kind": "batch", "materials": 6, "size": 512, "precision": "bf16"},
        # the encode's inner loop at the paper's scale
        {"name": "train 4096 bf16", "kind": "train", "w": 4096, "h": 4096, "batch": 65536, "precision": "bf16",
         "qat": False, "deterministic": False, **paper},
        # an FP32 step (the encode's default products) with the 8-bit grid in the loop
        {"name": "train 1024 fp32 qat", "kind": "train", "w": 1024, "h": 1024, "batch": 16384, "precision": "fp32",
         "qat": True, "deterministic": False, **mid},
        # the smallest training step: latency and launches
        {"name": "train 256 bf16", "kind": "train", "w": 256, "h": 256, "batch": 512, "precision": "bf16",
         "qat": False, "deterministic": False, **small},
        # the paper's inference table: a 4096^2 material of two BC1 and four BC4 textures, one model
        {"name": "paper infer 4096", "kind": "paper_infer", "w": 4096, "h": 4096, "u8": True, "formats": "ccssss"},
        # a training step of that layout
        {"name": "paper train 4096", "kind": "paper_train", "w": 4096, "h": 4096, "batch": 65536, "qat": False,
         "formats": "ccssss"},
        # the targets of an encode, their decode and the judge
        {"name": "codec 2048", "kind": "codec", "w": 2048, "h": 2048, "formats": "ccsss"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _four(rng, lo, hi):
    return 4 * _log(rng, lo // 4, hi // 4)


def _mix(rng, most):
    """A material's textures: up to two colour ones and up to `most` in all, as materials have them."""
    n = rng.randint(1, most)
    c = rng.randint(0 if n < 3 else 1, min(2, n))
    return "c" * c + "s" * (n - c)


def draw(rng):
    kind = rng.choice(["infer", "infer", "infer", "batch", "train", "train", "train", "paper_infer", "paper_train",
                       "codec"])
    if kind == "batch":
        return {"kind": kind, "materials": rng.randint(2, 6), "size": 4 * _log(rng, 32, 128),
                "precision": rng.choice(["bf16", "fp16"])}
    if kind == "codec":
        return {"kind": kind, "w": _four(rng, 64, 4096), "h": _four(rng, 64, 2048), "formats": _mix(rng, 5)}
    case = {"kind": kind, "w": _four(rng, 256, 4096), "h": _four(rng, 256, 4096)}
    if kind == "paper_infer":
        return {**case, "u8": rng.random() < 0.7, "formats": _mix(rng, 6)}
    if kind == "paper_train":
        return {**case, "batch": _log(rng, 1024, 65536), "qat": rng.random() < 0.3, "formats": _mix(rng, 6)}
    hidden = rng.choice([64, 128, 256])
    case.update(levels=rng.randint(4, 8 if min(case["w"], case["h"]) >= 1024 else 6), feats=rng.choice([4, 8]),
                hidden=hidden, n_hidden=rng.choice([2, 3, 3]), formats=_mix(rng, 5))
    if kind == "train":
        return {**case, "batch": _log(rng, 512, 65536), "precision": rng.choice(["bf16", "bf16", "fp32"]),
                "qat": rng.random() < 0.3, "deterministic": rng.random() < 0.2}
    case.update(u8=rng.random() < 0.7, precision=rng.choice(["bf16", "bf16", "fp16", "fp32"]))
    if case["precision"] == "fp32":
        case["w"], case["h"] = max(256, case["w"] // 8 * 4), max(256, case["h"] // 8 * 4)
    total = (case["w"] // 4) * (case["h"] // 4)
    first = rng.choice([0, 0, rng.randrange(total // 2)])
    count = total - first if first == 0 else rng.randint(1, total - first)
    return {**case, "first": first, "count": count, "heads": count <= 1 << 16 and rng.random() < 0.3}


# --------------------------------------------------------------------------------------------- sizes
def _formats(case):
    return [ntbc.BC1 if f == "c" else ntbc.BC4 for f in case["formats"]]


def _heads(formats):
    """(endpoint values, colour channels) of a block."""
    return sum(6 if f == "c" else 2 for f in formats), sum(3 if f == "c" else 1 for f in formats)


def _dims(case):
    e, c = _heads(case["formats"])
    return [case["levels"] * case["feats"]] + [case["hidden"]] * case["n_hidden"] + [e + 16 * c]


def _vertices(levels, base=8):
    return sum((base << l) ** 2 for l in range(levels))


def _macs(dims):
    return sum(i * o for i, o in zip(dims, dims[1:]))


def _params(dims):
    return sum((i + 1) * o for i, o in zip(dims, dims[1:]))


def _batch_models(case):
    """(width, size, formats) of every material of a load-time decode."""
    return [(64 << (m // 2 % 3), case["size"] << (m % 3), "cc" + "s" * (1 + m % 3)) for m in range(case["materials"])]


def _mips(n_w, n_h):
    sizes = []
    while n_w >= 1 and n_h >= 1:
        sizes.append((n_w, n_h))
        n_w, n_h = n_w // 2, n_h // 2
    return sizes


def work(case):
    """Bytes and operations of one pass: every input read once, every output written once."""
    kind = case["kind"]
    if kind == "infer":
        dims, v = _dims(case), _vertices(case["levels"]) * case["feats"]
        n, nt = case["count"], len(case["formats"])
        total = (case["w"] // 4) * (case["h"] // 4)
        grid = v * (1 if case["u8"] else 4) * n / total
        return {"bytes": grid + 4 * _params(dims) + 8 * n * nt + (4 * n * dims[-1] if case["heads"] else 0),
                "flops": 2 * _macs(dims) * n}
    if kind == "batch":
        b = f = 0
        for width, size, formats in _batch_models(case):
            dims = [64] + [width] * 3 + [_heads(formats)[0] + 16 * _heads(formats)[1]]
            n = sum(a * c for a, c in _mips(size // 4, size // 4))
            b += _vertices(8) * 8 + 4 * _params(dims) + 8 * n * len(formats)
            f += 2 * _macs(dims) * n
        return {"bytes": b, "flops": f}
    if kind == "train":
        dims, n = _dims(case), case["batch"]
        p = _vertices(case["levels"]) * case["feats"] + _params(dims)
        texels = 16 * _heads(case["formats"])[1] + 8 * len(case["formats"])
        # parameters and moments read and written, gradients written; three products a layer
        return {"bytes": 28 * p + n * (4 + texels), "flops": 6 * _macs(dims) * n}
    e, c = _heads(case["formats"])
    n_pos = (case["w"] // 4) * (case["h"] // 4)
    if kind in ("paper_infer", "paper_train"):
        ep, col = [14, 64, 64, 64, e], [16, 64, 64, 64, c]
        v = 2 * (_vertices(7, 16) + _vertices(8, 16))
        if kind == "paper_infer":
            return {"bytes": v * (1 if case["u8"] else 4) + 4 * (_params(ep) + _params(col)) + 8 * n_pos * len(case["formats"]),
                    "flops": 2 * (_macs(ep) + 16 * _macs(col)) * n_pos}
        n = case["batch"]
        return {"bytes": 28 * (v + _params(ep) + _params(col)) + n * (4 + 16 * c + 8 * len(case["formats"])),
                "flops": 6 * (_macs(ep) + 16 * _macs(col)) * n}
    # encode: texels in, words out; decode: words in, texels out; two errors a block; the judge
    nt = len(case["formats"])
    return {"bytes": n_pos * (16 * c * 3 + nt * (8 + 8 + 8 + 8 + 4 + 8 + 8 + 4 + 4 + 8)), "flops": 0}


# -------------------------------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _noise(gen, n, h, w, octaves=6):
    """n smooth fields [n, h, w] in (0, 1): octaves of bilinear value noise."""
    out, total = torch.zeros((n, h, w), device="cuda"), 0.0
    for o in range(octaves):
        r = 8 << o
        lat = torch.rand((1, n, min(r, h), min(r, w)), generator=gen, device="cuda")
        out += 0.5 ** o * F.interpolate(lat, size=(h, w), mode="bilinear", align_corners=False)[0]
        total += 0.5 ** o
    return out / total


def _textures(gen, case):
    """Correlated textures of a material from one height field: uint8 [h, w, 3] or [h, w]."""
    h, w = case["h"], case["w"]
    height = _noise(gen, 1, h, w)[0]
    out = []
    for k, f in enumerate(case["formats"]):
        if f == "c":
            x = 0.7 * height[..., None] * torch.rand(3, generator=gen, device="cuda") + \
                0.4 * _noise(gen, 3, h, w, 4 + k % 3).permute(1, 2, 0)
        else:
            x = 1.4 * (0.6 * height + 0.4 * _noise(gen, 1, h, w, 3 + k % 4)[0]) - 0.2
        out.append((x.clamp(0, 1) * 255 + 0.5).to(torch.uint8).contiguous())
    return out


def _blocks(tex):
    """[blocks, 16, channels] of a texture."""
    t = tex if tex.dim() == 3 else tex[..., None]
    h, w, c = t.shape
    return t.reshape(h // 4, 4, w // 4, 4, c).permute(0, 2, 1, 3, 4).reshape(-1, 16, c)


def _box_words(tex):
    """BC words whose endpoints are each block's value range (codes zero): targets of a training step.
    A quarter of the single-channel blocks take the six-value order."""
    b = _blocks(tex).to(torch.int64)
    hi, lo = b.amax(1), b.amin(1)
    if b.shape[2] == 3:
        q = torch.tensor([31, 63, 31], device=b.device)
        sh = torch.tensor([11, 5, 0], device=b.device)
        return (((hi * q + 127) // 255) << sh).sum(1) | ((((lo * q + 127) // 255) << sh).sum(1) << 16)
    hi, lo = hi[:, 0], lo[:, 0]
    six = torch.arange(len(hi), device=b.device) % 4 == 0
    return torch.where(six, lo | (hi << 8), hi | (lo << 8))


def _net(gen, dims, gain=2.0):
    """He-normal weights and small biases in the canonical flat layout."""
    parts = []
    for i, o in zip(dims, dims[1:]):
        parts.append(torch.randn(o * i, generator=gen, device="cuda") * math.sqrt(gain / i))
        parts.append(0.1 * torch.randn(o, generator=gen, device="cuda"))
    return torch.cat(parts)


def _u8_grid(gen, levels, base, feats):
    v = _vertices(levels, base)
    return (torch.randint(0, 256, (v, feats), dtype=torch.uint8, generator=gen, device="cuda"),
            torch.full((levels,), 0.7 / 128, device="cuda"), torch.full((levels,), 128, dtype=torch.int32, device="cuda"))


def _f32_grid(gen, levels, base, feats):
    return 0.4 * torch.randn((_vertices(levels, base), feats), generator=gen, device="cuda")


def _ids(gen, n, total):
    return torch.randint(0, total, (n,), dtype=torch.int32, generator=gen, device="cuda")


def _warm(gen, m, v, scale):
    """Adam moments of a run under way."""
    for a, b in zip(m, v):
        a.copy_(0.3 * scale * torch.randn(a.shape, generator=gen, device="cuda"))
        b.copy_((scale * (0.5 + torch.rand(b.shape, generator=gen, device="cuda"))) ** 2)


_STEPS = 22000  # a schedule's length; the steps timed here begin at _AT
_AT = 21900


def _model(gen, case):
    desc = ntbc.make_desc(case["levels"], 8, case["feats"], case["u8"], case["hidden"], case["n_hidden"], _formats(case),
                          case["w"] // 4, case["h"] // 4)
    weights = _net(gen, _dims(case))
    if case["u8"]:
        return ntbc.Model(desc, weights, *_u8_grid(gen, case["levels"], 8, case["feats"]))
    return ntbc.Model(desc, weights, _f32_grid(gen, case["levels"], 8, case["feats"]))


def _train_inputs(gen, case):
    tex = _textures(gen, case)
    words = torch.stack([_box_words(t) for t in tex])
    return tex, words, _ids(gen, case["batch"], words.shape[1])


def _prepare_train(gen, case):
    tex, words, ids = _train_inputs(gen, case)
    desc = ntbc.make_desc(case["levels"], 8, case["feats"], False, case["hidden"], case["n_hidden"], _formats(case),
                          case["w"] // 4, case["h"] // 4)
    tr = ntbc.Trainer(desc, _f32_grid(gen, case["levels"], 8, case["feats"]), _net(gen, _dims(case), 1.0),
                      ntbc.Targets(words, tex), case["batch"], _STEPS, precision=_PRECISION[case["precision"]],
                      deterministic=case["deterministic"])
    _warm(gen, (tr.m_grid, tr.m_w), (tr.v_grid, tr.v_w), 1e-3)
    return {"kind": "train", "trainer": tr, "ids": ids, "at": _AT, "qat": case["qat"]}


def _paper_inputs(gen, case, grid):
    e, c = _heads(case["formats"])
    return grid(gen, 7, 16, 2), grid(gen, 8, 16, 2), _net(gen, [14, 64, 64, 64, e], 1.0), _net(gen, [16, 64, 64, 64, c], 1.0)


def prepare(case, seed):
    gen, kind = _gen(seed), case["kind"]
    if kind == "infer":
        return {"kind": kind, "model": _model(gen, case), "precision": _PRECISION[case["precision"]],
                "first": case["first"], "count": case["count"], "heads": case["heads"]}
    if kind == "batch":
        entries = []
        for width, size, formats in _batch_models(case):
            m = _model(gen, {"levels": 8, "feats": 8, "hidden": width, "n_hidden": 3, "formats": formats, "u8": True,
                             "w": size, "h": size})
            for level, (bw, bh) in enumerate(_mips(size // 4, size // 4)):
                entries.append((m, ntbc.mip_desc(m.desc, level), 0, bw * bh))
        return {"kind": kind, "batch": ntbc.Batch(entries, _PRECISION[case["precision"]])}
    if kind == "train":
        return _prepare_train(gen, case)
    if kind == "paper_infer":
        eg, cg, ew, cw = _paper_inputs(gen, case, _u8_grid if case["u8"] else lambda *a: (_f32_grid(*a), None, None))
        return {"kind": kind, "model": ntbc.FaithfulModel(
            _formats(case), case["w"] // 4, case["h"] // 4, eg[0], cg[0], ew, cw, ep_scale=eg[1], ep_zero=eg[2],
            col_scale=cg[1], col_zero=cg[2])}
    if kind == "paper_train":
        tex, words, ids = _train_inputs(gen, case)
        tr = ntbc.FaithfulTrainer(_formats(case), case["w"] // 4, case["h"] // 4, *_paper_inputs(gen, case, _f32_grid),
                                  ntbc.Targets(words, tex), case["batch"], _STEPS)
        _warm(gen, tr.m, tr.v, 1e-3)
        return {"kind": kind, "trainer": tr, "ids": ids, "at": _AT, "qat": case["qat"]}
    tex = _textures(gen, case)
    # the network's blocks that the judge looks at: each block's value range with random codes
    words = [_box_words(t) | (torch.randint(0, 1 << 32, (t.shape[0] * t.shape[1] // 16,), generator=gen, device="cuda")
                              << 32) for t in tex]
    return {"kind": kind, "w": case["w"], "h": case["h"], "formats": _formats(case), "textures": tex, "words": words}


# ---------------------------------------------------------------------------------------------- runs
def run(state):
    kind = state["kind"]
    if kind == "infer":
        return state["model"].infer(state["precision"], state["first"], state["count"], heads=state["heads"])
    if kind == "batch":
        return state["batch"].run()
    if kind == "paper_infer":
        return state["model"].infer()
    if kind in ("train", "paper_train"):
        tr = state["trainer"]
        losses = tr.step(state["ids"], state["at"], qat=state["qat"])
        state["at"] = min(state["at"] + 1, _STEPS - 1)
        if kind == "train":
            return {"losses": losses, "d_grid": tr.d_grid, "d_weights": tr.d_w, "grid": tr.grid, "weights": tr.weights,
                    "m_grid": tr.m_grid, "m_weights": tr.m_w, "v_grid": tr.v_grid, "v_weights": tr.v_w}
        return {"losses": losses, "grads": tr.grads, "params": tr.params, "m": tr.m, "v": tr.v}
    out = []
    for tex, words, f in zip(state["textures"], state["words"], state["formats"]):
        ref = ntbc.encode_ref(tex, f)
        judged, replaced = ntbc.fallback(words, ref, ntbc.block_sse(words, tex, f), ntbc.block_sse(ref, tex, f), 4.0, 0.0)
        out.append((ref, judged, replaced, ntbc.decode(judged, state["w"], state["h"], f)))
    return out


# --------------------------------------------------------------------------------------------- exact
def _levels(grid, levels, base):
    out, at = [], 0
    for l in range(levels):
        r = base << l
        out.append(grid[at:at + r * r].reshape(r, r, -1))
        at += r * r
    return out


def _corner(b, blocks, res):
    p = ((2 * b + 1) * res - blocks).double() / (2 * blocks)
    p = p.clamp(0, res - 1)
    i = p.floor().clamp(max=res - 2)
    return i.long(), (p - i)[:, None]


def _features(grid, levels, base, x, y, n_w, n_h):
    out = []
    for g in _levels(grid, levels, base):
        i, fx = _corner(x, n_w, g.shape[0])
        j, fy = _corner(y, n_h, g.shape[0])
        out.append((1 - fx) * (1 - fy) * g[j, i] + fx * (1 - fy) * g[j, i + 1] + (1 - fx) * fy * g[j + 1, i] +
                   fx * fy * g[j + 1, i + 1])
    return torch.cat(out, 1)


def _mlp(flat, dims, x, act):
    at = 0
    for k, (i, o) in enumerate(zip(dims, dims[1:])):
        w, b = flat[at:at + i * o].reshape(o, i), flat[at + i * o:at + i * o + o]
        at += i * o + o
        x = x @ w.t() + b
        x = act(x) if k < len(dims) - 2 else torch.sigmoid(x)
    return x


def _fake_quant(grid, levels, base):
    """The grid through its 8-bit codes (float32 decisions, as the codes are stored) with the
    straight-through gradient."""
    out = []
    for g in _levels(grid, levels, base):
        v = g.detach().float()
        lo, hi = v.min().clamp(max=0.0), v.max().clamp(min=0.0)
        s = (hi - lo) / 255 if hi > lo else torch.ones_like(hi)
        z = torch.round(-lo / s).clamp(0, 255)
        t = torch.round(v / s) + z
        q = s.double() * (t.clamp(0, 255) - z).double()
        keep = ((t >= 0) & (t <= 255)).double()
        out.append((q + keep * (g - g.detach())).reshape(-1, g.shape[2]))
    return torch.cat(out)


def _palette(e0, e1, eight):
    """Palettes [n, N, channels] between two endpoints; eight: None for three channels, else the mode."""
    if eight is None:
        w = torch.arange(4, device=e0.device, dtype=torch.float64)[None, :, None] / 3
        return (1 - w) * e0[:, None] + w * e1[:, None]
    w = torch.arange(8, device=e0.device, dtype=torch.float64)[None, :, None] / 7
    p8 = (1 - w) * e0[:, None] + w * e1[:, None]
    w = torch.arange(6, device=e0.device, dtype=torch.float64)[None, :, None] / 5
    p6 = (1 - w) * e0[:, None] + w * e1[:, None]
    p6 = torch.cat([torch.zeros_like(p6[:, :1]), p6, torch.ones_like(p6[:, :1])], 1)
    return torch.where(eight[:, None, None], p8, p6)


def _chosen(delta, ref, c, count):
    """The decoded-colour loss: hard choice in the value, softmax expectation in the gradient."""
    sq = (delta ** 2).sum(-1)
    norm = torch.where(sq > 0, sq, torch.ones_like(sq)).sqrt() * (sq > 0)
    k = norm.argmin(2)
    x = torch.gather(ref[:, None].expand(-1, 16, -1, -1), 2, k[:, :, None, None].expand(-1, -1, 1, ref.shape[2]))[:, :, 0]
    soft = (torch.softmax(-norm / 0.01, 2)[..., None] * ref[:, None]).sum(2)
    value = ((x - c) ** 2).sum() / count
    through = (2 * (x - c) / count * soft).sum()
    return value.detach(), through


def _loss(y, tex, words, ids, formats):
    """(four losses, a sum whose gradient is the training gradient) of the heads y."""
    e_dim, c_dim = _heads(formats)
    n = y.shape[0]
    e_hat, c_hat = y[:, :e_dim], y[:, e_dim:].reshape(n, 16, c_dim)
    count = n * 16 * c_dim
    sums, through, e, c = [0.0] * 4, 0.0, 0, 0
    for f, t, w in zip(formats, tex, words):
        ch = 3 if f == "c" else 1
        col, w = _blocks(t)[ids].double() / 255, w[ids]
        if f == "c":
            def expand(v):
                r, g, b = (v >> 11) & 31, (v >> 5) & 63, v & 31
                return torch.stack([(r << 3) | (r >> 2), (g << 2) | (g >> 4), (b << 3) | (b >> 2)], 1).double() / 255
            r0, r1, mode = expand(w & 0xFFFF), expand((w >> 16) & 0xFFFF), None
        else:
            r0, r1 = ((w & 255).double() / 255)[:, None], (((w >> 8) & 255).double() / 255)[:, None]
            mode = (w & 255) > ((w >> 8) & 255)
        h0, h1, hat = e_hat[:, e:e + ch], e_hat[:, e + ch:e + 2 * ch], c_hat[:, :, c:c + ch]
        ref = _palette(r0, r1, mode)
        pred = _palette(h0, h1, None if f == "c" else (h0 > h1)[:, 0])
        l_e = ((h0 - r0) ** 2).sum() / (n * e_dim) + ((h1 - r1) ** 2).sum() / (n * e_dim)
        l_c = ((hat - col) ** 2).sum() / count
        v_e, t_e = _chosen(col[:, :, None] - pred[:, None], ref, col, count)
        v_c, t_c = _chosen(hat[:, :, None] - ref[:, None], ref, col, count)
        for k, v in enumerate((l_e.detach(), l_c.detach(), v_e, v_c)):
            sums[k] = sums[k] + v
        through = through + l_e + l_c + t_e + t_c
        e, c = e + 2 * ch, c + ch
    return torch.stack(sums + [torch.zeros_like(sums[0])]), through


def _adam(p, g, m, v, lr0, step=_AT, warmup=10):
    lr = lr0 * 0.5 * (1 + math.cos(math.pi * (step - warmup) / (_STEPS - warmup)))
    m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
    return p - lr * (m / (1 - 0.9 ** (step + 1))) / ((v / (1 - 0.999 ** (step + 1))).sqrt() + 1e-15), m, v


def _exact_train(case, seed):
    s = prepare(case, seed)
    gen = _gen(seed)
    tex, words, ids = _train_inputs(gen, case)
    ids, bw, bh = ids.long(), case["w"] // 4, case["h"] // 4
    tr = s["trainer"]
    if case["kind"] == "train":
        start, m, v = [tr.grid, tr.weights], [tr.m_grid, tr.m_w], [tr.v_grid, tr.v_w]
    else:
        start, m, v = tr.params, tr.m, tr.v
    p = [t.double().requires_grad_(True) for t in start]
    through_q = _fake_quant if case["qat"] else lambda g, levels, base: g
    if case["kind"] == "train":
        x = _features(through_q(p[0], case["levels"], 8), case["levels"], 8, ids % bw, ids // bw, bw, bh)
        y = _mlp(p[1], _dims(case), x, torch.relu)
    else:
        e, c = _heads(case["formats"])
        x = _features(through_q(p[0], 7, 16), 7, 16, ids % bw, ids // bw, bw, bh)
        i = torch.arange(16, device="cuda")
        tx = (4 * (ids % bw)[:, None] + i % 4).reshape(-1)
        ty = (4 * (ids // bw)[:, None] + i // 4).reshape(-1)
        xc = _features(through_q(p[1], 8, 16), 8, 16, tx, ty, 4 * bw, 4 * bh)
        y = torch.cat([_mlp(p[2], [14, 64, 64, 64, e], x, torch.selu),
                       _mlp(p[3], [16, 64, 64, 64, c], xc, torch.selu).reshape(len(ids), 16 * c)], 1)
    losses, through = _loss(y, tex, words, ids, case["formats"])
    through.backward()
    grads = [t.grad for t in p]
    rates = (0.01, 0.005) if case["kind"] == "train" else (0.01, 0.01, 0.005, 0.005)
    new = [_adam(t.detach(), t.grad, a.double(), b.double(), lr) for t, a, b, lr in zip(p, m, v, rates)]
    np_, nm, nv = ([t[k] for t in new] for k in range(3))
    if case["kind"] == "train":
        return {"losses": losses, "d_grid": grads[0], "d_weights": grads[1], "grid": np_[0], "weights": np_[1],
                "m_grid": nm[0], "m_weights": nm[1], "v_grid": nv[0], "v_weights": nv[1]}
    return {"losses": losses, "grads": grads, "params": np_, "m": nm, "v": nv}


def exact(case, seed):
    """The floating results in 64 bits: a training step's, and the heads of an inference (the blocks
    are whole numbers, decided in float32)."""
    if case["kind"] in ("train", "paper_train"):
        return _exact_train(case, seed)
    if case["kind"] != "infer" or not case["heads"]:
        return None
    m = prepare(case, seed)["model"]
    grid = m.grid.double()
    if case["u8"]:
        scale, zero = m.grid_scale.double(), m.grid_zero.double()
        grid = torch.cat([(g.reshape(-1, case["feats"]) - z) * s
                          for g, s, z in zip(_levels(grid, case["levels"], 8), scale, zero)])
    ids = torch.arange(case["first"], case["first"] + case["count"], device="cuda")
    bw, bh = case["w"] // 4, case["h"] // 4
    x = _features(grid, case["levels"], 8, ids % bw, ids // bw, bw, bh)
    return None, _mlp(m.weights.double(), _dims(case), x, torch.relu)
