"""The cases that this library's speed is measured on.

Each case is one call (or one short sequence of calls) that a user of the
library makes through paper_2003_06513_amd.binding, with the sizes of the
networks that the paper prunes (VGG-16 and ResNet-50 at 224x224, ResNet-18 on
CIFAR), of a 512-channel sweep layer, and generic odd sizes:

  stack    the 13 pruned convolutions of VGG-16 with ReLU, and the four 2x2
           max-pools in the convolution calls
  conv     one pruned 3x3 layer, stride 1 or 2, with or without a 2x2 pool,
           a bias and ReLU
  retrain  the backward of one pruned layer: dx (the layer's transposed
           packing applied to dy), the masked weight gradient and db
  admm     one iteration of the data-free ADMM pruning of a dense layer
  prune    dense weights to packed ones: projection, connectivity, packing
"""
import math

import numpy as np
import torch

from paper_2003_06513_amd import binding as B

_DT = {"f32": torch.float32, "f16": torch.float16}
_CODE = {"f32": B.PSC_F32, "f16": B.PSC_F16}
_VGG = [(3, 64, 224), (64, 64, 224), (64, 128, 112), (128, 128, 112), (128, 256, 56), (256, 256, 56),
        (256, 256, 56), (256, 512, 28), (512, 512, 28), (512, 512, 28), (512, 512, 14), (512, 512, 14),
        (512, 512, 14)]
_VGG_POOLS = (1, 3, 6, 9)


def _case(kind, dtype, n, cin, cout, h, w, m, drop, stride=1, pool=False, bias=False, relu=False, name=None):
    c = {"kind": kind, "dtype": dtype, "n": n, "cin": cin, "cout": cout, "h": h, "w": w, "m": m, "drop": drop,
         "stride": stride, "pool": pool, "bias": bias, "relu": relu}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # inference of a whole pruned network on one image (the headline of bench.py)
        {"name": "vgg16_b1_f32", "kind": "stack", "n": 1, "size": 224, "m": 8},
        # one layer on one image, where the launch is a large part of the time
        _case("conv", "f16", 1, 256, 256, 14, 14, 8, 60, name="resnet50_256c_14_b1_f16"),
        # a serving batch in half precision: the large and the small planes of ResNet-50
        _case("conv", "f16", 32, 64, 64, 56, 56, 8, 60, name="resnet50_64c_56_b32_f16"),
        _case("conv", "f16", 32, 512, 512, 7, 7, 8, 60, name="resnet50_512c_7_b32_f16"),
        # the largest layer of the sweep over library sizes and drop ratios
        _case("conv", "f16", 64, 512, 512, 28, 28, 8, 60, name="sweep_512c_28_b64_f16"),
        # single precision at a large batch: a stride-1 layer of ResNet-18 and a stage entry
        _case("conv", "f32", 256, 128, 128, 16, 16, 6, 70, name="cifar_128c_16_b256_f32"),
        _case("conv", "f32", 256, 64, 128, 32, 32, 6, 70, stride=2, relu=True, name="cifar_entry128_32_b256_f32"),
        # no size a multiple of anything, as in detection and segmentation inputs
        _case("conv", "f32", 3, 93, 77, 45, 61, 12, 50, bias=True, relu=True, name="ragged_93_77_45x61_b3_f32"),
        # retraining the pruned layers
        _case("retrain", "f16", 32, 128, 128, 28, 28, 8, 60, name="retrain_128c_28_b32_f16"),
        _case("retrain", "f32", 256, 256, 256, 8, 8, 6, 70, name="retrain_256c_8_b256_f32"),
        # pruning: one ADMM iteration on a batch of 32, and the packing of a layer
        _case("admm", "f32", 32, 64, 64, 32, 32, 8, 50, name="admm_64c_32_T32"),
        _case("prune", "f32", 0, 512, 512, 0, 0, 8, 66, name="prune_512c_f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("conv", "retrain", "admm", "prune"), (8, 3, 1, 1))[0]
    m, drop = rng.choice((4, 6, 8, 12)), rng.choice((0, 40, 50, 60, 70, 80))
    if kind == "prune":
        return _case(kind, rng.choice(("f32", "f16")), 0, _log(rng, 16, 512), _log(rng, 16, 512), 0, 0, m, drop)
    # multiply-adds of the dense layer: the slowest shapes stay under the listed cases' time
    most = {"conv": 8e9, "retrain": 2e9, "admm": 1.5e9}[kind]
    while True:
        n, cin, cout = _log(rng, 1, 256), _log(rng, 3, 512), _log(rng, 16, 512)
        h = _log(rng, 4, 224)
        w = h if rng.random() < 0.6 else max(4, min(224, int(h * rng.uniform(0.6, 1.7))))
        if rng.random() < 0.4:    # the channel counts and sizes that networks use
            cin, cout = 2 ** max(4, round(math.log2(cin))), 2 ** round(math.log2(cout))
            h = w = min((4, 7, 8, 14, 16, 28, 32, 56, 112, 224), key=lambda s: abs(math.log(s / h)))
        if kind == "admm":
            n, h, w = 32, min(h, 56), min(w, 56)
        if 2e7 <= 9 * n * cin * cout * h * w <= most and n * max(cin, cout) * h * w <= 6e7:
            break
    dtype = "f32" if kind == "admm" else rng.choice(("f32", "f16"))
    c = _case(kind, dtype, n, cin, cout, h, w, m, drop)
    if kind == "conv":
        c["stride"] = 2 if rng.random() < 0.2 else 1
        c["pool"] = c["stride"] == 1 and h % 2 == 0 and w % 2 == 0 and rng.random() < 0.2
        c["bias"], c["relu"] = rng.random() < 0.5, rng.random() < 0.5
    return c


def _layers(case):
    """(cin, cout, size, drop, pool) of a stack."""
    k = case["size"]
    return [(ci, co, s * k // 224, 0 if i == 0 else -1, i in _VGG_POOLS) for i, (ci, co, s) in enumerate(_VGG)]


def _keep(cin, cout, drop):
    k = cin * cout
    return k // 3 if drop < 0 else k - (k * drop + 99) // 100


def _weights(g, cout, cin, dtype):
    w = g.standard_normal((cout, cin, 3, 3), dtype=np.float32) * np.float32(math.sqrt(2.0 / (9.0 * cin)))
    return w.astype(np.float16 if dtype == "f16" else np.float32)


def _normal(shape, seed, dtype):
    t = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(shape, generator=t, device="cuda", dtype=torch.float32).to(_DT[dtype])


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _inputs(case, seed):
    """The inputs of a case, from the seed alone; weights are host arrays."""
    g = np.random.Generator(np.random.PCG64(seed))
    s = {}
    if case["kind"] == "stack":
        s["w"] = [_weights(g, co, ci, "f32") for ci, co, _, _, _ in _layers(case)]
        # synthetic images: integers 0..255 (the paper's Sec. 4.1)
        s["x"] = _dev(g.integers(0, 256, (case["n"], 3, case["size"], case["size"])).astype(np.float32))
        return s
    n, cin, cout, h, w, dt = (case[k] for k in ("n", "cin", "cout", "h", "w", "dtype"))
    s["w"] = _weights(g, cout, cin, dt)
    if case["kind"] == "conv":
        s["x"] = _normal((n, cin, h, w), seed + 1, dt)
        s["bias"] = _normal((cout,), seed + 2, dt) * 0.1 if case["bias"] else None
    elif case["kind"] == "retrain":
        s["x"] = _normal((n, cin, h, w), seed + 1, dt).relu_()
        s["dy"] = _normal((n, cout, h, w), seed + 2, dt) * 0.1
    elif case["kind"] == "admm":
        # in the middle of the pruning: W has left W0, the dual variable is not zero
        s["x"] = _normal((n, cin, h, w), seed + 1, dt).abs_()
        s["b"] = _normal((cout,), seed + 2, dt) * 0.1
        sd = math.sqrt(2.0 / (9.0 * cin))
        s["dev"] = _normal((cout, cin, 3, 3), seed + 3, dt) * (0.05 * sd)
        s["dual"] = _normal((cout, cin, 3, 3), seed + 4, dt) * (0.05 * sd)
    return s


_RHO = 1e-2


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["kind"] == "stack":
        masks = B.select_library(np.concatenate([v.reshape(-1, 3, 3) for v in s["w"]]), case["m"])
        s["layers"] = []
        for (ci, co, sz, drop, pool), v in zip(_layers(case), s.pop("w")):
            p = B.prepare(_dev(v), masks, _keep(ci, co, drop))
            o = sz // 2 if pool else sz
            s["layers"].append((p, pool, torch.empty((case["n"], co, o, o), device="cuda")))
        return s
    n, cin, cout, h, w, dt = (case[k] for k in ("n", "cin", "cout", "h", "w", "dtype"))
    keep = _keep(cin, cout, case["drop"])
    wh = s.pop("w")
    masks = B.select_library(wh, case["m"])
    wd = _dev(wh)
    if case["kind"] == "prune":
        s.update(w=wd, masks=masks, keep=keep)
        return s
    if case["kind"] == "admm":
        st = B.AdmmLayer(wd, s.pop("b"), masks, keep)
        s["target"] = st.target(s["x"])
        st.w.add_(s.pop("dev"))
        st.d.copy_(s.pop("dual"))
        s["admm"] = st
        return s
    prep = B.prepare(wd, masks, keep)
    s["prep"] = prep
    if case["kind"] == "conv":
        q = case["stride"]
        o = (h // 2, w // 2) if case["pool"] else ((h - 1) // q + 1, (w - 1) // q + 1)
        s["y"] = torch.empty((n, cout) + o, dtype=_DT[dt], device="cuda")
    else:
        s["prep_t"] = B.prepare_transposed(prep, wd)
        s["dx"] = torch.empty_like(s["x"])
        s["dv"] = torch.empty(4 * keep, device="cuda")
        s["db"] = torch.empty(cout, device="cuda")
        s["ws"] = B.conv3x3_bwd_weight_workspace(prep.layer, _CODE[dt], n, h, w)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "stack":
        x = s["x"]
        for p, pool, y in s["layers"]:
            (B.conv3x3_fwd_pool2 if pool else B.conv3x3_fwd)(p.layer, p.packed, x, y, relu=True)
            x = y
        return x
    if kind == "conv":
        p = s["prep"]
        if case["pool"]:
            B.conv3x3_fwd_pool2(p.layer, p.packed, s["x"], s["y"], bias=s["bias"], relu=case["relu"])
        elif case["stride"] == 2:
            B.conv3x3_fwd_strided(p.layer, p.packed, s["x"], s["y"], 2, bias=s["bias"], relu=case["relu"])
        else:
            B.conv3x3_fwd(p.layer, p.packed, s["x"], s["y"], bias=s["bias"], relu=case["relu"])
        return s["y"]
    if kind == "retrain":
        B.conv(s["prep_t"], s["dy"], out=s["dx"])
        B.conv3x3_bwd_weight(s["prep"].layer, s["prep"].packed, s["x"], s["dy"], s["dv"], s["db"], ws=s["ws"])
        return {"dx": s["dx"], "dv": s["dv"], "db": s["db"]}
    if kind == "admm":
        st = s["admm"]
        loss = st.iteration(s["x"], s["target"], _RHO, 1.0 / s["target"].numel())
        return {"loss": loss, "dw": st.dw, "db": st.db, "w": st.w, "b": st.b, "a": st.a, "d": st.d}
    r = B.prepare(s["w"], s["masks"], s["keep"])
    out = {k: getattr(r.packed, k) for k in B.PACKED_FIELDS}
    out.update(pat=r.pat, energy=r.energy, keep_mask=r.keep_mask)
    return out


def _packed_bytes(case, cin, cout, drop, elt):
    return _keep(cin, cout, drop) * (4 * elt + 5) + cout * (12 + 4 * (case["m"] + 1))


def work(case):
    if case["kind"] == "stack":
        n, b, f = case["n"], 0, 0
        for ci, co, s, drop, pool in _layers(case):
            # one layer's output is the next one's input: written once, read once
            b += 4 * n * (ci * s * s + co * (s * s // 4 if pool else s * s)) + _packed_bytes(case, ci, co, drop, 4)
            f += 8 * n * s * s * _keep(ci, co, drop)
        return {"bytes": b, "flops": f}
    n, cin, cout, h, w = (case[k] for k in ("n", "cin", "cout", "h", "w"))
    elt = 2 if case["dtype"] == "f16" else 4
    keep = _keep(cin, cout, case["drop"])
    pk = _packed_bytes(case, cin, cout, case["drop"], elt)
    if case["kind"] == "conv":
        q = case["stride"]
        oh, ow = (h - 1) // q + 1, (w - 1) // q + 1
        return {"bytes": elt * n * (cin * h * w + cout * oh * ow // (4 if case["pool"] else 1)) + pk,
                "flops": 8 * n * oh * ow * keep}
    if case["kind"] == "retrain":
        return {"bytes": elt * n * h * w * (2 * cin + cout) + 2 * pk + 16 * keep + 4 * cout, "flops": 16 * n * h * w * keep}
    k = cin * cout
    if case["kind"] == "admm":
        # x and the target once, W, A and D read and written; two dense contractions
        return {"bytes": 4 * n * h * w * (cin + cout) + 8 * 3 * 9 * k, "flops": 36 * n * h * w * k}
    return {"bytes": 9 * k * elt + 10 * k + pk, "flops": 2 * 9 * k}


def tolerance(case):
    if case["kind"] == "prune":
        return "exact"
    if case["kind"] == "stack":
        return {"rel": 1e-5}
    if case["kind"] == "admm":
        return {"rel": 2e-5}
    if case["kind"] == "retrain":
        return {"rel": 2e-3 if case["dtype"] == "f16" else 4e-6}
    return {"rel": 1e-3 if case["dtype"] == "f16" else 4e-6}


# ------------------------------------------------------------- 64-bit reference
def _energies(w, masks):
    """fp64 [K, m]: squares kept by each mask."""
    q = w.reshape(-1, 9).double() ** 2
    sel = torch.tensor([[(int(c) >> b) & 1 for b in range(9)] for c in masks], dtype=torch.float64, device=w.device)
    return q @ sel.T


def _pruned(w, masks, keep):
    """The pruned dense weights in fp64, and the kept (kernel, position) mask.
    Energies of one kernel that differ at all differ by far more than the
    rounding of a sum of four squares; equal ones take the lower index."""
    e = _energies(w, masks)
    best, pat = e.cpu().max(dim=1)
    order = torch.argsort(best, descending=True, stable=True)
    on = torch.zeros(e.shape[0], dtype=torch.bool)
    on[order[:keep]] = True
    bits = torch.tensor([[bool((int(c) >> b) & 1) for b in range(9)] for c in masks])
    sel = bits[pat] & on[:, None]
    sel = sel.to(w.device).reshape(w.shape)
    return w.double() * sel, sel


def _taps(x):
    """The nine shifted copies of x as [cin, n*h*w] matrices."""
    n, c, h, w = x.shape
    p = torch.nn.functional.pad(x, (1, 1, 1, 1))
    for q in range(9):
        yield q, p[:, :, q // 3:q // 3 + h, q % 3:q % 3 + w].permute(1, 0, 2, 3).reshape(c, -1)


def _conv64(x, wd):
    n, _, h, w = x.shape
    y = torch.zeros((wd.shape[0], n * h * w), dtype=torch.float64, device=x.device)
    for q, t in _taps(x.double()):
        y += torch.mm(wd[:, :, q // 3, q % 3].contiguous(), t)
    return y.reshape(-1, n, h, w).permute(1, 0, 2, 3)


def _wgrad64(x, dy):
    g = dy.double().permute(1, 0, 2, 3).reshape(dy.shape[1], -1)
    dw = torch.empty((dy.shape[1], x.shape[1], 3, 3), dtype=torch.float64, device=x.device)
    for q, t in _taps(x.double()):
        dw[:, :, q // 3, q % 3] = torch.mm(g, t.T.contiguous())
    return dw


def _pool(y):
    return torch.nn.functional.max_pool2d(y, 2)


def _in_storage_order(dw, wd, masks, keep, p):
    """The entries of dw at the stored positions, filter by filter as the
    packing of the case orders them."""
    cin = dw.shape[1]
    fp, ci = p.filter_ptr.long(), p.cin_idx.long()
    pos = torch.repeat_interleave(torch.arange(dw.shape[0], device=dw.device), fp[1:] - fp[:-1])
    k = p.filter_perm.long()[pos] * cin + ci
    bits = torch.tensor([[b for b in range(9) if (int(c) >> b) & 1] for c in masks], device=dw.device)
    return torch.gather(dw.reshape(-1, 9)[k], 1, bits[p.pat_id.long()]).reshape(-1)


def exact(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "stack":
        masks = B.select_library(np.concatenate([v.reshape(-1, 3, 3) for v in s["w"]]), case["m"])
        x = s["x"].double()
        for (ci, co, _, drop, pool), v in zip(_layers(case), s["w"]):
            x = _conv64(x, _pruned(_dev(v), masks, _keep(ci, co, drop))[0]).relu()
            x = _pool(x) if pool else x
        return x
    masks = B.select_library(s["w"], case["m"])
    keep = _keep(case["cin"], case["cout"], case["drop"])
    w = _dev(s["w"])
    if case["kind"] == "prune":
        out = {k: None for k in B.PACKED_FIELDS + ("pat", "keep_mask")}
        out["energy"] = _energies(w, masks).max(dim=1).values
        return out
    if case["kind"] == "admm":
        x, b, w0 = s["x"].double(), s["b"].double(), w.double()
        w1, d = (w + s["dev"]).double(), s["dual"].double()
        t = (_conv64(x, w0) + b[:, None, None]).relu()
        z = _conv64(x, w1) + b[:, None, None]
        c = 1.0 / t.numel()
        r = z.relu() - t
        g = 2 * c * r * (z > 0)
        dw, db = _wgrad64(x, g), g.sum((0, 2, 3))
        w2 = w1 - 1e-3 * (dw + _RHO * (w1 - w0 + d))
        return {"loss": (c * r.square().sum()).reshape(1), "dw": dw, "db": db, "w": w2, "b": b - 1e-3 * db,
                "a": None, "d": None}
    if case["kind"] == "conv":
        y = _conv64(s["x"], _pruned(w, masks, keep)[0])
        y = y[:, :, ::case["stride"], ::case["stride"]]
        if s["bias"] is not None:
            y = y + s["bias"].double()[:, None, None]
        y = y.relu() if case["relu"] else y
        return (_pool(y) if case["pool"] else y).contiguous()
    wd = _pruned(w, masks, keep)[0]
    dx = _conv64(s["dy"], wd.flip(2, 3).transpose(0, 1).contiguous())
    p = B.prepare(w, masks, keep).packed    # only the order in which dv is stored
    dv = _in_storage_order(_wgrad64(s["x"], s["dy"]), wd, masks, keep, p)
    return {"dx": dx.contiguous(), "dv": dv, "db": s["dy"].double().sum((0, 2, 3))}
