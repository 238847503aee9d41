"""The calls whose speed is followed: what users of the batched Muon step have it do.

Every case goes through the public Python entry points (`Muon.step`,
`Muon.orthogonalize`, `Muon.adamw_step`, `MuonAdamW.step`) on tensors that stay
on the GPU.  The shapes are this repository's workloads and the shapes its
views, stacks and ragged buckets are meant for.

A case is a dict of plain values:
  kind    "step", "orth", "adamw" or "optim"
  groups  the matrices, as words "layout:count:ROWSxCOLS" (see `_groups`)
  param, grad, ns   "bf16" or "f32": parameter, gradient and Newton-Schulz dtype
and the options of the entry point.  Matrices of one group live in one buffer
(each starts 256-byte aligned), so that a case has few outputs.
"""
import math

import numpy as np
import torch

from paper_2609_21594_amd.binding import Muon
from paper_2609_21594_amd.optim import MuonAdamW

DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}
QUINTIC = (3.4445, -4.7750, 2.0315)
LR, BETA = 0.02, 0.95


def listed():
    return [
        # one small fp32 matrix in fp32 throughout: a call's latency, nothing else
        dict(name="single-256x128-f32", kind="step", groups="mats:1:256x128", param="f32", grad="f32", ns="f32",
             wd=0.0),
        # one transformer block of a small model, as one training step's call
        dict(name="block-h2048", kind="step", groups="mats:4:2048x2048 mats:2:5632x2048 mats:1:2048x5632",
             param="bf16", grad="bf16", ns="bf16", wd=0.0),
        # two layers of a 7B-like model: the ordinary large call
        dict(name="layers-h4096", kind="step", groups="mats:8:4096x4096 mats:4:11008x4096 mats:2:4096x11008",
             param="bf16", grad="bf16", ns="bf16", wd=0.01),
        # what one owner holds of a 70B-like layer with grouped K and V: the largest matrices
        dict(name="owner-h8192", kind="step", groups="mats:2:8192x8192 mats:2:1024x8192 mats:1:8192x28672",
             param="bf16", grad="bf16", ns="bf16", wd=0.01),
        # the standalone orthogonalisation of a mixed batch, every 7th matrix 1e-4 in size
        dict(name="orth-mixed-512", kind="orth",
             groups="mats:96:1024x4096 mats:96:4096x1024 mats:256:512x512 mats:64:128x2048", grad="bf16", ns="bf16",
             noalloc=False),
        # the torch optimizer over a small language model: fp32 parameters, embedding and norms on AdamW
        dict(name="optim-h768", kind="optim", layers=12, hidden=768, ffn=3072, vocab=32000),
        # a layer's experts, gate and up packed side by side in one weight, down on its own; off the 256 grid
        dict(name="experts-2048x1408", kind="step", groups="packed:16:2048x1408 stack:16:1408x2048", param="bf16",
             grad="bf16", ns="bf16", wd=0.01),
        # Q, K and V of a fused projection, one 128 x hidden matrix per head
        dict(name="heads-128x4096", kind="step", groups="heads:32:128x4096", param="bf16", grad="bf16", ns="bf16",
             wd=0.0),
        # low-rank adapters: many thin matrices of both orientations, fp32 masters
        dict(name="adapters-16x4096", kind="step", groups="mats:56:16x4096 mats:56:4096x16", param="f32",
             grad="f32", ns="bf16", wd=0.0),
        # a mid-sized model whose user asks for fp32 Newton-Schulz
        dict(name="layers-h1024-f32", kind="step", groups="mats:16:1024x1024 mats:8:2816x1024 mats:4:1024x2816",
             param="f32", grad="f32", ns="f32", wd=0.01),
        # a few odd matrices from a loop that must not allocate
        dict(name="orth-odd-noalloc", kind="orth", groups="mats:3:333x1001 mats:2:1000x77 mats:4:641x515", grad="bf16",
             ns="bf16", noalloc=True),
        # embedding, output head and norms of a 7B-like model through AdamW
        dict(name="adamw-262m", kind="adamw", vecs="2:131072000 65:4096", param="bf16", grad="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo, hi):
    """A side between lo and hi: odd and ragged ones, and the multiples that models have."""
    v, q = _log_int(rng, lo, hi), rng.choice((1, 1, 8, 64, 128, 256))
    return max(lo, min(hi, (v + q // 2) // q * q if v >= q else v))


def draw(rng):
    kind = rng.choice(("step", "step", "step", "step", "orth", "orth", "optim", "adamw"))
    if kind == "adamw":
        return dict(kind="adamw", vecs="%d:%d %d:%d" % (rng.randint(1, 3), _log_int(rng, 1000, 50000000),
                                                       rng.randint(1, 99), _log_int(rng, 64, 16384)),
                    param=rng.choice(("bf16", "f32")), grad=rng.choice(("bf16", "f32")))
    if kind == "optim":
        h = _side(rng, 128, 1536)
        return dict(kind="optim", layers=rng.randint(1, 12), hidden=h, ffn=int(h * rng.uniform(2, 4)),
                    vocab=_log_int(rng, 1000, 32000))
    ns = rng.choice(("bf16", "bf16", "f32"))
    flops, elems = (1.2e13, 2.5e8) if ns == "bf16" else (1e12, 5e7)
    words, n_groups = [], rng.randint(1, 3)
    for _ in range(n_groups):
        layout = "mats" if kind == "orth" else rng.choice(("mats", "mats", "stack", "packed", "heads"))
        per = {"packed": 2, "heads": 3}.get(layout, 1)
        s = _side(rng, 16, 4096)
        l = min(16384, max(s, _side(rng, s, 8 * s)))
        while _dense(s, l, 5) * per * n_groups > flops or s * l * per * n_groups > elems:
            s, l = s // 2, l // 2
        rows, cols = (s, l) if rng.random() < 0.5 else (l, s)
        most = min(64 // per, 20 if kind == "orth" else 64, flops / n_groups / per / _dense(rows, cols, 5),
                   elems / n_groups / per / (rows * cols))
        words.append("%s:%d:%dx%d" % (layout, _log_int(rng, 1, max(1, most)), rows, cols))
    case = dict(kind=kind, groups=" ".join(words), grad=rng.choice(("bf16", "f32")), ns=ns)
    if kind == "orth":
        case["noalloc"] = False
    else:
        case.update(param=rng.choice(("bf16", "f32")), wd=rng.choice((0.0, 0.01, 0.1)))
    return case


def _dense(rows, cols, steps):
    s, l = min(rows, cols), max(rows, cols)
    return steps * (4.0 * s * s * l + 2.0 * s ** 3)


def _groups(case):
    """(layout, count, rows, cols) of each word; the matrices of a group are
    mats    `count` separate matrices
    stack   one [count, rows, cols] entry of independent matrices
    packed  two [count, rows, cols] entries, the column halves of one [count, rows, 2 cols] weight
    heads   three [count, rows, cols] entries, interleaved in one [count, 3, rows, cols] weight
    """
    if case["kind"] == "optim":
        n, h, f = case["layers"], case["hidden"], case["ffn"]
        return [("mats", 4 * n, h, h), ("mats", n, f, h), ("mats", n, h, f)]
    out = []
    for word in case["groups"].split():
        layout, n, shape = word.split(":")
        rows, cols = shape.split("x")
        out.append((layout, int(n), int(rows), int(cols)))
    return out


def _matrices(case):
    return [(n * {"packed": 2, "heads": 3}.get(layout, 1), r, c) for layout, n, r, c in _groups(case)]


def _vecs(case):
    """(count, numel) of the AdamW tensors."""
    if case["kind"] == "optim":
        return [(1, case["vocab"] * case["hidden"]), (2 * case["layers"] + 1, case["hidden"])]
    return [tuple(int(v) for v in word.split(":")) for word in case["vecs"].split()]


def _buffer(layout, n, rows, cols, dtype):
    """A zeroed buffer for a group, and its entries as views of it."""
    if layout == "packed":
        b = torch.zeros(n, rows, 2 * cols, dtype=dtype, device="cuda")
        return b, [b[:, :, :cols], b[:, :, cols:]]
    if layout == "heads":
        b = torch.zeros(n, 3, rows, cols, dtype=dtype, device="cuda")
        return b, [b[:, i] for i in range(3)]
    if layout == "stack":
        b = torch.zeros(n, rows, cols, dtype=dtype, device="cuda")
        return b, [b]
    b = torch.zeros(n, (rows * cols + 127) // 128 * 128, dtype=dtype, device="cuda")
    return b, [b[i, :rows * cols].view(rows, cols) for i in range(n)]


def _flat(n, numel, dtype):
    b = torch.zeros(n, (numel + 127) // 128 * 128, dtype=dtype, device="cuda")
    return b, [b[i, :numel] for i in range(n)]


def _randn(shape, sigma, gen):
    return torch.randn(shape, dtype=torch.float32, device="cuda", generator=gen).mul_(sigma)


def _gradient(t, sigma, gen):
    """Noise and a part of rank 4 of the same size: a gradient's spectrum is not flat."""
    g = _randn(t.shape, 0.7 * sigma, gen)
    rows, cols = t.shape[-2:]
    u, v = _randn(t.shape[:-1] + (4,), 0.35, gen), _randn(t.shape[:-2] + (4, cols), sigma, gen)
    for r in range(4):
        g.addcmul_(u[..., r:r + 1], v[..., r:r + 1, :])
    t.copy_(g)


def _matrix_inputs(case, seed):
    """Per group: (parameter, gradient, momentum) buffers and their entries."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    pd, gd = DTYPE[case.get("param", "f32")], DTYPE[case.get("grad", "f32")]
    out = []
    for group in _groups(case):
        w, g, m = _buffer(*group, pd), _buffer(*group, gd), _buffer(*group, torch.float32)
        for a, b, c in zip(w[1], g[1], m[1]):
            a.copy_(_randn(a.shape, 0.02, gen))
            _gradient(b, 1e-3, gen)
            c.copy_(_randn(c.shape, 1e-3, gen))
        out.append((w, g, m))
    return out


def _vec_inputs(case, seed):
    """Per word: (parameter, gradient, first and second moment) buffers and entries."""
    gen = torch.Generator(device="cuda").manual_seed(seed + 1)
    pd, gd = DTYPE[case.get("param", "f32")], DTYPE[case.get("grad", "f32")]
    out = []
    for n, numel in _vecs(case):
        four = [_flat(n, numel, d) for d in (pd, gd, torch.float32, torch.float32)]
        for p, g, m, v in zip(*(f[1] for f in four)):
            p.copy_(_randn(p.shape, 0.02, gen))
            g.copy_(_randn(g.shape, 1e-3, gen))
            m.copy_(_randn(m.shape, 3e-4, gen))
            v.copy_(_randn(v.shape, 1e-3, gen).square_())
        out.append(four)
    return out


def _orth_inputs(case, seed):
    """Per group: the input buffer and its entries; N(0, 1), every 7th matrix 1e-4 of that."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    out, i = [], 0
    for group in _groups(case):
        b, entries = _buffer(*group, DTYPE[case["grad"]])
        for t in entries:
            i += 1
            t.copy_(_randn(t.shape, 1e-4 if i % 7 == 0 else 1.0, gen))
        out.append((b, entries))
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "orth":
        ins = _orth_inputs(case, seed)
        outs = [_buffer(*g, DTYPE[case["grad"]]) for g in _groups(case)]
        return dict(case=case, muon=Muon(0), ins=[t for _, e in ins for t in e], outs=[t for _, e in outs for t in e],
                    result=[b for b, _ in outs])
    if kind == "adamw":
        four = _vec_inputs(case, seed)
        lists = [[t for word in four for t in word[k][1]] for k in range(4)]
        return dict(case=case, muon=Muon(0), lists=lists, result=[word[k][0] for word in four for k in (0, 2, 3)])
    three = _matrix_inputs(case, seed)
    lists = [[t for group in three for t in group[k][1]] for k in range(3)]
    result = [group[k][0] for group in three for k in (0, 2)]
    if kind == "step":
        return dict(case=case, muon=Muon(0), lists=lists, result=result)
    four = _vec_inputs(case, seed)
    vecs = [[t for word in four for t in word[k][1]] for k in range(4)]
    vecs = [[t[0].view(case["vocab"], case["hidden"])] + t[1:] for t in vecs]
    mats = [torch.nn.Parameter(t) for t in lists[0]]
    others = [torch.nn.Parameter(t) for t in vecs[0]]
    for p, g in zip(mats + others, lists[1] + vecs[1]):
        p.grad = g
    opt = MuonAdamW([dict(params=mats), dict(params=others, use_muon=False)], lr=LR, weight_decay=0.01,
                    adamw_lr=3e-4, adamw_weight_decay=0.1)
    for p, m in zip(mats, lists[2]):
        opt.state[p]["momentum_buffer"] = m
    for p, m, v in zip(others, vecs[2], vecs[3]):
        opt.state[p].update(step=torch.tensor(9), exp_avg=m, exp_avg_sq=v)
    return dict(case=case, opt=opt, result=result + [word[k][0] for word in four for k in (0, 2, 3)])


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "orth":
        state["muon"].orthogonalize(state["ins"], state["outs"], ns_precision=case["ns"], noalloc=case["noalloc"])
    elif kind == "step":
        state["muon"].step(*state["lists"], lr=LR, beta=BETA, weight_decay=case["wd"], ns_precision=case["ns"])
    elif kind == "adamw":
        state["muon"].adamw_step(*state["lists"], step=10, lr=3e-4, betas=(0.9, 0.95), weight_decay=0.1)
    else:
        state["opt"].step()
    return state["result"]


def work(case):
    """Each input read and each output written once; the products of Eq. (1)
    with the symmetric ones counted on one triangle."""
    size = lambda k: 2.0 if case.get(k, "f32") == "bf16" else 4.0
    nbytes = flops = 0.0
    if case["kind"] != "adamw":
        for n, rows, cols in _matrices(case):
            s, l = min(rows, cols), max(rows, cols)
            flops += n * 5 * (3.0 * s * s * l + float(s) ** 3)
            nbytes += n * rows * cols * (2 * size("grad") if case["kind"] == "orth" else
                                         size("grad") + 8 + 2 * size("param"))
    if case["kind"] in ("adamw", "optim"):
        for n, numel in _vecs(case):
            nbytes += n * numel * (2 * size("param") + size("grad") + 16)
            flops += n * numel * 15.0
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Measured against `exact`: bf16 Newton-Schulz rounds X, A and B to 8 bits
    after every product, which leaves an orthogonalised matrix 0.9e-2 to 1.3e-2
    from the exact one (two orders of the sums: 2e-2 from each other) and a
    stepped parameter 1.9e-3 to 3.3e-3.  fp32 throughout: 5e-7 on a parameter,
    7e-6 on an orthogonalised matrix; in bf16 storage its last bit, 2e-3.
    AdamW is element by element."""
    if case["kind"] == "adamw":
        return {"rel": 1e-3 if case["param"] == "bf16" else 1e-6, "max": 0.1}
    if case["kind"] == "orth":
        if case["ns"] == "bf16":
            return {"rel": 3e-2, "max": 0.5}
        return {"rel": 1e-3 if case["grad"] == "bf16" else 3e-5, "max": 0.1}
    if case["kind"] == "optim" or case["ns"] == "bf16":
        return {"rel": 1e-2, "max": 0.3}
    return {"rel": 1e-3 if case["param"] == "bf16" else 5e-6, "max": 0.1}


def _f32(v):
    return float(np.float32(v))


def _orthogonal(u):
    """Five quintic Newton-Schulz steps on u / (|u| + eps), in 64 bits, short side first."""
    if u.shape[0] > u.shape[1]:
        return _orthogonal(u.T.contiguous()).T
    a, b, c = (_f32(v) for v in QUINTIC)
    x = u / (torch.linalg.norm(u) + _f32(1e-7))
    for _ in range(5):
        g = x @ x.T.contiguous()
        x = a * x + (b * g + c * (g @ g)) @ x
    return x


def _planes(t):
    return [t] if t.dim() == 2 else list(t)


def _exact_vec(p, g, m, v, t):
    p, g, b1, b2 = p.double(), g.double(), _f32(0.9), _f32(0.95)
    m.mul_(b1).add_(g, alpha=1 - b1)
    v.mul_(b2).addcmul_(g, g, value=1 - b2)
    denom = (v / (1 - b2 ** t)).sqrt_().add_(_f32(1e-8))
    return p.mul_(1 - _f32(3e-4) * _f32(0.1)).sub_(_f32(3e-4) * (m / (1 - b1 ** t)) / denom)


def exact(case, seed):
    result = []
    if case["kind"] == "orth":
        for (_, ins), group in zip(_orth_inputs(case, seed), _groups(case)):
            b, outs = _buffer(*group, torch.float64)
            for x, o in zip(ins, outs):
                o.copy_(_orthogonal(x.double()))
            result.append(b)
        return result
    if case["kind"] in ("step", "optim"):
        wd, beta = _f32(case.get("wd", 0.01)), _f32(BETA)
        for group, (w, g, m) in zip(_groups(case), _matrix_inputs(case, seed)):
            (bw, ws), (bm, ms) = _buffer(*group, torch.float64), _buffer(*group, torch.float64)
            for entry in zip(w[1], g[1], m[1], ws, ms):
                for p, gr, mo, po, mm in zip(*(_planes(t) for t in entry)):
                    gr = gr.double()
                    mm.copy_(beta * mo.double() + (1 - beta) * gr)
                    o = _orthogonal((1 - beta) * gr + beta * mm)
                    po.copy_((1 - _f32(LR) * wd) * p.double() - _f32(LR) * 0.2 * math.sqrt(max(p.shape)) * o)
            result += [bw, bm]
    if case["kind"] in ("adamw", "optim"):
        for four, (n, numel) in zip(_vec_inputs(case, seed), _vecs(case)):
            out = [_flat(n, numel, torch.float64) for _ in range(3)]
            for k in range(n):
                p, g, m, v = (f[1][k] for f in four)
                out[1][1][k].copy_(m)
                out[2][1][k].copy_(v)
                out[0][1][k].copy_(_exact_vec(p, g, out[1][1][k], out[2][1][k], 10))
            result += [f[0] for f in out]
    return result
