"""The configurations of the tile kernel (256 x 256, 128 x 128, 128 x 128 with four
stages) give the same bits: which of them a launch takes depends on how many
matrices share it, and a matrix's result may not.  Each shape runs alone and
among more copies.  In the second test every product of a call meets every
configuration, also with A and B written by one and read by another, which the
calls' printed plans must show."""
import numpy as np
import pytest

from oracle import muon_ref as ref
from paper_2609_21594_amd import synth
from tests.gpu_util import decode, o_gate, require_gpu, route_recorder, to_bits, to_dev, to_host

pytestmark = pytest.mark.gpu

C0 = [(1.5, -0.5, 0.0)] * 3


def rng(*key):
    return np.random.Generator(np.random.PCG64(np.random.SeedSequence([synth.ROOT_SEED, 8400, *key])))


@pytest.mark.parametrize("prec", ["bf16", "f32"])
@pytest.mark.parametrize("shape", [(256, 256), (300, 700), (384, 520), (520, 384), (640, 640), (700, 1000), (1024, 513)])
def test_result_does_not_depend_on_the_batch(shape, prec):
    require_gpu()
    import torch
    from paper_2609_21594_amd.binding import Muon
    m = Muon(0)
    try:
        g = synth.draw(shape, 1.0, prec, rng(*shape))
        one = to_dev(g, prec)
        for coeffs in (None, C0):
            kw = dict(ns_steps=3, ns_precision=prec, ns_coeffs=coeffs or [ref.LEGACY_QUINTIC] * 3)
            alone = torch.full_like(one, float("nan"))
            m.orthogonalize([one], [alone], **kw)
            for n in (3, 7, 24, 60, 130, 300):
                outs = [torch.full_like(one, float("nan")) for _ in range(n)]
                ins = [one.clone() for _ in range(n)]
                m.orthogonalize(ins, outs, **kw)
                torch.cuda.synchronize()
                for i in (0, n // 2, n - 1):
                    assert np.array_equal(to_bits(outs[i]), to_bits(alone)), (shape, n, i)
                del outs, ins
            x = decode(g, prec)
            err, gate = o_gate(to_host(alone), ref.orthogonalize(x, 3, kw["ns_coeffs"]), prec, prec, 3,
                               kw["ns_coeffs"], G=x)
            print(f"tiles {prec} {shape} {'c0' if coeffs else 'quintic'}: O err {err:.2e}", flush=True)
            assert err <= gate, (shape, err, gate)
    finally:
        m.close()


# padded extents: 1408 x 1408, 1024 x 1408, 1408 x 2048
@pytest.mark.parametrize("prec", ["bf16", "f32"])
@pytest.mark.parametrize("shape", [(1300, 1300), (1000, 1400), (2000, 1390)])
def test_every_configuration_gives_the_same_bits(shape, prec, monkeypatch, capfd):
    require_gpu()
    import torch
    from paper_2609_21594_amd.binding import Muon
    routes = route_recorder(monkeypatch, capfd)
    s, l = sorted(shape)
    W, g, b = (synth.draw(shape, sd, dt, rng(70 + k, *shape)) for k, (sd, dt) in
               enumerate(((0.02, "bf16"), (1e-3, "bf16"), (1e-3, "f32"))))
    first, seen = {}, set()
    m = Muon(0)
    try:
        for n in (1, 2, 3, 4, 6, 8, 9, 16, 30):
            # a step on bf16 and one on fp32 parameters, and the orthogonalisation
            for kind in ("bf16", "f32", "orth"):
                if kind == "orth":
                    ins = [to_dev(g, "bf16") for _ in range(n)]
                    outs = [torch.full_like(t, float("nan")) for t in ins]
                    m.orthogonalize(ins, outs, ns_steps=3, ns_precision=prec)
                else:
                    outs = [to_dev(W, "bf16").to(torch.float32 if kind == "f32" else torch.bfloat16) for _ in range(n)]
                    m.step(outs, [to_dev(g, "bf16") for _ in range(n)], [to_dev(b, "f32") for _ in range(n)], lr=0.02,
                           beta=0.95, ns_steps=3, ns_precision=prec)
                torch.cuda.synchronize()
                seen.add(routes()[n, s, l])
                want = first.setdefault(kind, outs[0].clone())
                for i in range(n):
                    assert torch.equal(outs[i], want), (shape, kind, n, i)
    finally:
        m.close()
    print(f"{shape} {prec}: {sorted(seen)}", flush=True)
    for product in range(3):
        kinds = {r[product] for r in seen}
        assert kinds >= ({"256", "128", "128x4"} if prec == "bf16" else {"256", "128"}), (product, seen)
    assert any(r[0] == r[1] != r[2] for r in seen)  # A and B written by one, read by another


# The lines between the routes, where both sides were measured: one fp32 matrix
# took up to 40% longer in slices below these, and two 4096^2 beside a 4096 x 11008
# 3% longer on 128 x 128 tiles at a near tie (0.96) of the model.
@pytest.mark.parametrize("n,s,l,prec,want", [
    (1, 32, 576, "f32", "fused"), (1, 32, 577, "f32", "slices"), (1, 64, 768, "f32", "fused"), (1, 64, 769, "f32", "slices"),
    (1, 65, 1025, "f32", "fused"), (1, 96, 1536, "f32", "fused"), (1, 96, 1537, "f32", "slices"),
    (1, 97, 1408, "f32", "fused"), (1, 128, 1409, "f32", "slices"), (1, 32, 256, "bf16", "fused"),
    (1, 32, 257, "bf16", "slices"), (1, 33, 384, "bf16", "fused"), (1, 128, 385, "bf16", "slices"),
    (2, 4096, 4096, "bf16", ("256", "256", "256")), (1, 1024, 4096, "bf16", ("128x4", "128x4", "128x4"))])
def test_routes_at_the_lines(n, s, l, prec, want, monkeypatch, capfd):
    require_gpu()
    import torch
    from paper_2609_21594_amd.binding import Muon
    routes = route_recorder(monkeypatch, capfd)
    m = Muon(0)
    try:
        ins = [torch.randn(s, l, device="cuda") for _ in range(n)]
        m.orthogonalize(ins, [torch.empty_like(t) for t in ins], ns_steps=1, ns_precision=prec)
        torch.cuda.synchronize()
    finally:
        m.close()
    assert routes()[n, s, l] == want
