"""The tile kernel at extents that are odd multiples of 128 (padded), against
the oracle with the flat gates (every short side here is at least 129).  Few
matrices run on 128 x 128 tiles (the first test: both sides of the edge, both
orientations, parameter rows with and without 16-byte accesses, a table with
c = 0, whose polynomial is a scaling of A).  Eight of 1300 x 1950 run on 256 x 256
tiles, of which the last row and column are half inside the matrix (the second
test: the call's printed plan must say so, so that another cost model cannot
empty it).  fp32 Newton-Schulz runs on three bfloat16 planes a value."""
import numpy as np
import pytest

from oracle import muon_ref as ref
from paper_2609_21594_amd import synth
from tests.gpu_util import (MOMENTUM_TOL, TOL, decode, rel, require_gpu, route_recorder, to_dev, to_host,
                            w_gate)

pytestmark = pytest.mark.gpu

SHAPES = [(129, 129), (384, 384), (300, 384), (384, 520), (520, 384), (640, 1408), (1400, 640), (257, 301), (512, 648)]
TABLES = {"quintic": None, "c0": [(1.5, -0.5, 0.0)] * 5}


def rng(*key):
    return np.random.Generator(np.random.PCG64(np.random.SeedSequence([synth.ROOT_SEED, 8300, *key])))


@pytest.mark.parametrize("table", sorted(TABLES))
@pytest.mark.parametrize("prec", ["bf16", "f32"])
@pytest.mark.parametrize("pdt", ["bf16", "f32"])
def test_half_tiles_match_oracle(pdt, prec, table):
    require_gpu()
    import torch
    from paper_2609_21594_amd.binding import Muon
    coeffs = TABLES[table]
    hp = ref.MuonHParams(lr=0.02, beta=0.95, weight_decay=0.1, nesterov=True,
                         **({"ns_coeffs": coeffs} if coeffs else {}))
    Ws = [synth.draw(s, 0.02, pdt, rng(i, 0)) for i, s in enumerate(SHAPES)]
    gs = [synth.draw(s, 1e-3, "bf16", rng(i, 1)) for i, s in enumerate(SHAPES)]
    bs = [synth.draw(s, 1e-3, "f32", rng(i, 2)) for i, s in enumerate(SHAPES)]
    dW, dg, db = [to_dev(w, pdt) for w in Ws], [to_dev(g, "bf16") for g in gs], [to_dev(b, "f32") for b in bs]
    m = Muon(0)
    try:
        m.step(dW, dg, db, lr=hp.lr, beta=hp.beta, weight_decay=hp.weight_decay, ns_coeffs=coeffs,
               ns_precision=prec)
        torch.cuda.synchronize()
    finally:
        m.close()
    for s, W, g, b, w_dev, b_dev in zip(SHAPES, Ws, gs, bs, dW, db):
        W0 = decode(W, pdt)
        r = ref.muon_step_matrix(W0, decode(g, "bf16"), np.asarray(b, np.float64), hp)
        err, rho = w_gate(to_host(w_dev), r.W_new, W0, pdt)
        print(f"odd extents {pdt} {prec} NS {table} {s}: W err {err:.2e} (rho {rho:.1e})", flush=True)
        assert err <= TOL[prec] + rho, (s, err, rho)
        assert rel(to_host(b_dev), r.buf_new) <= MOMENTUM_TOL, s


@pytest.mark.parametrize("shape", [(1300, 1950), (1950, 1300)])
@pytest.mark.parametrize("prec", ["bf16", "f32"])
@pytest.mark.parametrize("pdt,shift", [("bf16", 0), ("bf16", 1), ("f32", 0), ("f32", 1)])
def test_half_tiles_of_the_256_kernel_match_oracle(pdt, shift, prec, shape, monkeypatch, capfd):
    """shift: W starts one element past a 16-byte boundary."""
    require_gpu()
    import torch
    from paper_2609_21594_amd.binding import Muon
    n = 8
    hp = ref.MuonHParams(lr=0.02, beta=0.95, weight_decay=0.1, nesterov=True)
    data = [[synth.draw(shape, sd, dt, rng(90, k, i % 2)) for k, (sd, dt) in
             enumerate(((0.02, pdt), (1e-3, "bf16"), (1e-3, "f32")))] for i in range(2)]
    buf = torch.full((n, shape[0] * shape[1] + 8), 7.0, dtype=torch.float32 if pdt == "f32" else torch.bfloat16,
                     device="cuda")
    dW = [b[shift:shift + shape[0] * shape[1]].view(shape) for b in buf]
    for i, w in enumerate(dW):
        w.copy_(to_dev(data[i % 2][0], pdt))
    dg = [to_dev(data[i % 2][1], "bf16") for i in range(n)]
    db = [to_dev(data[i % 2][2], "f32") for i in range(n)]
    routes = route_recorder(monkeypatch, capfd)
    m = Muon(0)
    try:
        m.step(dW, dg, db, lr=hp.lr, beta=hp.beta, weight_decay=hp.weight_decay, ns_precision=prec)
        torch.cuda.synchronize()
    finally:
        m.close()
    assert routes()[n, 1300, 1950] == ("256", "256", "256")
    for i in range(2):
        W, g, b = data[i]
        W0 = decode(W, pdt)
        r = ref.muon_step_matrix(W0, decode(g, "bf16"), np.asarray(b, np.float64), hp)
        err, rho = w_gate(to_host(dW[i]), r.W_new, W0, pdt)
        print(f"half tiles {pdt}+{shift} {prec} NS {shape}: W err {err:.2e} (rho {rho:.1e})", flush=True)
        assert err <= TOL[prec] + rho, (i, err, rho)
        assert rel(to_host(db[i]), r.buf_new) <= MOMENTUM_TOL, i
    for i in range(2, n):  # the same matrices again: the same bits
        assert torch.equal(dW[i], dW[i % 2]) and torch.equal(db[i], db[i % 2]), i
    assert bool((buf[:, :shift] == 7.0).all()) and bool((buf[:, shift + shape[0] * shape[1]:] == 7.0).all())
