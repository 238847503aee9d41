"""The 256 x 256 tile kernel at extents that are odd multiples of 128 (padded):
its last tile-row or column is half inside the matrix.  Both sides of the
edge, both orientations, parameter rows with and without 16-byte accesses, a
table with c = 0 (the A term read in the epilogue), against the oracle with
the flat gates (every short side here is at least 129); fp32 Newton-Schulz
runs there on three bfloat16 planes a value."""
import numpy as np
import pytest

from oracle import muon_ref as ref
from paper_2609_21594_amd import synth
from tests.gpu_util import MOMENTUM_TOL, TOL, decode, rel, require_gpu, to_dev, to_host, w_gate

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
        print(f"half tiles {pdt} {prec} NS {table} {s}: W err {err:.2e} (rho {rho:.1e})", flush=True)
        assert err <= TOL[prec] + rho, (s, err, rho)
        assert rel(to_host(b_dev), r.buf_new) <= MOMENTUM_TOL, s
