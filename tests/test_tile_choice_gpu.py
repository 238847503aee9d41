"""The 256 x 256 and the 128 x 128 configuration of the tile kernel give the
same bits: which of them a launch takes depends on how many matrices share
it, and a matrix's result may not.  Each shape runs alone and among enough
copies to fill the chip, so that its products move from one to the other
(also one product at a time: A written by one, read by the other)."""
import numpy as np
import pytest

from oracle import muon_ref as ref
from paper_2609_21594_amd import synth
from tests.gpu_util import decode, o_gate, require_gpu, to_bits, to_dev, to_host

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
