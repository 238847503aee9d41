"""fp32 Newton-Schulz on the tile kernel multiplies values split into three
bfloat16 planes.  Its error against the 64-bit oracle is compared with that
of the same iteration in plain binary32 on the CPU, on the same input: at
most twice that (the sums of the CPU's blocked products round in another
order), plus one binary32 rounding.  Inputs: flat spectrum, rows decaying
over four decades, a few dominant directions, and a norm far below eps,
where O is 484.9 X0 and only the term a X of each step matters: also at the
bottom of binary32's range, where bfloat16 planes of the values themselves
would end before 24 bits, with the default eps and with one that leaves O
there."""
import numpy as np
import pytest

from oracle import muon_ref as ref
from paper_2609_21594_amd import synth
from tests.gpu_util import rel, require_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu


def make(kind, shape):
    rng = np.random.Generator(np.random.PCG64(np.random.SeedSequence([synth.ROOT_SEED, 8500, *shape])))
    g = rng.standard_normal(shape, dtype=np.float32)
    if kind == "decay":
        g *= np.logspace(0, -4, shape[0], dtype=np.float32)[:, None]
    elif kind == "dominant":
        g = np.float32(0.01) * g + rng.standard_normal((shape[0], 4), dtype=np.float32) @ rng.standard_normal(
            (4, shape[1]), dtype=np.float32)
    elif kind == "tiny":
        g *= np.float32(1e-13)
    elif kind.startswith("bottom"):
        g *= np.float32(1e-36)
    return g


def plain_f32(g, eps):
    import torch
    a, b, c = (torch.tensor(v, dtype=torch.float32) for v in ref.LEGACY_QUINTIC)
    u = torch.from_numpy(g)
    x = (u.double() / (torch.linalg.norm(u.double()) + eps)).float()
    for _ in range(5):
        s = x @ x.T
        x = a * x + (b * s + c * (s @ s)) @ x
    return x.double().numpy()


@pytest.mark.parametrize("kind", ["gauss", "decay", "dominant", "tiny", "bottom", "bottom, eps 1"])
@pytest.mark.parametrize("shape", [(130, 400), (256, 256), (384, 1000), (512, 2048)])
def test_split_error_is_that_of_fp32(shape, kind):
    require_gpu()
    import torch
    from paper_2609_21594_amd.binding import Muon
    g = make(kind, shape)
    eps = 1.0 if kind.endswith("eps 1") else 1e-7
    want = ref.orthogonalize(g.astype(np.float64), 5, eps=eps)
    m = Muon(0)
    try:
        d = to_dev(g, "f32")
        out = torch.full_like(d, float("nan"))
        m.orthogonalize([d], [out], ns_precision="f32", eps=eps)
        torch.cuda.synchronize()
        err = rel(to_host(out), want)
    finally:
        m.close()
    plain = rel(plain_f32(g, eps), want)
    print(f"split {kind} {shape}: O err {err:.2e}, plain fp32 {plain:.2e}", flush=True)
    assert err <= 2 * plain + 6e-8, (shape, kind, err, plain)
