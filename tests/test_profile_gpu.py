"""Launch accounting and workspace reservation through the C ABI.

With profiling on, every launch is bracketed by events on its stream and
counted under its kernel family; the flop figures are the ones the bench's
roofline divides by the measured time, so they are checked here against the
dense count of Eq. 1 (2 s^2 l per Gram and update product, 2 s^3 per
polynomial product) and against the MFMA work of the kernels that the call
runs on (whole tiles, upper ones only of the symmetric products; which tiles,
the call's printed plan says).  Profiling must not change results.
"""
import numpy as np
import pytest

from paper_2609_21594_amd import synth
from tests.gpu_util import require_gpu, route_recorder, to_bits, to_dev

pytestmark = pytest.mark.gpu


def rng(*key):
    return np.random.Generator(np.random.PCG64(np.random.SeedSequence([9191, *key])))


def inputs(shapes):
    W = [to_dev(synth.draw(s, 0.02, "bf16", rng(i, 0)), "bf16") for i, s in enumerate(shapes)]
    G = [to_dev(synth.draw(s, 1e-3, "bf16", rng(i, 1)), "bf16") for i, s in enumerate(shapes)]
    M = [to_dev(synth.draw(s, 1e-3, "f32", rng(i, 2)), "f32") for i, s in enumerate(shapes)]
    return W, G, M


def test_profile_counts_and_flops_and_no_effect_on_results():
    require_gpu()
    import torch
    from paper_2609_21594_amd.binding import Muon
    K = 5
    s, l, n = 512, 1024, 3  # one chunk of three 512 x 1024 matrices on the tile kernel
    shapes = [(s, l)] * n
    plain = Muon(0)
    prof = Muon(0)
    try:
        W1, G1, M1 = inputs(shapes)
        W2, G2, M2 = inputs(shapes)
        plain.step(W1, G1, M1, ns_steps=K)
        prof.profile(True)
        prof.profile_read(reset=True)
        prof.step(W2, G2, M2, ns_steps=K)
        st = prof.profile_read(reset=True)
        torch.cuda.synchronize()
        for a, b in zip(W1 + M1, W2 + M2):
            np.testing.assert_array_equal(to_bits(a), to_bits(b))
    finally:
        plain.close()
        prof.close()
    launches = {k: v["launches"] for k, v in st.items()}
    assert launches["momentum_norm"] == 1 and launches["norm_finalize"] == 1 and launches["rescale"] == 1
    assert launches["gram_syrk"] == K and launches["poly_syrk"] == K
    assert launches["update_gemm"] == K - 1 and launches["update_apply_gemm"] == 1
    assert launches["apply_x0"] == 0 and launches["adamw"] == 0
    for k, v in st.items():
        assert v["total_ms"] >= 0 and (v["launches"] > 0 or v["total_ms"] == 0), k
        if v["flops"]:
            assert v["total_ms"] > 0, k
    assert st["gram_syrk"]["flops"] == pytest.approx(K * n * 2 * s * s * l, rel=1e-12)
    assert st["poly_syrk"]["flops"] == pytest.approx(K * n * 2 * s ** 3, rel=1e-12)
    assert st["update_gemm"]["flops"] == pytest.approx((K - 1) * n * 2 * s * s * l, rel=1e-12)
    assert st["update_apply_gemm"]["flops"] == pytest.approx(n * 2 * s * s * l, rel=1e-12)


def up(v, m):
    return (v + m - 1) // m * m


# (matrices, s, l, Newton-Schulz precision): all three tile configurations, the
# last 256 x 256 tile half inside the padded extent, three planes
@pytest.mark.parametrize("n,s,l,prec", [(3, 512, 1024, "bf16"), (1, 640, 700, "bf16"), (8, 1408, 2048, "bf16"),
                                        (1, 1408, 2048, "bf16"), (2, 300, 520, "f32"), (40, 640, 640, "f32")])
def test_executed_flops_are_those_of_the_tiles_that_run(n, s, l, prec, monkeypatch, capfd):
    require_gpu()
    import torch
    from paper_2609_21594_amd.binding import Muon
    coeffs = [(3.4445, -4.7750, 2.0315)] * 2 + [(1.5, -0.5, 0.0)]  # c = 0: a scaling, no product
    routes = route_recorder(monkeypatch, capfd)
    m = Muon(0)
    try:
        m.set_streams(1)
        ins = [torch.randn(s, l, device="cuda") for _ in range(n)]
        outs = [torch.empty_like(t) for t in ins]
        m.profile(True)
        m.profile_read(reset=True)
        m.orthogonalize(ins, outs, ns_steps=3, ns_coeffs=coeffs, ns_precision=prec)
        st = m.profile_read(reset=True)
    finally:
        m.close()
    tiles = routes()[n, s, l]
    print(f"{n} x {s} x {l} {prec}: {tiles}", flush=True)
    S, L, pairs = up(s, 128), up(l, 128), 6 if prec == "f32" else 1
    side = [int(t.split("x")[0]) for t in tiles]
    upper = lambda t: (up(S, t) // t) * (up(S, t) // t + 1) / 2 * t * t
    want = {"gram_syrk": 3 * 2 * upper(side[0]) * L, "poly_syrk": 2 * 2 * upper(side[1]) * S,
            "update_gemm": 2 * 2 * up(S, side[2]) * up(L, side[2]) * S,
            "update_apply_gemm": 2 * up(S, side[2]) * up(L, side[2]) * S}
    for k, v in want.items():
        assert st[k]["exec_flops"] == pytest.approx(n * pairs * v, rel=1e-12), k


@pytest.mark.parametrize("n,s,l,prec", [(3, 20, 1100, "bf16"), (3, 64, 1100, "bf16"), (2, 128, 1300, "bf16"),
                                        (2, 30, 700, "f32"), (2, 100, 1500, "f32")])
def test_executed_flops_of_column_slices(n, s, l, prec):
    """Upper blocks of 32 rows of the Gram product and X' over all columns; B in
    every slice (1024 / row blocks wide; half that in fp32 and in the last step)."""
    require_gpu()
    import torch
    from paper_2609_21594_amd.binding import Muon
    m = Muon(0)
    try:
        ins = [torch.randn(s, l, device="cuda") for _ in range(n)]
        outs = [torch.empty_like(t) for t in ins]
        m.profile(True)
        m.profile_read(reset=True)
        m.orthogonalize(ins, outs, ns_precision=prec)
        st = m.profile_read(reset=True)["ns_small"]
    finally:
        m.close()
    Sx, L = (32 if s <= 32 else 64 if s <= 64 else 128), up(l, 128)
    rb = Sx // 32
    w = (1024 if prec == "bf16" else 512) // rb
    slices = 4 * -(-L // w) + -(-L // (512 // rb))
    want = 5 * 2 * L * (rb * (rb + 1) / 2 * 1024 + Sx * Sx) + 2 * Sx ** 3 * slices
    assert st["launches"] == 1 and st["exec_flops"] == pytest.approx(n * want, rel=1e-12)
    assert st["flops"] == pytest.approx(n * 5 * (4 * s * s * l + 2 * s ** 3), rel=1e-12)


def test_reserve_presizes_the_workspace():
    require_gpu()
    import torch
    from paper_2609_21594_amd.binding import Muon
    shapes = [(512, 1024)] * 2 + [(256, 256)]
    m = Muon(0)
    try:
        m.reserve(64 << 20)
        assert m.workspace_bytes >= 64 << 20
        before = m.workspace_bytes
        W, G, M = inputs(shapes)
        m.step(W, G, M)
        torch.cuda.synchronize()
        assert m.workspace_bytes == before  # the plan fitted: nothing was reallocated
    finally:
        m.close()
    from paper_2609_21594_amd.binding import MuonError
    capped = Muon(0)
    try:
        capped.set_workspace_limit(1 << 20)
        with pytest.raises(MuonError) as e:
            capped.reserve(2 << 20)
        assert e.value.status == 3 and capped.workspace_bytes == 0
    finally:
        capped.close()
