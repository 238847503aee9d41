"""The binding's reading of torch tensors as logical matrices (host only).

The C ABI reads a zero stride as "dense default", so the binding must turn
every real layout into explicit strides and refuse layouts whose rows,
blocks or planes overlap (expanded or broadcast tensors)."""
import pytest

torch = pytest.importorskip("torch")

from paper_2609_21594_amd.binding import RowBlocks, _view  # noqa: E402


def fields(x):
    return _view(x)[1:]  # (batch, rows, cols, ld, row_block, block_stride, plane_stride)


def test_dense_and_strided_views():
    W = torch.zeros(12, 8)
    assert fields(W) == (1, 12, 8, 8, 0, 0, 0)
    assert fields(W[:, 2:6]) == (1, 12, 4, 8, 0, 0, 0)
    assert fields(W.view(3, 4, 8)) == (3, 4, 8, 8, 0, 0, 32)
    assert fields(RowBlocks(W.view(2, 3, 2, 8)[:, 0])) == (1, 4, 8, 8, 2, 48, 0)
    assert fields(torch.zeros(4, 6, 10)[:, :, 5:]) == (4, 6, 5, 10, 0, 0, 60)


def test_singleton_dimensions_take_dense_strides():
    assert fields(torch.zeros(1, 5)) == (1, 1, 5, 5, 0, 0, 0)
    assert fields(torch.zeros(7, 1)) == (1, 7, 1, 1, 0, 0, 0)
    one_row_blocks = RowBlocks(torch.zeros(3, 1, 16))  # 3 blocks of 1 row
    assert fields(one_row_blocks) == (1, 3, 16, 16, 1, 16, 0)


@pytest.mark.parametrize("make", [
    lambda: torch.zeros(1, 8).expand(16, 8),               # rows share storage
    lambda: torch.zeros(8, 8).as_strided((8, 8), (4, 1)),  # rows overlap
    lambda: torch.zeros(1, 4, 8).expand(3, 4, 8),          # planes share storage
    lambda: RowBlocks(torch.zeros(1, 2, 8).expand(3, 2, 8)),  # blocks share storage
])
def test_overlapping_layouts_are_refused(make):
    with pytest.raises(ValueError):
        _view(make())


def test_columns_must_be_contiguous():
    with pytest.raises(ValueError):
        _view(torch.zeros(8, 8).t())


def test_tensors_off_the_handles_device_are_refused():
    from paper_2609_21594_amd.binding import _check_device
    W = torch.zeros(4, 8)
    with pytest.raises(ValueError, match="cuda:0"):
        _check_device([W], 0)
    with pytest.raises(ValueError):
        _check_device([RowBlocks(W.view(2, 2, 8))], 0)
    _check_device([], 0)


def test_coefficient_tables_must_match_the_step_count():
    # the library reads 3 * ns_steps values from the table
    from paper_2609_21594_amd.binding import make_hparams
    make_hparams(ns_coeffs=[(1.5, -0.5, 0.0)] * 3, ns_steps=3)
    with pytest.raises(ValueError):
        make_hparams(ns_coeffs=[(1.5, -0.5, 0.0)] * 2, ns_steps=3)
    with pytest.raises(ValueError):
        make_hparams(ns_coeffs=[(1.5, -0.5)] * 3, ns_steps=3)


def test_optimizer_needs_gpu_parameters():
    from paper_2609_21594_amd.optim import MuonAdamW
    with pytest.raises(ValueError, match="one GPU"):
        MuonAdamW([torch.nn.Parameter(torch.zeros(4, 4))])


def test_plain_entries_pack_the_same_structs_as_the_general_path():
    """Calls whose entries are all contiguous take a packed path: it must give
    the bytes that the general path gives, and hand over every other call."""
    import ctypes
    import torch
    from paper_2609_21594_amd import binding as B
    assert B._PARAM_PACK.size == ctypes.sizeof(B.MuonParam)
    shapes = [(4, 6), (1, 5), (5, 1), (1, 1), (3, 4, 6), (1, 4, 6), (3, 1, 6), (2, 6, 1)]
    for pd, gd in ((torch.float32, torch.float32), (torch.bfloat16, torch.float32), (torch.bfloat16, torch.bfloat16)):
        W = [torch.zeros(s, dtype=pd) for s in shapes]
        g = [torch.zeros(s, dtype=gd) for s in shapes]
        m = [torch.zeros(s) for s in shapes]
        assert B._plain_params(W, g, m) is not None
        fast, _ = B.params_array(W, g, m)
        slow, _ = B.params_array(W, g, m, entry_coeffs=[None] * len(shapes))
        assert bytes(fast) == bytes(slow)
    W, g, m = torch.zeros(4, 6), torch.zeros(4, 6), torch.zeros(4, 6)
    wide = torch.zeros(4, 8)[:, :6]
    others = [([wide], [torch.zeros(4, 8)[:, :6]], [m]), ([W], [g], [torch.zeros(1, 4, 6)]),
              ([B.RowBlocks(torch.zeros(2, 2, 6))], [B.RowBlocks(torch.zeros(2, 2, 6))], [m]),
              ([torch.zeros(0, 6)], [torch.zeros(0, 6)], [torch.zeros(0, 6)])]
    for p, q, r in others:
        assert B._plain_params(p, q, r) is None
    for bad in (([W], [torch.zeros(6, 4)], [m]), ([W.double()], [g], [m]), ([W], [g], [m.bfloat16()]),
                ([W.t()], [g.t()], [m.t()])):
        assert B._plain_params(*bad) is None
        with pytest.raises((ValueError, TypeError)):
            B.params_array(*bad)


def test_subclass_of_row_blocks_takes_the_general_path():
    import torch
    from paper_2609_21594_amd import binding as B

    class Heads(B.RowBlocks):
        pass

    for wrap in (B.RowBlocks, Heads):
        W, g, m = torch.zeros(2, 3, 2, 6)[:, 0], torch.zeros(2, 3, 2, 6)[:, 0], torch.zeros(4, 6)
        for momentum in (m, wrap(torch.zeros(2, 3, 2, 6)[:, 0])):
            arr, _ = B.params_array([wrap(W)], [wrap(g)], [momentum])
            assert (arr[0].rows, arr[0].cols) == (4, 6)
