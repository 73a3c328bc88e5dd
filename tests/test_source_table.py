"""Columns of a SourceTable are tensors of their own: a program may write
into one, differentiate through another, keep, save or resize one, and the
others know nothing of it.  (On the CPU: the binding's buffers only.)"""
import io

import torch

import paper_2502_10783_amd as ipp
from paper_2502_10783_amd import _lib as L


def _table(capacity=1000, n_frames=2):
    return ipp.SourceTable(capacity, n_frames, "cpu")


def _all(t):
    return list(t.cols.values()) + [t.n_total, t.frame_offsets]


def test_columns_start_at_zero_with_their_types():
    for capacity in (0, 1, 63, 64, 65, 1000):
        t = _table(capacity)
        assert list(t.cols) == [name for name, _ in L.SOURCE_COLUMNS]
        for name, dt in L.SOURCE_COLUMNS:
            c = t.cols[name]
            assert c.dtype == ipp.SourceTable.DT[dt]
            assert c.shape == (max(1, capacity),) and c.is_contiguous()
            assert not c.any()
        assert t.n_total.shape == (1,) and t.frame_offsets.shape == (3,)
        assert t.n_total.dtype == t.frame_offsets.dtype == torch.int64
        assert t.count() == 0 and not t.frame_offsets.any()


def test_a_column_takes_values_that_require_gradients():
    t = _table()
    x = torch.linspace(0.0, 9.0, 1000, dtype=torch.float64,
                       requires_grad=True)
    t.cols["x"].copy_(x)
    t.cols["y"][:10] = x[:10]
    (t.cols["x"].sum() + t.cols["y"].sum()).backward()
    want = torch.ones(1000, dtype=torch.float64)
    want[:10] = 2.0
    assert torch.equal(x.grad, want)


def test_a_column_may_be_written_while_a_graph_holds_another():
    t = _table()
    w = torch.ones(1000, dtype=torch.float64, requires_grad=True)
    t.cols["flux_ap"].fill_(2.0)
    y = (t.cols["flux_ap"] * w).sum()
    t.cols["x"].fill_(3.0)
    t.cols["flags"].fill_(1)
    t.frame_offsets.fill_(4)
    y.backward()
    assert torch.equal(w.grad, torch.full_like(w, 2.0))


def test_a_column_has_its_own_storage():
    t = _table()
    assert len({c.untyped_storage().data_ptr() for c in _all(t)}) == len(_all(t))
    f = io.BytesIO()
    torch.save(t.cols["x"], f)
    assert f.tell() < 2 * 8 * 1000
    t.cols["x"].resize_(4000).fill_(7.0)
    assert all(not c.any() for k, c in t.cols.items() if k != "x")
