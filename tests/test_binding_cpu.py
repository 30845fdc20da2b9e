"""Argument checks of the Python binding (CPU only, nothing is launched).

The C ABI receives raw pointers, so the binding refuses tensors whose element type,
size or device the library would misread: an fp16 tensor read as float32, int64
positions read as pairs of int32, or a host pointer handed to a kernel."""
import pytest
import torch

import paper_2609_33334_amd as dge


def test_rope_refuses_fp16_rows():
    x = torch.zeros(2, 8, 128, dtype=torch.float16)
    with pytest.raises(TypeError, match="bfloat16 or float32"):
        dge.rope(x, torch.arange(8, dtype=torch.int32))


def test_rope_refuses_int64_positions():
    x = torch.zeros(2, 8, 128, dtype=torch.bfloat16)
    with pytest.raises(TypeError, match="int32"):
        dge.rope(x, torch.arange(8))


def test_rope_refuses_short_positions_and_host_tensors():
    x = torch.zeros(2, 8, 128, dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="at least 8"):
        dge.rope(x, torch.arange(5, dtype=torch.int32))
    with pytest.raises(ValueError, match="needs a GPU tensor"):
        dge.rope(x, torch.arange(8, dtype=torch.int32))


def test_score_refuses_wrong_dtype_size_and_device():
    g = dge.Geometry(4, 2, 64, 2, 1, [40, 50], dtype=dge.DGE_BF16, device="cpu")
    q = torch.zeros(4, 2 * 3, 64, dtype=torch.bfloat16)
    k = torch.zeros(2, 90, 64, dtype=torch.bfloat16)
    raw = torch.zeros(2, 90, dtype=torch.float32)
    with pytest.raises(TypeError, match="dtype"):
        dge.score(g, dge.ROWS_WINDOW_DRAFT, q.float(), k, raw=raw)
    with pytest.raises(ValueError, match="elements"):
        dge.score(g, dge.ROWS_WINDOW_DRAFT, q, k[:, :60].contiguous(), raw=raw)
    with pytest.raises(ValueError, match="needs a GPU tensor"):
        dge.score(g, dge.ROWS_WINDOW_DRAFT, q, k, raw=raw)


@pytest.mark.parametrize("full", [False, True])
def test_score_allocates_for_its_rows(monkeypatch, full):
    """Without a workspace, score takes what its own row mode uses (scores by window rows never
    keep logits, however large K is), and the partials alone where the device is full."""
    g = dge.Geometry(1024, 256, 128, 32, 2, [16384], dtype=dge.DGE_BF16, device="cpu")
    got = []
    empty = torch.empty

    def alloc(*shape, **kw):
        if kw.get("dtype") is torch.uint8:
            got.append(shape[0])
            if full and shape[0] > 64 << 20:
                raise torch.OutOfMemoryError("full")
            return empty(16, **kw)
        return empty(*shape, **kw)

    monkeypatch.setattr(torch, "empty", alloc)
    monkeypatch.setattr(dge, "_need", lambda *a, **kw: None)
    for call in (dge.score, dge.score_with_lse):
        for rows in (dge.ROWS_WINDOW_DRAFT, dge.ROWS_WINDOW, dge.ROWS_DRAFT):
            got.clear()
            with pytest.raises(ValueError, match="needs a GPU tensor"):
                call(g, rows, empty(4), empty(4), raw=empty(4))
            if rows != dge.ROWS_DRAFT:
                assert len(got) == 1 and got[0] < 16 << 20
            else:
                assert got[0] > 128 << 20 and got[1:] == ([dge.score_workspace_size(g, rows)[1]] if full else [])


def test_select_and_compact_refuse_wrong_index_types():
    g = dge.Geometry(4, 2, 64, 2, 1, [40, 50], dtype=dge.DGE_F32, device="cpu")
    scores = torch.zeros(2, 90, dtype=torch.float32)
    with pytest.raises(TypeError, match="dtype"):
        dge.select_topb(g, scores.double(), 1, 3, 4, idx=torch.zeros(2, 2, 4, dtype=torch.int32),
                        n_kept=torch.zeros(2, dtype=torch.int32))
    k = torch.zeros(2, 90, 64)
    with pytest.raises(TypeError, match="dtype"):
        dge.compact(g, torch.zeros(2, 2, 4, dtype=torch.int64), torch.zeros(2, dtype=torch.int32),
                    4, 3, k, k, k_out=torch.zeros(2, 2, 7, 64), v_out=torch.zeros(2, 2, 7, 64))
