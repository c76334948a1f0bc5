"""cf_prefill_attention_static near its 32 MiB, on the shapes outside the 16-bit kernels': long tables and single rows, whose
plans must not be charged for the rows a block is padded to, and a shape that only the row-by-row kernel can serve."""

import numpy as np
import pytest
import torch

from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import pipeline as pl

HALF, INTER = cf.CF_ROPE_HALF, cf.CF_ROPE_INTERLEAVED

# dtype, pairing, heads, head size, queries, rows, table stride; every row has an entry of each table: (rows * (stride + 1)) * 8 bytes
SERVED = [("bf16", INTER, 32, 128, 64, 1, 128), ("bf16", INTER, 32, 128, 32, 1, 256), ("f32", HALF, 32, 128, 16, 130, 58)]
# one row per kv head: the slots' sums in double are as large as the statistics, and the plan is past the buffer
ROW_BY_ROW = ("f32", HALF, 64, 16, 256, 1, 250)


def _desc(dtype, pairing, heads, d):
    return cf.make_desc(heads, heads, d, dtype, 1.0e4, 4096, pairing)


def _rows_bytes(dtype, pairing, heads, d, batch, tq, stride):
    return batch * tq * heads * (stride + 1) * 8


@pytest.mark.parametrize("shape", SERVED)
def test_plans_of_long_tables_fit_where_the_row_by_row_kernel_did(shape):
    *head, batch, tq, stride = shape
    assert _rows_bytes(*shape) <= cf.CF_STATIC_SCRATCH_BYTES
    assert 0 < cf.cf_prefill_workspace_bytes(_desc(*head), batch, tq, stride, 3000) <= cf.CF_STATIC_SCRATCH_BYTES


def test_a_plan_past_the_buffer_that_the_row_by_row_kernel_fits():
    *head, batch, tq, stride = ROW_BY_ROW
    assert _rows_bytes(*ROW_BY_ROW) <= cf.CF_STATIC_SCRATCH_BYTES < cf.cf_prefill_workspace_bytes(_desc(*head), batch, tq, stride, 260)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SERVED + [ROW_BY_ROW])
def test_static_entry_serves_them(shape):
    dtype, pairing, heads, d, batch, tq, stride = shape
    print(f"static {shape}", flush=True)
    desc = _desc(dtype, pairing, heads, d)
    docs = stride - 2
    rng = np.random.default_rng(stride)
    lens = rng.integers(1, 4, size=(batch, docs))
    n_store = 600
    off = rng.integers(4, n_store - 4, size=(batch, docs))
    pb = pl.PrefillBatch(desc, off, lens, tq, 4, 4, n_store)
    gen = torch.Generator(device="cuda").manual_seed(stride)
    normal = lambda n: torch.randn((n, heads, d), generator=gen, device="cuda").to(pl.TORCH_DTYPE[dtype])
    q, k1, v1 = (normal(batch * tq) for _ in range(3))
    ks, vs = normal(n_store), normal(n_store)
    pb.allocate_initial()
    res = []
    for static in (False, True):
        out, mass, score = torch.full_like(q, 7.0), torch.full_like(pb.mass, -1.0), torch.zeros_like(pb.score)
        args = (desc, q, pb.q_off, 0, pb.q_start, ks, vs, n_store, k1, v1, pb.segs, pb.n_seg, stride, batch, tq, pb.max_kv_tokens, out,
                mass, score, pb.stride)
        if static:
            cf.cf_prefill_attention_static(*args, pb.dev_flag)
        else:
            pb.workspace.fill_(0xFF)
            cf.cf_prefill_attention(*args, pb.workspace, pb.ws_bytes, pb.dev_flag)
        torch.cuda.synchronize()
        assert pb.flags() == 0
        res.append((out, mass, score))
    if shape == ROW_BY_ROW:                  # two kernels, both fp32 throughout: sums of some 500 terms in another order
        for a, b in zip(*res):
            assert (a - b).abs().max() <= 1e-5 * a.abs().max()
    else:
        for a, b in zip(*res):
            assert torch.equal(a, b)
    assert torch.allclose(res[0][1].sum(dim=1), torch.full((batch,), float(heads * tq), device="cuda"), rtol=1e-5)
