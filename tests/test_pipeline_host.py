"""Host side of PrefillBatch.layer: which tables and scalars reach cf_prefill_layer, with the call itself recorded instead
of made.  No GPU: the batch's tables are CPU tensors that nothing reads."""

import gc
import weakref

import numpy as np
import pytest
import torch

from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import pipeline as pl

DESC = cf.make_desc(4, 2, 128, "bf16", 1.0e4, 4096)


@pytest.fixture
def batch(monkeypatch):
    pb = pl.PrefillBatch(DESC, np.arange(6).reshape(2, 3) * 40 + 8, np.full((2, 3), 40), 5, 8, 8, 300, device="cpu")
    pb.calls = []

    def record(desc, q, q_off, q_stored, q_new, ks, vs, n_store, k1, v1, segs, n_seg, seg_stride, n, max_tq, max_kv, out, mass,
               score, score_stride, workspace, ws_bytes, prune=None, dev_flag=None, stream=None, n_pending=0, defer=False):
        step = None if prune is None else cf.cf_prune_step.from_buffer_copy(prune)
        pb.calls.append(dict(q_new=q_new, segs=segs, n_seg=n_seg, workspace=workspace, mass=mass, score=score, step=step))

    monkeypatch.setattr(cf, "cf_prefill_layer", record)
    return pb


def _layer(pb, **kw):
    x = torch.zeros(1)
    pb.layer(x, x, x, x, x, x, keep=2, **kw)
    return pb.calls[-1]


def _address(x):
    return x if isinstance(x, int) else x.data_ptr()


def test_prune_step_takes_the_scalars_of_the_moment(batch):
    """A batch reused after its prefix or document positions changed: the fused prune step must build the next table
    from the new values, also when advance() comes back to an arrangement of the tables that has been used before."""
    first = _layer(batch)["step"]
    assert (first.prefix_len, first.doc_stored_start, first.stride) == (8, 8, 3)
    batch.advance()
    _layer(batch)
    batch.advance()
    batch.prefix_len, batch.doc_stored_start = 0, 16
    again = _layer(batch)["step"]
    assert (again.prefix_len, again.doc_stored_start) == (0, 16)
    batch.doc_stored_start = 24                       # and with no advance() in between
    assert _layer(batch)["step"].doc_stored_start == 24


def test_tables_follow_advance(batch):
    """Every call gets the current tables, and its prune step the other ones to write."""
    for _ in range(5):
        c = _layer(batch)
        assert _address(c["segs"]) == batch.segs.data_ptr() and _address(c["n_seg"]) == batch.n_seg.data_ptr()
        assert _address(c["q_new"]) == batch.q_start.data_ptr() and _address(c["score"]) == batch.score.data_ptr()
        s = c["step"]
        assert (s.cand, s.order, s.next_segs, s.q_start) == tuple(
            t.data_ptr() for t in (batch.cand, batch.order, batch.next_segs, batch.next_q_start))
        batch.advance()


def test_nothing_is_kept_by_a_tensors_identity(batch):
    """After advance() neither a replaced workspace is kept alive nor the old storage of a table that got a new one used."""
    _layer(batch)
    old = weakref.ref(batch.workspace)
    batch.workspace = torch.zeros(batch.ws_bytes, dtype=torch.uint8)
    batch.advance()
    gc.collect()
    assert old() is None
    for _ in range(2):                                # both arrangements seen
        _layer(batch)
        batch.advance()
    keep_alive = batch.mass.data
    batch.mass.data = torch.zeros_like(batch.mass)    # the same tensor object, other memory
    assert _address(_layer(batch)["mass"]) == batch.mass.data_ptr() != keep_alive.data_ptr()
