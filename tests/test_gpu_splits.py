"""GPU parity of the 16-bit attention path where the number of (query, kv head) units does not divide the 256 compute units:
batches on both sides of the points where a call goes from three splits to two and from two to one."""

import pytest

from paper_2502_11101_amd import workloads as wl
from tests.test_gpu_parity import _run_single_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,hkv", [(17, 5), (43, 2), (16, 8), (43, 3), (15, 17)])     # 85, 86, 128, 129, 255 units
def test_split_counts(batch, hkv):
    cfg = wl.scaled(wl.CONFIGS["tiny_f32"], name=f"splits_{batch * hkv}", geometry=wl.Geometry(2 * hkv, hkv, 128, "bf16", 1.0e4, 8192),
                    n_store_docs=batch * 2, docs_per_query=2, batch=batch, doc_len_range=(90, 200), tq=24, prefix_len=32,
                    doc_stored_start=32, n_planted=1)
    # few rows and tokens: the plain oracle's masses to the bound of the other edge shapes, the rounded-key reference's tight
    _run_single_layer(cfg, seed=batch, mass_tol=2e-3, layout="head")
