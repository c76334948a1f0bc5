"""Values on the attention path outside the 16-bit kernels' shapes, on tables made by hand: what must come out exactly, and what
must not be lost."""

import numpy as np
import pytest
import torch

from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import pipeline as pl

pytestmark = pytest.mark.gpu

INTER = cf.CF_ROPE_INTERLEAVED
I32 = dict(dtype=torch.int32, device="cuda")
D = 64


def _attend(dtype, q, ks, vs, lens, own=None, tq=1):
    """Every query attends the first sum(lens) tokens of the store as segments of these lengths, nothing moved, then its own block
    (keys, values) if there is one.  One head of D channels.  Returns outputs and masses."""
    batch = q.shape[0] // tq
    n_seg = len(lens) + (own is not None)
    off = np.concatenate([[0], np.cumsum(lens)])
    tables = []
    for b in range(batch):
        tables += [(int(off[i]), int(l), 0, 0, cf.CF_SEG_DOC, i) for i, l in enumerate(lens)]
        if own is not None:
            tables.append((b * tq, tq, 0, 0, cf.CF_SEG_SELF, -1))
    desc = cf.make_desc(1, 1, D, dtype, 1.0e4, 8192, INTER)
    dev = [pl.to_device(np.ascontiguousarray(x), dtype) if x is not None else None for x in (q, ks, vs, *(own or (None, None)))]
    kv = int(off[-1]) + (tq if own is not None else 0)
    ws_bytes = cf.cf_prefill_workspace_bytes(desc, batch, tq, n_seg, kv)
    ws = torch.full((ws_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    out, mass = torch.full_like(dev[0], 7.0), torch.full((batch, n_seg), -1.0, device="cuda")
    flag = torch.zeros(1, **I32)
    cf.cf_prefill_attention(desc, dev[0], torch.arange(0, (batch + 1) * tq, tq, **I32), 0, torch.zeros(batch, **I32), dev[1], dev[2],
                            ks.shape[0], dev[3], dev[4], cf.segments_to_device(cf.segments_array(tables)),
                            torch.full((batch,), n_seg, **I32), n_seg, batch, tq, kv, out, mass, None, 0, ws, ws_bytes, flag)
    torch.cuda.synchronize()
    assert flag.item() == 0
    return out.float().cpu().numpy(), mass.cpu().numpy()


@pytest.mark.parametrize("far", [0, 700])          # without and with splits to merge
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_the_mass_of_all_a_row_sees_is_one(dtype, far):
    """13 tokens in one tile have the whole weight of the row: sum over sum, which a division gives as exactly 1 (a product with the
    rounded reciprocal misses it by 2^-24 in some rows).  The other tokens' weights are below the smallest fp32 number."""
    rng = np.random.default_rng(13)
    print(f"mass {dtype} far={far}", flush=True)
    q, ks, vs = (rng.standard_normal((n, 1, D), dtype=np.float32) for n in (64, 13 + far, 13 + far))
    q[:, :, 0], ks[:13, :, 0], ks[13:, :, 0] = 8.0, 0.0, -1000.0
    _, mass = _attend(dtype, q, ks, vs, [13, far] if far else [13])
    assert np.array_equal(mass[:, 0], np.ones(64, np.float32))
    assert np.all(mass[:, 1:] == 0.0)


@pytest.mark.parametrize("small", [20, 28, 33, 36])
@pytest.mark.parametrize("far", [0, 700])          # without and with splits to merge
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_small_probabilities_keep_their_bits(dtype, far, small):
    """A token with 2^-small of the largest probability carries the only values there are: the outputs are its products alone,
    and as exact as the type they are stored in."""
    print(f"small {dtype} far={far} 2^-{small}", flush=True)
    n, tokens = 16, 13 + far
    q, ks, vs = np.zeros((n, 1, D), np.float32), np.zeros((tokens, 1, D), np.float32), np.zeros((tokens, 1, D), np.float32)
    q[:, 0, 0] = 1.0 + np.arange(n) / 128.0         # exact in every type
    ks[5, 0, 0] = -np.float32(np.round(small * np.log(2.0) * np.sqrt(D)))
    ks[13:, 0, 0] = -1200.0
    vs[5] = np.where(np.arange(D) % 2, 1.0, -1.5) * 2.0 ** 15
    out, _ = _attend(dtype, q, ks, vs, [13, far] if far else [13])
    s = np.float64(q[:, 0, 0])[:, None] * np.float64(ks[:, 0, 0])[None] / np.sqrt(D)
    p = np.exp(s - s.max(axis=1, keepdims=True))
    ref = (p / p.sum(axis=1, keepdims=True)) @ np.float64(vs[:, 0])
    # scores up to 2^40 apart in fp32 (two roundings of a number below 64), and one rounding of the result (fp16: to multiples of 2^-24
    # below 2^-14)
    bound = np.abs(ref) * ({"f32": 0.0, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype] + 64 * 2.0 ** -23) + (2.0 ** -25 if dtype == "f16" else 0.0)
    assert np.all(np.abs(out[:, 0] - ref) <= bound)
