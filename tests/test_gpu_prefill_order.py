"""The orders in which prefill.hip deals its items out, at the edges of their
rule: heaviest first over all (fewer KV heads and head groups than XCDs), within
each XCD's share (shares that cut a unit), and KV head major where every item
has a compute unit to itself.  Every row has to be written; rows of every block
are compared with the oracle."""

import ctypes

import numpy as np
import pytest
import torch

import paper_2510_08726_amd as pa
from paper_2510_08726_amd.workloads import alibi_slopes, random_tensors
from gpu_common import assert_close, host32, oracle_fwd

pytestmark = pytest.mark.gpu

# B, Hq, Hkv, Lq, Lk, D, dtype, alibi, softcap, window, order
CASES = [
    (1, 2, 2, 16500, 16500, 64, "f16", False, None, None, 2),     # 2 units of 129 blocks: 258 items
    (1, 4, 1, 9000, 9000, 64, "bf16", False, None, 8000, 2),      # 1 unit of 282 blocks
    (3, 1, 1, 13000, 13100, 128, "f16", True, None, None, 2),     # 3 units
    (1, 28, 7, 1201, 1201, 128, "bf16", False, 20.0, None, 2),    # 7 units of 38 blocks: 266
    (1, 24, 6, 3300, 3300, 64, "f16", False, None, None, 2),      # 6 units of 104: 624 items, two rounds
    (1, 32, 8, 1100, 1100, 128, "f16", False, None, None, 1),     # 8 units: the shares are units
    (3, 12, 3, 1600, 1650, 64, "bf16", True, None, 900, 1),       # 9 units: shares cut them
    (5, 13, 13, 600, 600, 128, "f16", False, None, None, 1),      # 65 units of 5 blocks
    (2, 4, 4, 4200, 4200, 64, "f16", False, 10.0, None, 1),       # 8 units of 33: 264 items
    (1, 32, 32, 782, 782, 128, "bf16", False, None, None, 0),     # 224 items
    (300, 1, 1, 100, 100, 64, "f16", False, None, None, 0),       # units of one block
]


def _order(case):
    """The rule's answer, by the sizes that the launcher gives it."""
    B, Hq, Hkv, Lq, Lk, D, dt, alibi, cap, win, _ = case
    f = pa.load_library()._ZN4attn13prefill_orderEiiibiil         # attn::prefill_order
    f.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.c_int, ctypes.c_int, ctypes.c_int64]
    f.restype = ctypes.c_int
    hg = next(h for h in (4, 2, 1) if (Hq // Hkv) % h == 0)
    nqb = -(-Lq // (128 // hg))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return f(nqb * (B * Hq // hg), nqb, 2 * cus, True, win or 0, Lk, B * Hkv * Lk * D * 4)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_every_row_is_written(case):
    B, Hq, Hkv, Lq, Lk, D, dt, alibi, cap, win, order = case
    torch_dt = {"f16": torch.float16, "bf16": torch.bfloat16}[dt]
    assert _order(case) == order
    assert pa.attn_fwd_call_kernels(B, Hq, Hkv, Lq, Lk, D, torch_dt, True, alibi, cap, win)[0].startswith("prefill_kernel")
    print(f"prefill order {case}", flush=True)
    q, k, v = random_tensors([(B, Hq, Lq, D), (B, Hkv, Lk, D), (B, Hkv, Lk, D)], dt, seed=Lq)
    sl = alibi_slopes(Hq) if alibi else None
    o = torch.full(q.shape, float("nan"), dtype=q.dtype, device="cuda")
    pa.attn_fwd(q.cuda(), k.cuda(), v.cuda(), o, causal=True, scale=D ** -0.5, alibi_slopes=None if sl is None else sl.cuda(),
                softcap=cap, window=win)
    torch.cuda.synchronize()
    assert not torch.isnan(o).any()
    heads = [(b, h) for b in {0, B // 2, B - 1} for h in {0, Hq // 3, Hq - 1}]
    rows = np.unique(np.concatenate([np.arange(0, Lq, 32), np.arange(19, Lq, 128), [Lq - 1]]))
    if len(rows) > 200:
        rows = rows[np.random.default_rng(Lq).choice(len(rows), 200, replace=False)]
    ref = oracle_fwd(q, k, v, scale=D ** -0.5, causal=True, slopes=sl, softcap=cap, window=win, rows=rows, heads=heads)
    got = host32(o)[:, :, rows]
    for b, h in heads:
        assert_close(got[b, h], ref[b, h], f"prefill order {case}, batch {b}, head {h}")
