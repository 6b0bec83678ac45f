"""Rows whose first visible key lies in their wave's second tile.

With ALiBi or SoftCap, whole key tiles after a wave's first one fold each
row's reference maximum into the scores, which needs every row to have seen a
key.  One row of every 32-row wave has seen none after the first tile when the
window's lower edge (keys run forward: SoftCap) or the causal diagonal (keys
run backward: ALiBi) of that row falls on a tile boundary: with
Lk - Lq - window a multiple of 32, or Lk - Lq one less than a multiple of 32.
Each row is compared by itself, so that one wrong row in 32 shows."""

import numpy as np
import pytest

import paper_2510_08726_amd as pa
from paper_2510_08726_amd.workloads import alibi_slopes, random_tensors
from gpu_common import host32, oracle_fwd, run_fwd

pytestmark = pytest.mark.gpu

CASES = [  # B, Hq, Hkv, Lq, Lk, D, dtype, alibi, softcap, window
    (1, 4, 2, 333, 333, 128, "f16", False, 50.0, 64),
    (1, 4, 4, 200, 360, 64, "f16", False, 5.0, 96),      # Lk - Lq - window = 64
    (1, 2, 1, 100, 131, 128, "bf16", False, 50.0, 31),   # 0, the window as long as the offset
    (1, 4, 4, 300, 331, 128, "f16", True, None, None),
    (2, 4, 1, 129, 192, 64, "bf16", True, None, None),
    (1, 4, 2, 170, 297, 64, "f16", True, None, 50),
    (1, 4, 4, 170, 201, 128, "f16", True, None, 32),
]


# The batch is repeated until the items outnumber the compute units, so that
# prefill_kernel runs; as they are, the small cases run the split kernel.
WIDE = 140


@pytest.mark.parametrize("wide", [True, False], ids=["wide", "small"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_rows_that_see_nothing_of_the_first_tile(case, wide):
    B, Hq, Hkv, Lq, Lk, D, dt, alibi, cap, win = case
    assert (Lk - Lq) % 32 == 31 if alibi else (Lk - Lq - win) % 32 == 0
    print(f"first-tile case {case} {wide}", flush=True)
    q, k, v = random_tensors([(B, Hq, Lq, D), (B, Hkv, Lk, D), (B, Hkv, Lk, D)], dt, seed=Lq + Lk)
    sl = alibi_slopes(Hq) if alibi else None
    kw = dict(scale=D ** -0.5, causal=True, slopes=sl, softcap=cap, window=win)
    R = WIDE if wide else 1
    if wide:
        name = pa.attn_fwd_call_kernels(B * R, Hq, Hkv, Lq, Lk, D, q.dtype, True, alibi, cap, win)
        assert name == [f"prefill_kernel<{D},{dt},1,{int(alibi)},{int(bool(cap))},{int(bool(win))}>"]
    o = run_fwd(*(t.repeat(R, 1, 1, 1) for t in (q, k, v)), **kw)
    assert all((o[b * B:(b + 1) * B] == o[:B]).all() for b in range(1, R))
    got, ref = host32(o[:B]).astype(np.float64), oracle_fwd(q, k, v, **kw)
    row = np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    # P and O are each rounded to the input type: at most half an ulp per
    # value, 2^-11 (fp16) or 2^-8 (bf16), in weights and output together twice
    # that; weights computed against no reference miss by tens of per cent.
    assert row.max() <= 2 * (2.0 ** -11 if dt == "f16" else 2.0 ** -8), (case, row.max(), np.argwhere(row > 1e-2)[:5])
