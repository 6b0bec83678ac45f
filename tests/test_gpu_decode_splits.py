"""The library's chunk counts at the edges of their rule (workgroups just below
and above the compute units), the combine of few, many and empty chunks, and a
workspace kept from a smaller chunk count."""

import pytest
import torch

import paper_2510_08726_amd as pa
from paper_2510_08726_amd.workloads import random_tensors
from gpu_common import assert_close, host32, oracle_fwd

pytestmark = pytest.mark.gpu


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def test_grouped_chunks_fill_one_round():
    cu = _cus()
    for B in (1, 5, 6, 11, 16, 17):
        S = pa.attn_decode_num_splits(B, 64, 16, 1 << 20, 128)
        assert S == max(cu // (16 * B), 1) and (B * 16 > cu or B * 16 * S <= cu)


# B, Hq, Hkv, Lk, D, dtype, num_splits
CASES = [(6, 16, 8, 700, 128, "f16", 0), (11, 32, 16, 300, 64, "bf16", 0), (3, 12, 12, 3000, 64, "f16", 0),
         (9, 16, 16, 1000, 128, "bf16", 0), (2, 8, 2, 500, 128, "f16", 7), (2, 4, 4, 500, 64, "f16", 33),
         (1, 4, 2, 90, 128, "bf16", 90), (1, 4, 4, 40, 64, "bf16", 300), (1, 8, 2, 2000, 64, "f16", 65)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_chunks_and_combine(case):
    B, Hq, Hkv, Lk, D, dt, S = case
    print(f"decode chunks {case}", flush=True)
    q, k, v = random_tensors([(B, Hq, 1, D), (B, Hkv, Lk, D), (B, Hkv, Lk, D)], dt, seed=Lk)
    o = pa.attn_decode(q.cuda(), k.cuda(), v.cuda(), scale=D ** -0.5, num_splits=S)
    torch.cuda.synchronize()
    assert_close(host32(o), oracle_fwd(q, k, v, scale=D ** -0.5, causal=True), f"decode {case}")


def test_workspace_kept_from_a_smaller_chunk_count():
    cu = _cus()
    B, H, Lk, D = 3, 32, 4000, 64                                   # 96 heads: 5 chunks of 256 compute units, once 3
    q, k, v = (t.cuda() for t in random_tensors([(B, H, 1, D), (B, H, Lk, D), (B, H, Lk, D)], "f16", seed=3))
    S, kept = pa.attn_decode_num_splits(B, H, H, Lk, D), -(-cu // (B * H))
    ref = pa.attn_decode(q, k, v, num_splits=kept)
    ws = torch.empty(pa.attn_decode_workspace_bytes(B, H, D, kept), dtype=torch.uint8, device="cuda")
    assert torch.equal(pa.attn_decode(q, k, v, workspace=ws), ref if S > kept else pa.attn_decode(q, k, v))
    if kept > 1:
        with pytest.raises(pa.AttnError):
            pa.attn_decode(q, k, v, workspace=ws[:ws.numel() - 256])


@pytest.mark.parametrize("case", [(1, 4, 2, 2500, 128, 7), (1, 4, 4, 700, 64, 3), (2, 8, 2, 90, 64, 90), (1, 4, 2, 2500, 64, 16)],
                         ids=lambda c: "x".join(map(str, c)))
def test_infinite_values_in_the_last_chunk(case):
    """Chunk counts that leave lanes of the combine without a chunk: infinite
    values stay infinite (every weight is above 0), the other dims are as
    without them."""
    B, Hq, Hkv, Lk, D, S = case
    print(f"decode infinities {case}", flush=True)
    q, k, v = random_tensors([(B, Hq, 1, D), (B, Hkv, Lk, D), (B, Hkv, Lk, D)], "f16", seed=Lk)
    v[..., -1, 5], v[..., -1, 6] = float("inf"), float("-inf")
    o = host32(pa.attn_decode(q.cuda(), k.cuda(), v.cuda(), num_splits=S))
    assert (o[..., 5] == float("inf")).all() and (o[..., 6] == float("-inf")).all()
    v[..., 5:7] = 0.0
    o[..., 5:7] = 0.0
    assert_close(o, oracle_fwd(q, k, v, scale=D ** -0.5, causal=True), f"decode infinities {case}")


@pytest.mark.parametrize("case", [(11, 24, 12, 1500, "f16"), (3, 64, 32, 2600, "bf16"), (1, 8, 2, 150000, "f16")],
                         ids=lambda c: "x".join(map(str, c)))
def test_grouped_chunks_at_head_dim_64(case):
    """Two workgroups per compute unit (D = 64, long chunks), and a workspace
    for one: each against the oracle."""
    B, Hq, Hkv, Lk, dt = case
    cu = _cus()
    S, one = pa.attn_decode_num_splits(B, Hq, Hkv, Lk, 64), max(cu // (B * Hkv), 1)
    print(f"decode D 64 {case} {S} chunks, {one}", flush=True)
    if Lk / one >= 1200:
        assert S == 2 * cu // (B * Hkv)
    q, k, v = random_tensors([(B, Hq, 1, 64), (B, Hkv, Lk, 64), (B, Hkv, Lk, 64)], dt, seed=Lk)
    ref = oracle_fwd(q, k, v, scale=0.125, causal=True)
    q, k, v = q.cuda(), k.cuda(), v.cuda()
    assert_close(host32(pa.attn_decode(q, k, v)), ref, f"decode {case}, {S} chunks")
    ws = torch.empty(pa.attn_decode_workspace_bytes(B, Hq, 64, one), dtype=torch.uint8, device="cuda")
    o = pa.attn_decode(q, k, v, workspace=ws)
    assert torch.equal(o, pa.attn_decode(q, k, v, num_splits=one))
    assert_close(host32(o), ref, f"decode {case}, {one} chunks")


def test_output_at_any_element():
    """O may begin at any element (the combine stores 8 bytes a lane)."""
    q, k, v = (t.cuda() for t in random_tensors([(2, 8, 1, 64), (2, 2, 900, 64), (2, 2, 900, 64)], "f16", seed=4))
    ref = pa.attn_decode(q, k, v, num_splits=5)
    for shift in (1, 2, 3):
        o = torch.zeros(q.numel() + 8, dtype=q.dtype, device="cuda")
        part = o[shift:shift + q.numel()].view(q.shape)
        assert torch.equal(pa.attn_decode(q, k, v, part, num_splits=5), ref)
        assert not o[:shift].any() and not o[shift + q.numel():].any()
