"""Prompts with few query rows (keys split inside the workgroup, and with a
workspace over workgroups), at the sizes where that can go wrong: one row,
row blocks of 32 and pairs of them, groups of one, an odd and an even number of
heads, key groups and key ranges without keys, rows without keys; and the wide
kernel at small ragged sizes, with enough heads that it runs."""

import ctypes

import numpy as np
import pytest
import torch

import paper_2510_08726_amd as pa
from paper_2510_08726_amd.workloads import alibi_slopes, random_tensors
from gpu_common import MEAN_ABS, assert_close, host32, oracle_fwd, run_fwd
from kernel_cases import PREFILL_SPLIT_CASES, PREFILL_VARIANT_CASES, WIDE_BATCH, case_id

pytestmark = pytest.mark.gpu

# B, Hq, Hkv, Lq, Lk, D, dtype, causal, alibi, softcap, window
# (Edges; PREFILL_SPLIT_CASES has every instantiation.)
CASES = [
    (1, 4, 2, 1, 1, 128, "f16", True, False, None, None),
    (1, 4, 4, 33, 31, 64, "bf16", True, False, None, None),       # rows without keys, odd block pair
    (2, 6, 2, 32, 129, 128, "bf16", True, False, None, None),     # 3 heads per KV head: row pairs
    (1, 4, 1, 65, 200, 64, "f16", False, False, None, None),
    (1, 2, 2, 64, 2500, 128, "f16", True, False, None, None),     # key ranges over workgroups
    (1, 8, 2, 31, 4100, 64, "bf16", True, True, None, None),
    (1, 4, 2, 40, 3001, 128, "f16", True, False, 4.0, None),
    (1, 4, 4, 70, 3000, 64, "f16", True, False, None, 1500),
    (1, 4, 2, 70, 3000, 128, "bf16", True, False, 5.0, 2047),
    (1, 4, 2, 70, 3031, 128, "f16", True, True, None, 2000),
    (1, 2, 1, 100, 5000, 128, "bf16", False, True, None, None),
    (2, 4, 2, 2100, 40, 64, "f16", True, False, None, None),      # most rows without keys
    (1, 16, 8, 700, 900, 64, "bf16", False, False, None, None),
    (2, 12, 3, 33, 2600, 128, "f16", True, False, None, None),    # 4 heads per KV head
]


def _inputs(case):
    B, Hq, Hkv, Lq, Lk, D, dt, causal, alibi, cap, win = case
    q, k, v = random_tensors([(B, Hq, Lq, D), (B, Hkv, Lk, D), (B, Hkv, Lk, D)], dt, seed=Lq + Lk)
    if cap:
        q = (q.float() * 4).to(q.dtype)
    return q, k, v, alibi_slopes(Hq) if alibi else None


def _ranges(case):
    B, Hq, Hkv, Lq, Lk, D, dt, causal, alibi, cap, win = case
    return pa.load_library().attn_fwd_num_splits(B, Hq, Hkv, Lq, Lk, D, int(causal), win or 0)


def _assert_rounded(got, ref, mag, dt, what):
    """Each output within what rounding gives: the weights are rounded to the
    input type (in the numerator and in the sum: 2 u sum p |v|), the output
    again (u |o|), with u = 2^-11 (fp16) or 2^-8 (bf16); 2e-5 for fp32 sums of
    values up to 5.  For ALiBi in bf16, whose steep slopes leave few keys their
    weight, so that outputs are as large as values of V and half an ulp alone
    is up to 2^-6."""
    u = 2.0 ** -11 if dt == "f16" else 2.0 ** -8
    d = np.abs(got.astype(np.float64) - ref) - (u * np.abs(ref) + 2 * u * mag + 2e-5)
    assert d.max() <= 0, (what, d.max())
    assert np.abs(got - ref).mean() <= MEAN_ABS, what


def test_some_cases_use_key_ranges():
    assert sum(_ranges(c) > 1 for c in CASES) >= 5 and sum(_ranges(c) == 1 for c in CASES) >= 4


@pytest.mark.parametrize("case", CASES + PREFILL_SPLIT_CASES, ids=case_id)
def test_few_rows_match_the_oracle(case):
    B, Hq, Hkv, Lq, Lk, D, dt, causal, alibi, cap, win = case
    print(f"prefill split case {case}, {_ranges(case)} key ranges", flush=True)
    q, k, v, sl = _inputs(case)
    kw = dict(scale=D ** -0.5, causal=causal, slopes=sl, softcap=cap, window=win)
    ref = oracle_fwd(q, k, v, **kw)
    o = run_fwd(q, k, v, **kw)
    if alibi and dt == "bf16":
        mag = oracle_fwd(q, k, v.abs(), **kw)
        close = lambda got, what: _assert_rounded(got, ref, mag, dt, what)
    else:
        close = lambda got, what: assert_close(got, ref, what)
    close(host32(o), f"prefill split {case}")
    assert torch.equal(o, run_fwd(q, k, v, **kw))                 # the same bits again
    # Without a workspace the keys stay in one range.
    dev, vp = torch.device("cuda"), ctypes.c_void_p
    qd, kd, vd = q.to(dev), k.to(dev), v.to(dev)
    sd = None if sl is None else sl.to(dev)
    o1 = torch.full_like(qd, float("nan"))
    rc = pa.load_library().attn_fwd_mod(vp(qd.data_ptr()), vp(kd.data_ptr()), vp(vd.data_ptr()), vp(o1.data_ptr()), B, Hq,
                                        Hkv, Lq, Lk, D, int(causal), D ** -0.5, None if sd is None else vp(sd.data_ptr()),
                                        float(cap or 0), win or 0, 0 if dt == "f16" else 1,
                                        vp(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert rc == 0
    close(host32(o1), f"prefill split {case}, one range")


def test_negative_and_zero_scale_and_constant_values():
    q, k, v, _ = _inputs((1, 4, 2, 50, 3000, 128, "f16", True, False, None, None))
    for scale in (-0.05, 0.0):
        ref = oracle_fwd(q, k, v, scale=scale, causal=True)
        assert_close(host32(run_fwd(q, k, v, scale=scale, causal=True)), ref, f"scale {scale}")
    one = torch.full_like(v, 1.5)
    assert torch.all(run_fwd(q, k, one, scale=0.1, causal=True) == 1.5)


@pytest.mark.parametrize("case", PREFILL_VARIANT_CASES, ids=case_id)
def test_wide_kernel_at_small_ragged_sizes(case):
    """The small cases of every prefill kernel, with the batch repeated until
    the wide kernel runs; a few (batch, head) slices against the oracle, the
    repeats bit for bit."""
    B, Hq, Hkv, Lq, Lk, D, dt, causal, alibi, cap, win = case
    R = WIDE_BATCH
    q, k, v, sl = _inputs(case)
    dev = torch.device("cuda")
    rep = [t.to(dev).repeat(R, 1, 1, 1) for t in (q, k, v)]
    hg = next(h for h in (4, 2, 1) if (Hq // Hkv) % h == 0)
    assert -(-Lq // (128 // hg)) * (R * Hq // hg) > 256          # past any threshold of the narrow path
    o = pa.attn_fwd(*rep, causal=causal, scale=D ** -0.5, alibi_slopes=None if sl is None else sl.to(dev), softcap=cap,
                    window=win)
    torch.cuda.synchronize()
    for b in range(1, R):
        assert torch.equal(o[b], o[0]), b
    ref = oracle_fwd(q, k, v, scale=D ** -0.5, causal=causal, slopes=sl, softcap=cap, window=win)
    assert_close(host32(o[:1]), ref, f"wide kernel {case}")


def test_capture_in_a_graph_with_key_ranges():
    case = CASES[4]
    q, k, v, _ = _inputs(case)
    assert _ranges(case) > 1
    q, k, v = q.cuda(), k.cuda(), v.cuda()
    eager = pa.attn_fwd(q, k, v, causal=True)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        o = pa.attn_fwd(q, k, v, causal=True)
    for _ in range(3):
        o.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, eager)
        assert torch.equal(pa.attn_fwd(q, k, v, causal=True), eager)


def test_runs_without_memory_for_the_workspace():
    case = (1, 32, 8, 64, 16000, 128, "f16", True, False, None, None)
    S = _ranges(case)
    assert S > 1
    q, k, v, _ = _inputs(case)
    q, k, v = q.cuda(), k.cuda(), v.cuda()
    ref, o, one = pa.attn_fwd(q, k, v, causal=True), torch.empty_like(q), torch.empty_like(q)
    rc = pa.load_library().attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), one.data_ptr(), 1, 32, 8, 64, 16000, 128, 1,
                                    128 ** -0.5, None, 0, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0 and not torch.equal(one, ref)                  # one range has other bits
    torch.cuda.empty_cache()
    held = torch.cuda.memory_reserved()
    nbytes = pa.load_library().attn_fwd_workspace_bytes(1, 32, 64, 128, S)
    try:                                     # the allocator refuses what is past what it holds now
        torch.cuda.set_per_process_memory_fraction(held / torch.cuda.get_device_properties(0).total_memory)
        hog = []                             # and what it holds free is taken
        with pytest.raises(torch.cuda.OutOfMemoryError):
            while True:
                hog.append(torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
        assert pa.attn_fwd(q, k, v, o, causal=True) is o
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
        hog.clear()
    assert torch.equal(o, one)
    assert_close(host32(o), host32(ref), "prefill without a workspace")


def test_infinite_values_with_key_ranges():
    """A number of key ranges that leaves lanes of the combine without one:
    infinite values stay infinite (every row sees them, with a weight above 0),
    the other dims are as without them."""
    case = (1, 2, 1, 100, 3000, 128, "bf16", False, False, None, None)
    assert _ranges(case) > 1 and _ranges(case) % 8 != 0
    q, k, v, _ = _inputs(case)
    v[..., -1, 5], v[..., -1, 6] = float("inf"), float("-inf")
    o = host32(run_fwd(q, k, v, scale=0.05))
    assert (o[..., 5] == float("inf")).all() and (o[..., 6] == float("-inf")).all()
    v[..., 5:7] = 0.0
    o[..., 5:7] = 0.0
    assert_close(o, oracle_fwd(q, k, v, scale=0.05), "infinite values")


@pytest.mark.parametrize("B", [1, 70])
@pytest.mark.parametrize("mod", [dict(), dict(softcap=5.0), dict(alibi=True)], ids=str)
def test_windows_past_the_keys(B, mod):
    """A window of at least Lk keys is no window, up to the largest int, also
    for rows before the first key (Lq > Lk): the split and the wide kernel."""
    q, k, v = (t.cuda().repeat(B, 1, 1, 1) for t in random_tensors([(1, 4, 200, 64), (1, 4, 100, 64), (1, 4, 100, 64)], "f16", seed=8))
    mod = dict(mod)
    sl = alibi_slopes(4).cuda() if mod.pop("alibi", False) else None
    ref = pa.attn_fwd(q, k, v, causal=True, alibi_slopes=sl, window=100, **mod)
    plain = pa.attn_fwd(q, k, v, causal=True, alibi_slopes=sl, **mod)
    assert (ref.float() - plain.float()).abs().max() < 4e-3
    for window in (101, 1 << 20, 2 ** 31 - 1):
        assert torch.equal(pa.attn_fwd(q, k, v, causal=True, alibi_slopes=sl, window=window, **mod), ref), window
