"""The row kernels at the row lengths where their shape changes (a wave per
row with 1, 2, 4 or 8 vectors a lane; 256, 512 or 1024 lanes with 4 or 16),
one vector below, at and above each, with few rows and with a row for every
compute unit; chunks whose last batch is nearly empty; and the values that a
maximum or a sum can trip over."""

import numpy as np
import pytest
import torch

import paper_2510_08726_amd as pa
from oracle import norms
from paper_2510_08726_amd.workloads import NORM_DTYPES

pytestmark = pytest.mark.gpu

# fp32 sums of at most 2^17 squares in a tree of batches and fp32 divisions:
# a few ulps of fp32 (2^-24) each; y is rounded once more to its own type.
RTOL = 2e-6
RTOL_Y = {"f16": 2.0 ** -11 + RTOL, "bf16": 2.0 ** -8 + RTOL, "f32": RTOL}

EDGES = [1, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16384]
CASES = [(3, v, ("f16", "bf16", "f32")[i % 3]) for i, v in enumerate(EDGES)]
CASES += [(5, v - 1, ("bf16", "f32", "f16")[i % 3]) for i, v in enumerate(EDGES[1:])]
CASES += [(261, v, ("bf16", "f32")[i % 2]) for i, v in enumerate((511, 2049, 4096, 4097, 5001))]


def _rows(N, M, dt, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    x = g.standard_normal(size=(N, M), dtype=np.float32) * np.exp(g.standard_normal((N, 1), dtype=np.float32))
    x[N // 2] = -np.abs(x[N // 2])        # a row whose maximum is negative
    return torch.from_numpy(x).to(NORM_DTYPES[dt])


def _check(x, chunks, dt):
    eps = 1e-6
    out = pa.norm_l2(x.cuda(), chunks=chunks)
    y, m = pa.rmsnorm_rowmax(x.cuda(), eps=eps, chunks=chunks)
    torch.cuda.synchronize()
    x64 = x.double().numpy()
    yr, mr = norms.rmsnorm_rowmax(x64, eps)
    np.testing.assert_allclose(out.cpu().double().numpy(), norms.l2_norm(x64), rtol=RTOL)
    np.testing.assert_allclose(m.cpu().double().numpy(), mr, rtol=RTOL)
    assert np.all(np.abs(y.cpu().double().numpy() - yr) <= RTOL_Y[dt] * np.abs(yr) + 6e-8)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_row_kernels_at_their_edges(case):
    N, nv, dt = case
    print(f"norm rows {case}", flush=True)
    _check(_rows(N, nv * (4 if dt == "f32" else 8), dt, nv), 1, dt)


@pytest.mark.parametrize("nv,chunks", [(513, 1), (1023, 2), (1025, 2), (2051, 1), (3071, 3), (4097, 2), (9000, 70)])
def test_chunks_with_a_nearly_empty_last_batch(nv, chunks):
    print(f"norm chunks {nv} {chunks}", flush=True)
    for dt in ("bf16", "f32"):
        _check(_rows(4, nv * (4 if dt == "f32" else 8), dt, nv), chunks, dt)


@pytest.mark.parametrize("M,chunks", [(1000, 1), (2056, 1), (9000, 1), (40000, 1), (9000, 3)])
def test_special_rows(M, chunks):
    """Zero rows, rows whose mean square overflows fp32, infinities and NaN, a
    zero eps and one so small that x / sqrt(eps) overflows."""
    x = _rows(8, M, "f32", M)
    x[1] = 0.0
    x[2] *= 1e25
    x[3, M // 3] = float("inf")
    x[4, M - 1] = float("nan")
    x[5] = -1e30
    x[6, :-1] = 0.0
    x[6, -1] = -2.0
    norm = pa.norm_l2(x.cuda(), chunks=chunks).cpu()
    ref = x.double().square().sum(1).sqrt()
    ok = [0, 1, 2, 5, 6, 7]
    np.testing.assert_allclose(norm[ok].double().numpy(), ref[ok].numpy(), rtol=RTOL)
    assert not np.isfinite(norm[3].item()) and np.isnan(norm[4].item())
    for eps in (0.0, 1e-36, 1e-6):
        y, m = (t.cpu().double() for t in pa.rmsnorm_rowmax(x.cuda(), eps=eps, chunks=chunks))
        yr, mr = norms.rmsnorm_rowmax(x[[0, 6, 7]].double().numpy(), eps)
        np.testing.assert_allclose(m[[0, 6, 7]].numpy(), mr, rtol=RTOL, atol=1e-30)
        np.testing.assert_allclose(y[[0, 6, 7]].numpy(), yr, rtol=RTOL, atol=1e-30)
        assert torch.all(y[2] == 0)                        # the mean square overflows: a scale of 0
        if chunks == 1:
            assert m[2] == 0 and m[5] == 0 and m[3] == 0   # finite values over an infinite norm
        assert torch.all(torch.isnan(y[4]))
        if eps:
            assert m[1] == 0 and torch.all(y[1] == 0)


def test_chunk_rule_for_short_and_medium_rows():
    """The library's choice: one chunk for rows of at most 64 KiB, and of at
    most 208 KiB with a row for half the compute units."""
    bf16, f32 = torch.bfloat16, torch.float32
    for op in ("l2", "rms"):
        assert pa.norm_chunks(op, 40, 32768, bf16) == 1 and pa.norm_chunks(op, 40, 32776, bf16) > 1
        cu = torch.cuda.get_device_properties(0).multi_processor_count
        assert pa.norm_chunks(op, cu // 2, 53248, f32) == 1
        assert pa.norm_chunks(op, cu // 2 - 1, 53248, f32) > 1 and pa.norm_chunks(op, cu // 2, 53252, f32) > 1
