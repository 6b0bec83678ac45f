"""Host logic of the split of prompts with few rows (no device here: 256
compute units), and the checks of its workspace."""

import ctypes

import pytest

import paper_2510_08726_amd as pa

FAKE = ctypes.c_void_p(0x10000)


@pytest.fixture(scope="module")
def lib():
    try:
        lib = pa.load_library()
    except RuntimeError:
        import __graft_entry__
        __graft_entry__.build()
        lib = pa.load_library()
    lib.attn_fwd_workspace_bytes.restype = ctypes.c_size_t
    return lib


def test_key_ranges(lib):
    S = lib.attn_fwd_num_splits
    assert S(4, 32, 32, 2048, 2048, 128, 1, 0) == 1        # enough rows
    assert S(1, 32, 8, 64, 16000, 128, 1, 0) == 8          # 32 workgroups of 256
    assert S(1, 32, 8, 500, 6100, 128, 1, 0) == 1          # 256 workgroups in one range
    assert S(2, 32, 16, 130, 13392, 128, 1, 0) == 2
    assert S(1, 32, 8, 64, 500, 128, 1, 0) == 1            # too few keys to pay for a second kernel
    assert S(1, 32, 8, 64, 16000, 128, 1, 300) == 1        # nor in the window
    assert S(0, 32, 8, 64, 16000, 128, 1, 0) == 0 and S(1, 32, 8, 64, 16000, 96, 1, 0) == 0
    assert 1 <= S(1, 1, 1, 1, 8000000, 128, 0, 0) <= 32


def test_workspace(lib):
    W = lib.attn_fwd_workspace_bytes
    assert W(1, 32, 64, 128, 1) == 0 and W(0, 32, 64, 128, 4) == 0 and W(1, 32, 64, 96, 4) == 0
    assert W(1, 32, 64, 128, 8) == 32 * 64 * 8 * 130 * 4

    def call(ws, nbytes):
        return lib.attn_fwd_split(FAKE, FAKE, FAKE, FAKE, 1, 32, 8, 64, 16000, 128, 1, ctypes.c_float(0.1), None,
                                  ctypes.c_float(0.0), 0, ws, ctypes.c_size_t(nbytes), 0, None)

    need = W(1, 32, 64, 128, 8)
    assert call(FAKE, need - 1) == pa.ATTN_ERR_WORKSPACE
    assert call(ctypes.c_void_p(0x10008), need) == pa.ATTN_ERR_WORKSPACE


def test_the_names_are_of_the_kernels_that_run(lib):
    """Many rows, few rows, and few rows on many keys with and without a
    workspace."""
    import torch
    f16, bf16 = torch.float16, torch.bfloat16
    K = pa.attn_fwd_call_kernels
    assert K(4, 32, 32, 2048, 2048, 128, f16, 1, 0) == ["prefill_kernel<128,f16,1,0,0,0>"]
    assert K(1, 32, 8, 500, 6100, 128, bf16, 1, 0) == ["prefill_split_kernel<128,bf16,4,0,0>"]
    assert K(1, 32, 8, 64, 16000, 128, f16, 1, 1) == ["prefill_split_kernel<128,f16,4,1,0>",
                                                      "prefill_combine_kernel<128,f16>"]
    assert len(K(1, 32, 8, 64, 16000, 128, f16, 1, 1, workspace=False)) == 1
    assert K(1, 32, 8, 64, 16000, 64, bf16, 1, 0, 30.0, 9000) == ["prefill_split_kernel<64,bf16,4,0,1>",
                                                                 "prefill_combine_kernel<64,bf16>"]
    for bad in ((0, 32, 8, 64, 64, 128, f16, 1, 0), (1, 32, 5, 64, 64, 128, f16, 1, 0), (1, 32, 8, 64, 64, 96, f16, 1, 0),
                (1, 32, 8, 64, 64, 128, f16, 0, 0, 0.0, 7), (1, 32, 8, 64, 64, 128, f16, 1, 1, 3.0)):
        with pytest.raises(pa.AttnError):
            K(*bad)


@pytest.mark.parametrize("call,name", [
    # prefill.hip is the faster one: one or two tiles at D = 64, and more
    # workgroups of the split kernel than compute units at D = 128
    ((4, 2, 1, 8, 8, 64, 0, 0), "prefill_kernel<64"), ((1, 32, 8, 30, 30, 64, 1, 0), "prefill_kernel<64"),
    ((3, 64, 8, 78, 78, 64, 0, 0), "prefill_kernel<64"), ((6, 8, 8, 361, 361, 128, 1, 0), "prefill_kernel<128"),
    ((1, 32, 32, 782, 782, 128, 1, 0), "prefill_kernel<128"), ((4, 64, 32, 65, 65, 64, 1, 0, 30.0), "prefill_kernel<64"),
    ((1, 2, 1, 54, 88, 128, 1, 0, 30.0), "prefill_kernel<128"),
    # and here the split kernel: long masks' and slopes' set-up, more tiles
    ((1, 32, 32, 1, 1, 64, 1, 1), "prefill_split_kernel<64"), ((1, 16, 16, 35, 175, 128, 1, 1, 0.0, 129), "prefill_split_kernel<128"),
    ((1, 12, 4, 15, 15, 128, 1, 0, 0.0, 11), "prefill_split_kernel<128"), ((1, 32, 32, 482, 482, 128, 1, 0), "prefill_split_kernel<128"),
    ((4, 8, 2, 568, 568, 64, 1, 0, 30.0, 516), "prefill_split_kernel<64"),
])
def test_the_faster_kernel_runs(lib, call, name):
    """Calls measured under both kernels, the two at least 5 % apart."""
    import torch
    B, Hq, Hkv, Lq, Lk, D, causal, alibi, *mod = call
    assert pa.attn_fwd_call_kernels(B, Hq, Hkv, Lq, Lk, D, torch.float16, causal, alibi, *mod)[0].startswith(name)


def test_the_modifiers_do_not_change_the_ranges(lib):
    """attn_fwd_num_splits, which sizes the workspace, takes no modifiers: the
    call with one has as many ranges."""
    import random
    import torch
    rng = random.Random(1)
    for _ in range(2000):
        Hkv = rng.choice([1, 2, 4, 8])
        Lq, more = int(2 ** rng.uniform(0, 10)), int(2 ** rng.uniform(0, 14))
        sizes = (rng.choice([1, 2, 4]), Hkv * rng.choice([1, 2, 3, 4]), Hkv, Lq, Lq + more, rng.choice([64, 128]))
        window = rng.choice([0, rng.randrange(1, Lq + more)])
        S = lib.attn_fwd_num_splits(*sizes, 1, window)
        for alibi, cap in ((0, 0.0), (1, 0.0), (0, 30.0)):
            names = pa.attn_fwd_call_kernels(*sizes, torch.float16, 1, alibi, cap, window)
            assert (len(names) == 2) == (S > 1) and (S == 1 or "split" in names[0])
