"""Host logic of the decode chunk counts (no device here: 256 compute units)
and of the workspaces that are refused.  Pointers passed here are never
dereferenced."""

import ctypes

import pytest

import paper_2510_08726_amd as pa

FAKE = ctypes.c_void_p(0x10000)


@pytest.fixture(scope="module")
def lib():
    try:
        return pa.load_library()
    except RuntimeError:
        import __graft_entry__
        __graft_entry__.build()
        return pa.load_library()


def _decode(lib, B, Hq, Hkv, Lk, D, nbytes, num_splits=0):
    return lib.attn_decode_mod(FAKE, FAKE, FAKE, FAKE, B, Hq, Hkv, Lk, D, ctypes.c_float(0.1), None, ctypes.c_float(0.0),
                               num_splits, FAKE, ctypes.c_size_t(nbytes), 0, None)


@pytest.mark.parametrize("case", [(1, 32, 8, 3001, 128), (2, 8, 4, 900, 64), (11, 32, 16, 3000, 128)])
def test_grouped_decode_refuses_a_short_workspace(lib, case):
    """A grouped call's own chunk count is the only one it takes where its
    workgroups are at most one per compute unit."""
    B, Hq, Hkv, Lk, D = case
    S = lib.attn_decode_num_splits(B, Hq, Hkv, Lk, D)
    need = lib.attn_decode_workspace_bytes(B, Hq, D, S)
    assert _decode(lib, B, Hq, Hkv, Lk, D, need - 256) == pa.ATTN_ERR_WORKSPACE
    if S > 2:
        half = lib.attn_decode_workspace_bytes(B, Hq, D, S // 2)
        assert _decode(lib, B, Hq, Hkv, Lk, D, half) == pa.ATTN_ERR_WORKSPACE


def test_per_head_decode_refuses_less_than_one_workgroup_per_compute_unit(lib):
    assert lib.attn_decode_num_splits(3, 32, 32, 4000, 64) == 5           # 96 heads: up to two per compute unit
    least = lib.attn_decode_workspace_bytes(3, 32, 64, 3)                 # ceil(256 / 96)
    assert _decode(lib, 3, 32, 32, 4000, 64, least - 256) == pa.ATTN_ERR_WORKSPACE


@pytest.mark.parametrize("case,S", [
    ((11, 24, 12, 12222, 64), 3),      # 132 KV heads: one chunk each would read at half the rate
    ((9, 64, 16, 4959, 64), 3),
    ((1, 16, 4, 100000, 64), 128),     # the compute units' divisors too
    ((16, 32, 16, 9000, 64), 2),
    ((11, 24, 12, 1199, 64), 1),       # short chunks: one per compute unit
    ((11, 24, 12, 12222, 128), 1),     # D = 128: a workgroup takes the compute unit's LDS
    ((40, 32, 8, 9000, 64), 1),        # more KV heads than compute units
    ((1, 8, 2, 2000, 64), 16),         # chunks of at least 128 keys
])
def test_grouped_decode_at_head_dim_64(lib, case, S):
    """Up to two workgroups per compute unit where the chunks are long; less
    than a workspace for one per compute unit is refused."""
    B, Hq, Hkv, Lk, D = case
    assert lib.attn_decode_num_splits(B, Hq, Hkv, Lk, D) == S
    one = min(max(256 // (B * Hkv), 1), -(-Lk // 128))
    least = lib.attn_decode_workspace_bytes(B, Hq, D, one)
    assert _decode(lib, B, Hq, Hkv, Lk, D, least - 256) == pa.ATTN_ERR_WORKSPACE
