"""One small case per compiled kernel instantiation.

``tests/test_kernel_coverage.py`` (CPU) checks that the kernels these cases
dispatch to, as named by the library's own dispatch (attn_fwd_call_kernels /
attn_decode_kernels), are exactly the kernels in the build;
``tests/test_gpu_variants.py`` runs every case on the GPU against the oracle,
``tests/test_gpu_norms.py`` every row-reduction case (both operations),
``tests/test_gpu_prefill_split.py`` the prefill cases with the batch repeated
WIDE_BATCH times (so that prefill_kernel runs) and those of the split kernel.
"""

# Prefill: (B, Hq, Hkv, Lq, Lk, D, dtype, causal, alibi, softcap, window).
# The flag combinations are the eight kernels per (head dim, type): plain and
# ALiBi without the mask, causal, causal ALiBi, causal SoftCap, and the
# sliding window alone, with ALiBi and with SoftCap.
_FLAGS = [
    (False, False, None, None),
    (False, True, None, None),
    (True, False, None, None),
    (True, True, None, None),
    (True, False, 2.0, None),
    (True, False, None, 77),
    (True, True, None, 77),
    (True, False, 2.0, 77),
]
PREFILL_VARIANT_CASES = []
for _D in (64, 128):
    for _dt in ("f16", "bf16"):
        for _n, (_c, _a, _cap, _w) in enumerate(_FLAGS):
            # vary the shape a little between cases: GQA groups, Lq != Lk
            _Hq, _Hkv = [(4, 4), (4, 2), (6, 3), (8, 1)][_n % 4]
            _Lq, _Lk = [(300, 300), (257, 410), (333, 333), (150, 150)][(_n + _D // 64) % 4]
            PREFILL_VARIANT_CASES.append((1, _Hq, _Hkv, _Lq, _Lk, _D, _dt, _c, _a, _cap, _w))

# With the batch repeated this often, every one of them gives more workgroups
# than there are compute units, whatever its shape.
WIDE_BATCH = 66

# Few query rows (the same fields): for each head dim, number of key groups
# (two or four) and score (plain, ALiBi, SoftCap) a shape with one key range and
# one with several, each with more tiles per key group than its LDS ring holds.
_SPLIT = [
    (6, 32, 8, 65, 345, 64, True, False, None, 306), (6, 32, 8, 17, 3367, 64, True, False, None, None),
    (4, 24, 8, 225, 293, 64, True, True, None, None), (6, 32, 8, 17, 3857, 64, False, True, None, None),
    (6, 12, 3, 298, 298, 64, True, False, 3.0, 224), (6, 16, 4, 34, 2841, 64, True, False, 3.0, None),
    (6, 4, 1, 31, 577, 64, True, False, None, None), (2, 24, 8, 17, 2934, 64, True, False, None, None),
    (4, 6, 2, 33, 581, 64, False, True, None, None), (6, 4, 4, 17, 4907, 64, True, True, None, None),
    (6, 2, 2, 61, 577, 64, True, False, 3.0, None), (1, 24, 8, 18, 4648, 64, True, False, 3.0, None),
    (4, 16, 8, 263, 326, 128, True, False, None, 322), (2, 24, 8, 65, 2846, 128, False, False, None, None),
    (4, 24, 8, 157, 289, 128, True, True, None, None), (6, 16, 8, 36, 2820, 128, True, True, None, None),
    (3, 32, 8, 174, 298, 128, True, False, 3.0, 265), (6, 32, 8, 17, 4070, 128, True, False, 3.0, None),
    (1, 32, 8, 37, 578, 128, True, False, None, None), (6, 4, 4, 19, 4892, 128, True, False, None, None),
    (4, 6, 2, 49, 585, 128, True, True, None, None), (3, 24, 8, 17, 1919, 128, False, True, None, None),
    (4, 2, 1, 147, 595, 128, True, False, 3.0, None), (1, 24, 8, 19, 5582, 128, True, False, 3.0, None),
]
PREFILL_SPLIT_CASES = [c[:6] + (dt,) + c[6:] for c in _SPLIT for dt in ("f16", "bf16")]

# Decode: (B, Hq, Hkv, Lk, D, dtype, alibi, softcap, num_splits).  Query heads
# per KV head: 1 (vector kernel, one head a workgroup), 4 (matrix kernel),
# 34, 36 and 64 (vector kernel with 2, 4 and 8 heads a workgroup).
DECODE_VARIANT_CASES = []
for _D in (64, 128):
    for _dt in ("f16", "bf16"):
        for _Hq, _Hkv in [(4, 4), (8, 2), (34, 1), (36, 1), (64, 1)]:
            for _a in (False, True):
                for _cap in (None, 2.0):
                    _Lk = 333 + 50 * len(DECODE_VARIANT_CASES) % 400
                    DECODE_VARIANT_CASES.append((1, _Hq, _Hkv, _Lk, _D, _dt, _a, _cap, 3))


# Row reductions: (N, M, dtype, chunks), chunks 0 for the library's choice.
# Every dtype has cases with several chunks per row (chunk partials and a
# second kernel) and with one (a workgroup per row); RMSNorm's one-pass
# kernel at its longest row and one vector past it (then the two kernels run
# with one chunk).
NORM_CASES = [
    (3, 8, "f16", 0),            # one vector per row
    (32, 1024, "bf16", 0),       # the smallest paper shape
    (7, 1000, "f16", 3),         # chunks of 336 elements: the last one short
    (5, 4104, "bf16", 5),        # ragged chunk ends
    (2, 64, "f16", 40),          # more chunks than vectors: empty chunks
    (9, 3000, "f32", 4),
    (4, 4, "f32", 0),
    (64, 1 << 15, "bf16", 0),
    (5, 1000, "f16", 1),         # one chunk: 125 vectors, most lanes idle
    (3, 1 << 17, "bf16", 1),     # the longest row held in registers: 16 vectors every lane
    (2, 1 << 16, "f32", 1),      # the same in fp32
    (2, (1 << 17) + 8, "bf16", 1),   # one vector longer: RMSNorm's two kernels, one chunk
    (300, 2048, "f16", 1),       # more rows than compute units
]


def case_id(c):
    return "x".join(str(x) for x in c)
