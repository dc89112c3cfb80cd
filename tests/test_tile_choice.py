"""How a forward's grouped GEMMs are cut, asked through the host-side query: which small batches are
streamed, what the cuts know, what choosing costs.  No device work."""
import ctypes
import time

import numpy as np
import pytest

from paper_2603_28768_amd import binding, synth


def test_tile_choice_knows_the_weight_format():
    # a busy rank, its cold slots carried by the gate/up tiles of the busy ones in E4M3 only: 4099 rows
    # 207 us with riders, 216 without (bf16 as fast without)
    lib = binding.lib()
    rows = np.array([1542, 1010, 514, 476, 228, 126, 57, 36, 34, 21, 14, 12, 9, 6, 6, 4, 4], dtype=np.int64)
    plan = binding.Plan(rows[None, None], 1, 0)
    a = binding.FwdArgs()
    a.dtype, a.T, a.H, a.I, a.k = 1, int(rows.sum()), 4096, 1536, 1
    a.w_gateup_packed = a.w_down_packed = 0x1000
    out = [ctypes.c_int32() for _ in range(4)]
    got = {}
    for fmt in (binding.CRAFT_W_E4M3, binding.CRAFT_W_BF16, binding.CRAFT_W_E4M3):      # (kept apart in the plan)
        a.weight_format = fmt
        assert lib.craft_moe_rank_forward_tiles(plan._h, 0, 0, ctypes.byref(a), *out) == 0
        got.setdefault(fmt, set()).add(tuple(v.value for v in out))
    assert got == {binding.CRAFT_W_E4M3: {(224, 256, 1, 0)}, binding.CRAFT_W_BF16: {(224, 256, 0, 0)}}


def test_tile_choice_for_a_new_batch_size_is_quick():
    # host time of the first forward of a shape, the least of many: packed tiles play their cuts through
    # (0.15 ms; with every one of them to its end 0.6 to 1.4 ms), row-major and streamed batches have no
    # choice to make (0.002 ms; they took as long)
    lib = binding.lib()
    g = np.random.default_rng(3)
    W = g.multinomial(8 * 4096, synth.popularity(128, 1.0, 2, 0), size=(4, 1)).astype(np.int64)
    plan = binding.Plan(W, 8, 8)
    a = binding.FwdArgs()
    a.dtype, a.H, a.I, a.k = 1, 4096, 1536, 8

    def least(first, calls=60):
        best = 1.0
        for T in range(first, first + calls):
            a.T = T
            t = time.perf_counter()
            assert lib.craft_moe_rank_forward_tiles(plan._h, 0, 0, ctypes.byref(a), None, None, None, None) == 0
            best = min(best, time.perf_counter() - t)
        return best

    rowmajor = max(least(64), least(1700), least(4096))
    a.w_gateup_packed = a.w_down_packed = 0x1000
    packed = least(4096)
    print(f"  a new batch size: row-major {rowmajor * 1e6:.1f} us, packed {packed * 1e6:.0f} us")
    assert packed < 450e-6 and rowmajor < 50e-6


# One rank that holds `slots` experts with `rows` tokens each; us streamed / tiled where it was measured.
STREAM_CASES = [
    ("bf16", 7168, 2048, 2, 14, True),          # 53 / 74
    ("bf16", 7168, 2048, 1, 126, True),         # 62 / 144
    ("bf16", 7168, 2048, 3, 44, False),         # 98 / 85
    ("bf16", 7168, 2048, 8, 62, False),         # 193 / 137
    ("bf16", 4096, 1536, 2, 62, True),          # 45 / 60
    ("bf16", 4096, 1536, 8, 44, False),         # 96 / 72
    ("bf16", 2048, 768, 4, 28, True),           # 29 / 39
    ("bf16", 2048, 768, 16, 62, False),         # 68 / 56
    ("e4m3", 7168, 2048, 3, 14, True),          # 56 / 72
    ("e4m3", 7168, 2048, 6, 14, True),          # 81 / 87
    ("e4m3", 7168, 2048, 4, 62, False),         # 92 / 76
    ("e4m3", 7168, 2048, 8, 62, False),         # 152 / 97
    ("rowmajor", 7168, 2048, 4, 62, True),      # 137 / 163
    ("rowmajor", 7168, 2048, 8, 62, False),     # 235 / 188
    ("rowmajor", 7168, 2048, 16, 44, False),    # 454 / 273
    ("rowmajor", 4096, 1536, 8, 14, True),      # 84 / 95
    ("rowmajor", 4096, 1536, 16, 44, False),    # 207 / 143
    ("rowmajor", 2048, 768, 10, 28, True),      # 50 / 61
    ("rowmajor", 2880, 1536, 22, 5, False),     # 152 / 130 (narrow tiles)
]


@pytest.mark.parametrize("weights,H,I,slots,rows,streamed", STREAM_CASES)
def test_small_batches_are_streamed_where_that_is_faster(weights, H, I, slots, rows, streamed):
    lib = binding.lib()
    plan = binding.Plan(np.full((1, 1, slots), rows, dtype=np.int64), 1, 0)
    a = binding.FwdArgs()
    a.dtype, a.T, a.H, a.I, a.k = 1, slots * rows, H, I, 1
    if weights != "rowmajor":
        a.w_gateup_packed = a.w_down_packed = 0x1000
        a.weight_format = binding.CRAFT_W_E4M3 if weights == "e4m3" else binding.CRAFT_W_BF16
    gu, dn = ctypes.c_int32(), ctypes.c_int32()
    assert lib.craft_moe_rank_forward_tiles(plan._h, 0, 0, ctypes.byref(a), gu, dn, None, None) == 0
    assert ((gu.value, dn.value) == (64, 64)) == streamed
