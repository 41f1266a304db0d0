"""The algorithmic byte counts bench.py divides by the measured times (CPU only): the whole
path's bytes follow the compulsory-traffic formula per (layer, KV head, context token) at
d = 128 — read K and V once, write the 8-bit codes and the fp32 scale (644 B), plus per
kept token the re-read of its K row, codes and scale and the write of the compact cache and
index (780 B) — and the per-launch counts of step 2 add up over its launches."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import bench  # noqa: E402
from synth import workloads as W  # noqa: E402


def _kept(w):
    from oracle import taskpress_oracle as o

    return sum(o.keep_count(n, w.keep_ratio, w.keep_budget) for n in w.ctx_lens)


def test_path_bytes_128k():
    w = W.llama8b_128k()
    k = _kept(w)
    assert k == 13107
    per, path = bench.algorithmic_bytes(w, k)
    LH, n = w.L * w.Hkv, w.n_tot
    q_bytes = w.L * w.Hq * w.g_tot * w.d * 2
    assert path == LH * (644 * n + 780 * k) + q_bytes
    assert abs(path / 1e9 - 24.24) < 0.01
    # step 2's launches (7/20 of the rows beside each score pass on the second stream at 256 guide
    # rows, the rest between the passes) cover every V row once
    row = 2 * w.d + w.d + 4
    assert per["k_quantize"] + 2 * per["k_quantize_lean"] == LH * n * row
    assert per["k_quantize_lean"] == (LH * n * 7 // 20 // 64 * 64) * row
    # with the normalisers given: the last 3/10 on the second stream, the rest before pass 2
    per_g, _ = bench.algorithmic_bytes(w, k, normalisers_given=True)
    assert per_g["k_quantize"] + per_g["k_quantize_lean"] == LH * n * row
    assert per_g["k_quantize_lean"] == (LH * n * 3 // 10 // 64 * 64) * row
    assert bench.LEAN_LAUNCHES == {False: 2, True: 1}
    # scales only: half beside each pass; with the normalisers given, 3/5 on the second stream
    per_s, _ = bench.algorithmic_bytes(w, k, full_codes=False)
    row_s = 2 * w.d + 4
    assert per_s["k_quantize"] + 2 * per_s["k_quantize_lean"] == LH * n * row_s
    assert per_s["k_quantize_lean"] == (LH * n // 2 // 64 * 64) * row_s
    per_gs, _ = bench.algorithmic_bytes(w, k, full_codes=False, normalisers_given=True)
    assert per_gs["k_quantize_lean"] == (LH * n * 3 // 5 // 64 * 64) * row_s
    # the parts by guide rows a context token meets (4 per guide token here, in 64s): codes two passes,
    # normalisers given, scales only two passes, normalisers given
    for g, want in ((16, [(1, 5), (1, 5), (3, 10), (1, 5)]), (17, [(1, 5), (1, 5), (3, 10), (3, 5)]),
                    (48, [(1, 5), (1, 5), (3, 10), (3, 5)]), (49, [(7, 20), (3, 10), (1, 2), (3, 5)]),
                    (64, [(7, 20), (3, 10), (1, 2), (3, 5)]), (65, [(2, 5), (1, 2), (1, 2), (3, 5)])):
        wg = w.with_(guide_lens=(g,))
        assert [bench.lean_part(wg, c, l) for c in (True, False) for l in (False, True)] == want
    # a batch counts the rows beyond 128 of each sequence: half of the tokens with 64 rows, half with 320
    mixed = w.with_(ctx_lens=(65536, 65536), guide_lens=(16, 80))
    assert bench.lean_part(mixed) == (7, 20) and bench.lean_part(mixed, True, True) == (3, 10)
    assert bench.lean_part(mixed.with_(ctx_lens=(65536, 32768))) == (1, 5)
    assert bench.lean_part(mixed, False) == (1, 2) and bench.lean_part(W.ragged8()) == (2, 5)
    w64 = w.with_(d=64, guide_lens=(16,))
    assert [bench.lean_part(w64, c, l) for c in (True, False) for l in (False, True)] == [(2, 5), (1, 2), (1, 2), (3, 5)]


def test_stages_follow_the_kernels_that_run():
    """The stages between tp_evict's events on both sides of the library's lines: the selection of one
    workgroup per segment, step 2 beside the score passes, the merge of the normalisers."""
    w = W.llama8b_128k()
    assert bench.stage_names(w) == bench.STAGES
    assert bench.stage_names(w, False, True) == [None, None, "k_quantize", "k_guide_attn", "k_sel_score", "k_select",
                                                 "k_compact_quant"]
    assert bench.stage_names(W.llama8b_32k()) == bench.STAGES[:4] + ["k_sel_one", None, "k_compact"]
    assert bench.stage_names(W.llama8b_32k(), True, True, True) == [None, None, None, "k_guide_attn", "k_sel_one", None,
                                                                   "k_compact"]
    assert bench.stage_names(W.tiny())[1] is None
    assert bench.stage_names(W.llama8b_32k().with_(rule=1))[4:6] == ["k_guide_pool", "k_sel_one"]
    assert bench.stage_names(w.with_(rule=1))[4:6] == ["k_guide_pool", "k_select"]
    one = lambda lens, **kw: bench.selects_in_one(w.with_(ctx_lens=lens, guide_lens=(8,) * len(lens), **kw))
    assert one((65536,)) and not one((65537,))                    # 256 segments
    assert one((65532, 65533)) and one((65533, 65532)) and not one((65534, 65532))  # misaligned segments
    assert one((57344,), L=1) and not one((57345,), L=1) and one((57345,), L=4)     # 8 and 32 segments
    assert one((4096,), pool_k=9) and not one((4096,), pool_k=11) and one((4096,), pool_k=11, rule=1)
    seg = w.L * w.Hkv * w.d * 2
    for given, line in ((False, 640 << 20), (True, 1024 << 20)):
        n = line // seg
        assert bench.step2_overlaps(w.with_(ctx_lens=(n,)), given)
        below = w.with_(ctx_lens=(n - 1,))
        assert not bench.step2_overlaps(below, given)
        per, _ = bench.algorithmic_bytes(below, _kept(below), normalisers_given=given)
        assert per["k_quantize"] == w.L * w.Hkv * (n - 1) * (2 * w.d + w.d + 4) and "k_quantize_lean" not in per
    per, _ = bench.algorithmic_bytes(W.llama8b_32k(), 6553)
    assert per["k_sel_one"] == w.L * w.Hkv * (32768 * 16 + 6553 * 4)


def test_path_bytes_scales_only_and_int4():
    w = W.llama8b_128k()
    k = _kept(w)
    LH, n = w.L * w.Hkv, w.n_tot
    q_bytes = w.L * w.Hq * w.g_tot * w.d * 2
    _, path = bench.algorithmic_bytes(w, k, full_codes=False)
    # scales only (516 B per token-head), the kept rows re-read in bf16 and quantised
    assert path == LH * (516 * n + k * (256 + 256 + 4 + 256 + 128 + 4)) + q_bytes
    w4 = w.with_(bits=4)
    _, path4 = bench.algorithmic_bytes(w4, k)
    assert path4 == LH * ((256 + 256 + 64 + 4) * n + k * (2 * (256 + 64 + 4) + 4)) + q_bytes


def test_kernel_source_lists_name_existing_files():
    """Every source a traffic summary is keyed on exists (a renamed file would otherwise leave
    every summary stale without notice)."""
    for kernel, names in bench.KERNEL_SOURCES.items():
        for name in names:
            assert os.path.exists(os.path.join(ROOT, "paper_2608_03276_amd", "csrc", name)), (kernel, name)


def test_attention_bytes_128k():
    """The guide rows' attention at 128K, counted by hand: K and V of the context
    (2 x 32 x 8 x 131072 x 128 x 2 B), Q (32 x 32 x 64 x 128 x 2 B) and O (x 4 B), the
    guide tokens' K and V (2 x 32 x 8 x 64 x 128 x 2 B); with step 2, int8 codes and a
    4-byte scale per context token-head."""
    w = W.llama8b_128k()
    plain = 17_179_869_184 + 16_777_216 + 33_554_432 + 8_388_608
    assert bench.attention_bytes(w, False) == plain
    assert bench.attention_bytes(w, True) == plain + 32 * 8 * 131072 * (128 + 4) == 21_667_774_464
    w4 = w.with_(bits=4)  # nibbles: 64 code bytes per row
    assert bench.attention_bytes(w4, True) == plain + 32 * 8 * 131072 * (64 + 4)
