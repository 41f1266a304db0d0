"""The launch rules that depend on sizes: each side of every line, on ragged and smallest shapes,
against the CPU oracle (the comparison rules are parity_util's)."""
import numpy as np
import pytest
import torch

import synth
from oracle import taskpress_oracle as o
from paper_2608_03276_amd import binding as B
from synth import workloads as W

import parity_util as pu
import test_gpu_guide_attention as tga
import test_gpu_parity as tgp

pytestmark = pytest.mark.gpu

# Score-pass chunks: multiples of 256 tokens, cut evenly per sequence; up to 768 workgroups pass 2
# merges the chunks' statistics itself, beyond that a kernel does.
CHUNK_CASES = [
    ("unit-edges", 1, 8, 2, 128, [255, 256, 257, 511, 513, 1], [16, 3, 64, 9, 33, 1], synth.DIST_NORMAL, 5),
    ("even-cuts", 1, 8, 2, 64, [4097, 2333, 7681], [16, 80, 40], synth.DIST_STUDENT_T3, 3),
    # one chunk per sequence: 0 to 9 sub-tiles per wave, so each way in and out of the two-tile loop,
    # for every number of row blocks, with and without a ragged last sub-tile
    ("tile-counts", 1, 8, 2, 128, [33, 800, 1030, 1290, 1600, 2085], [16, 33, 48, 64, 20, 5], synth.DIST_STUDENT_T3, 5),
    ("tile-counts-64", 1, 8, 2, 64, [2070, 31, 1536, 1056, 511, 768], [64, 48, 16, 33, 20, 5], synth.DIST_NORMAL, 1),
    # three row-block pairs: without a class of four (launched apart), and beside one with too many
    # workgroups to be padded to it
    ("three-pairs", 1, 8, 2, 128, [800, 2085, 33, 1290], [33, 48, 40, 5], synth.DIST_STUDENT_T3, 5),
    ("three-pairs-64", 1, 8, 2, 64, [1536, 31, 511], [48, 33, 35], synth.DIST_NORMAL, 3),
    ("three-beside-four", 14, 32, 8, 64, [2600, 70, 300], [40, 64, 5], synth.DIST_NORMAL, 5),
    ("merge-kernel", 14, 32, 8, 64, [513, 70, 300], [64, 130, 5], synth.DIST_NORMAL, 5),  # > 768 workgroups
]


@pytest.mark.parametrize("guide_keys", [False, True])
@pytest.mark.parametrize("case", CHUNK_CASES, ids=[c[0] for c in CHUNK_CASES])
def test_score_pass_chunks(gpu_lib, case, guide_keys):
    tgp._guide_case(case, guide_keys)


def _select(rng, L, Hkv, lens, rule, ratio, budget, ties):
    sk, g = tgp._select_inputs(rng, L, Hkv, lens, ties)
    dd = B.dims(L, Hkv, Hkv, 64)
    bt = B.Batch(np.concatenate([[0], np.cumsum(lens)]).tolist())
    ko = B.kept_offsets_for(bt, ratio, budget)
    kept = torch.full((L * Hkv * ko[-1],), -1, dtype=torch.int32, device="cuda")
    s_out = torch.empty(L * Hkv * sum(lens), dtype=torch.float32, device="cuda")
    B.tp_combine_select_topk(dd, bt, torch.from_numpy(sk).cuda(), torch.from_numpy(g).cuda(), rule, ratio, budget, ko,
                             kept, s_out)
    torch.cuda.synchronize()
    S, kept = s_out.cpu().numpy().reshape(L * Hkv, -1), kept.cpu().numpy().reshape(L * Hkv, -1)
    sk, g = sk.reshape(L * Hkv, -1), g.reshape(L * Hkv, -1)
    for s in range(L * Hkv):
        for b, n in enumerate(lens):
            a, e = bt.ctx_offsets[b], bt.ctx_offsets[b + 1]
            ref = o.combine(sk[s, a:e], g[s, a:e], rule)
            tag = f"rule={rule} lens={lens} seg={s} b={b}"
            if rule == o.COMBINE_NORM_ADD:  # fp64 norms summed in another order: at most an fp32 rounding apart
                assert np.all(np.abs(S[s, a:e] - ref) <= 2.0 ** -23 * np.abs(ref)), tag
            else:
                assert np.array_equal(S[s, a:e].view(np.uint32), ref.view(np.uint32)), tag
            # the kept set of the scores the call itself wrote, exactly
            k = o.keep_count(n, ratio or None, budget or None)
            assert np.array_equal(kept[s, ko[b]:ko[b + 1]], o.select(S[s, a:e], k)), tag


# Each size class of the one-workgroup selection at its last aligned and first unaligned length
# and one past it, and the split selection beyond (from 57345 tokens in these calls of few segments).
SELECT_LENS = [[4096], [4093, 3], [4094, 3], [8192], [8190, 2, 7], [16384], [16381, 1], [32768], [32767, 5], [57344], [57345],
               [57341, 1], [65536], [65533, 1], [65534, 6], [65537], [100003, 70000, 1]]


@pytest.mark.parametrize("rule", [0, 1, 2, 3])
@pytest.mark.parametrize("lens", SELECT_LENS, ids=lambda v: "-".join(map(str, v)))
def test_select_size_classes(gpu_lib, lens, rule):
    rng = np.random.default_rng(71 + rule)
    _select(rng, 1, 3, lens, rule, 0.13, 0, 0)
    _select(rng, 1, 2, lens, rule, 0.0, 777, 5)  # five levels: ties at the threshold


@pytest.mark.parametrize("layers", [16, 17])  # 256 short segments, and just beyond: workgroups of 1024 threads, of 256
def test_select_many_short_segments(gpu_lib, layers):
    _select(np.random.default_rng(77), layers, 8, [290, 1031], 0, 0.13, 0, 5)


@pytest.mark.parametrize("lens", [[65536], [65533, 9], [300, 40001]], ids=lambda v: "-".join(map(str, v)))
def test_select_many_long_segments(gpu_lib, lens):
    """32 segments and more keep the one-workgroup selection up to its last length, and skip the
    register groups that the batch's short sequences do not reach."""
    _select(np.random.default_rng(78), 4, 8, lens, 0, 0.2, 0, 0)


@pytest.mark.parametrize("lens", [[900], [4099, 3000], [20000, 33], [65530, 9], [66000, 12000]],
                         ids=lambda v: "-".join(map(str, v)))
@pytest.mark.parametrize("pool", [1, 3, 5, 7, 9, 11])
def test_pooling_inside_selection(gpu_lib, lens, pool):
    """tp_evict's selection pools the raw sums itself: bit for bit the pooling kernel's scores of
    the separate calls (half-widths up to 4 across lanes, wider ones through LDS), one and two row groups."""
    glens = [70] * len(lens)  # R * G = 280 rows: two row groups
    w = W.Workload("pool", 1, 8, 2, 64, tuple(lens), tuple(glens), synth.Stream(81, synth.TAG_Q),
                   synth.Stream(81, synth.TAG_K), synth.Stream(81, synth.TAG_V), keep_ratio=0.2, pool_k=pool)
    q, k, v = pu.device_inputs(w)
    a, b = pu.run_gpu(w, q, k, v, fused=True), pu.run_gpu(w, q, k, v, fused=False)
    for name in ("s_key", "s_comb", "scales", "kept_idx", "k_c", "v_q_c", "scales_c"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name


# The pooled one-workgroup selection in its larger register classes (16384, 32768 and 65536 tokens,
# whose pooling exchanges neighbours across lanes and waves), and its 256-thread class of more than 256
# short segments: (layers, KV heads, lengths).
POOLED_CLASSES = [(1, 2, [12000, 8195]), (1, 2, [32767, 17003]), (1, 2, [40001, 300]), (1, 2, [57341, 1]),
                  (2, 8, [65533, 9]), (8, 4, [57346]), (22, 4, [4093, 77, 1300])]


@pytest.mark.parametrize("L,Hkv,lens", POOLED_CLASSES, ids=lambda v: str(v).replace(", ", "-"))
@pytest.mark.parametrize("pool", [1, 3, 5, 7, 9])
def test_pooling_inside_selection_classes(gpu_lib, L, Hkv, lens, pool):
    w = W.Workload("pool", L, 4 * Hkv, Hkv, 64, tuple(lens), (70,) * len(lens), synth.Stream(82, synth.TAG_Q),
                   synth.Stream(82, synth.TAG_K), synth.Stream(82, synth.TAG_V), keep_ratio=0.2, pool_k=pool)
    q, k, v = pu.device_inputs(w)
    a, b = pu.run_gpu(w, q, k, v, fused=True), pu.run_gpu(w, q, k, v, fused=False)
    for name in ("s_key", "s_comb", "scales", "kept_idx", "k_c", "v_q_c", "scales_c"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name


# tp_evict's second stream: V just below and just above each line (with pass 1; normalisers given),
# bit for bit the separate calls, the overlapped ones also under capture and replayed.
@pytest.mark.parametrize("given_lse,full_codes,heads", [(False, True, 79), (False, True, 80), (False, False, 80),
                                                        (True, True, 127), (True, True, 128), (True, False, 129)])
def test_evict_overlap_line(gpu_lib, given_lse, full_codes, heads):
    w = W.Workload("line", 1, heads, heads, 128, (32768,), (8,), synth.Stream(91, synth.TAG_Q),
                   synth.Stream(91, synth.TAG_K, synth.DIST_STUDENT_T3), synth.Stream(91, synth.TAG_V), keep_ratio=0.1)
    assert heads * 32768 * 128 * 2 == heads * (8 << 20)  # V: 640 MB at 80 heads, 1 GB at 128
    q, k, v = pu.device_inputs(w)
    d, bt = B.dims(1, heads, heads, 128), B.Batch(w.ctx_offsets(), w.guide_offsets())
    kw = dict(softmax_scale=w.softmax_scale, pool_k=5, qfmt=0, bits=8, keep_ratio=0.1)
    names = ["s_key", "s_comb", "scales", "kept_idx", "k_c", "v_q_c", "scales_c"] + (["v_q"] if full_codes else [])
    lse = None
    ref = B.evict(d, bt, q, k, v, **kw)
    if given_lse:  # the separate calls with these normalisers
        lse = torch.linspace(9.0, 12.0, heads * 8, device="cuda")
        B.tp_guide_scores_lse(d, bt, q, k, lse, w.softmax_scale, 5, ref.s_key, ref.ws_evict)
        B.tp_combine_select_topk(d, bt, ref.s_key, ref.scales, 0, 0.1, 0, ref.kept_offsets, ref.kept_idx, ref.s_comb)
        B.tp_compact_kv(d, bt, ref.kept_offsets, ref.kept_idx, k, ref.v_q, ref.scales, 0, 8, ref.k_c, ref.v_q_c,
                        ref.scales_c)
    got = B.EvictBuffers(d, bt, 0, 8, ref.kept_offsets)
    B.evict_fused(d, bt, q, k, v, bufs=got, guide_lse=lse, full_codes=full_codes, **kw)
    torch.cuda.synchronize()
    for name in names:
        assert torch.equal(getattr(got, name), getattr(ref, name)), name
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        B.evict_fused(d, bt, q, k, v, bufs=got, guide_lse=lse, full_codes=full_codes, **kw)
    for _ in range(3):
        for name in names:
            getattr(got, name).zero_()
        g.replay()
        torch.cuda.synchronize()
        for name in names:
            assert torch.equal(getattr(got, name), getattr(ref, name)), name


OVERLAP_NAMES = ("s_key", "s_comb", "scales", "kept_idx", "k_c", "v_q_c", "scales_c", "v_q")


def _overlap_workload(L, Hq, Hkv, d, lens, glens, **kw):
    w = W.Workload("overlap", L, Hq, Hkv, d, tuple(lens), tuple(glens), synth.Stream(93, synth.TAG_Q),
                   synth.Stream(93, synth.TAG_K, synth.DIST_STUDENT_T3), synth.Stream(93, synth.TAG_V), keep_ratio=0.1,
                   **kw)
    assert w.L * w.Hkv * w.n_tot * w.d * 2 >= 640 << 20  # the second stream is used
    return w


# The overlapped step 2 in each code format, both head sizes, every size of its parts (by the guide
# rows a token meets) and ragged batches whose parts begin and end inside a segment: (layers, query
# heads, KV heads, head_dim, context lengths, guide lengths, options).
OVERLAP_CASES = {
    "int4-ragged": (3, 16, 8, 128, [60001, 30003, 20007], [9, 70, 33], dict(bits=4)),
    "int5-256-rows": (1, 64, 16, 128, [90001, 74001], [60, 64], dict(bits=5)),  # 7/20 beside each pass
    "int2-short-guide": (2, 16, 16, 128, [82001], [48], dict(bits=2)),
    "e4m3-long-guide": (2, 32, 8, 128, [100003, 64001], [80, 65], dict(qfmt=1)),  # 2/5 beside each pass
    "int8-d64": (4, 16, 16, 64, [50001, 32003], [16, 5], dict()),
    "int4-d64": (4, 16, 16, 64, [82005], [40], dict(bits=4)),
    "int6-d64": (4, 16, 16, 64, [82005], [3], dict(bits=6)),
    "e4m3-d64": (4, 16, 16, 64, [41001, 41003], [7, 7], dict(qfmt=1)),
    "norm-add": (2, 32, 16, 128, [82005], [20], dict(rule=1)),
    "harmonic-wide-pool": (2, 32, 16, 128, [50001, 32004], [20, 90], dict(rule=2, pool_k=13)),
}


@pytest.mark.parametrize("guide_keys,full_codes", [(False, True), (True, False)])
@pytest.mark.parametrize("name", OVERLAP_CASES)
def test_evict_overlapped_forms(gpu_lib, name, guide_keys, full_codes):
    *shape, kw = OVERLAP_CASES[name]
    w = _overlap_workload(*shape, **kw)
    q, k, v = pu.device_inputs(w)
    kg = pu.device_guide_keys(w) if guide_keys else None
    d, bt = B.dims(w.L, w.Hq, w.Hkv, w.d), B.Batch(w.ctx_offsets(), w.guide_offsets())
    opts = dict(softmax_scale=w.softmax_scale, pool_k=w.pool_k, qfmt=w.qfmt, bits=w.bits, rule=w.rule, keep_ratio=0.1,
                k_guide=kg)
    ref = B.evict(d, bt, q, k, v, **opts)
    got = B.evict_fused(d, bt, q, k, v, full_codes=full_codes, **opts)
    torch.cuda.synchronize()
    for n in OVERLAP_NAMES if full_codes else OVERLAP_NAMES[:-1]:
        assert torch.equal(getattr(got, n), getattr(ref, n)), n


# With the normalisers given the line is 1 GB of V; parts of 1/5, 3/10 and 1/2 beside pass 2, and for
# scales only 1/5 in one workgroup per CU and 3/5 in two.
@pytest.mark.parametrize("full_codes", [True, False])
@pytest.mark.parametrize("name,lens,glens,kw", [("int4", [131073, 131077], [9, 17], dict(bits=4)),
                                                ("e4m3-256-rows", [262147], [64], dict(qfmt=1)),
                                                ("int7-long-guide", [200001, 62147], [70, 90], dict(bits=7)),
                                                ("d64", [262147, 262145], [16, 16], dict(d=64))])
def test_evict_overlapped_given_normalisers(gpu_lib, name, lens, glens, kw, full_codes):
    kw = dict(kw)
    w = _overlap_workload(2, 32, 8, kw.pop("d", 128), lens, glens, **kw)
    assert w.L * w.Hkv * w.n_tot * w.d * 2 >= 1 << 30
    q, k, v = pu.device_inputs(w)
    d, bt = B.dims(w.L, w.Hq, w.Hkv, w.d), B.Batch(w.ctx_offsets(), w.guide_offsets())
    opts = dict(softmax_scale=w.softmax_scale, pool_k=w.pool_k, qfmt=w.qfmt, bits=w.bits, keep_ratio=0.1)
    lse = torch.linspace(9.0, 12.0, w.L * w.Hq * w.g_tot, device="cuda")
    got = B.evict_fused(d, bt, q, k, v, guide_lse=lse, full_codes=full_codes, **opts)
    ref = B.EvictBuffers(d, bt, w.qfmt, w.bits, got.kept_offsets)
    B.tp_guide_scores_lse(d, bt, q, k, lse, w.softmax_scale, w.pool_k, ref.s_key, ref.ws_evict)
    B.tp_quantize_v_scales(d, bt, v, w.qfmt, w.bits, ref.scales, ref.v_q)
    B.tp_combine_select_topk(d, bt, ref.s_key, ref.scales, w.rule, 0.1, 0, ref.kept_offsets, ref.kept_idx, ref.s_comb)
    B.tp_compact_kv(d, bt, ref.kept_offsets, ref.kept_idx, k, ref.v_q, ref.scales, w.qfmt, w.bits, ref.k_c, ref.v_q_c,
                    ref.scales_c)
    torch.cuda.synchronize()
    for n in OVERLAP_NAMES if full_codes else OVERLAP_NAMES[:-1]:
        assert torch.equal(getattr(got, n), getattr(ref, n)), n


def test_evict_overlapped_threads(gpu_lib):
    """Two host threads with overlapped calls at the same time, each on its own stream with its own
    buffers: the calls share the device's second stream and events, whose use a lock serialises
    while enqueueing; every result equals the separate calls'."""
    import threading

    w = _overlap_workload(1, 80, 80, 128, [32769], [8])
    q, k, v = pu.device_inputs(w)
    d, bt = B.dims(w.L, w.Hq, w.Hkv, w.d), B.Batch(w.ctx_offsets(), w.guide_offsets())
    opts = dict(softmax_scale=w.softmax_scale, pool_k=w.pool_k, qfmt=w.qfmt, bits=w.bits, keep_ratio=0.1)
    ref = B.evict(d, bt, q, k, v, **opts)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    bufs = [B.EvictBuffers(d, bt, w.qfmt, w.bits, ref.kept_offsets) for _ in streams]
    for st in streams:
        st.wait_stream(torch.cuda.current_stream())
    errors = []

    def worker(i):
        try:
            for _ in range(4):
                B.evict_fused(d, bt, q, k, v, bufs=bufs[i], stream=streams[i], **opts)
            streams[i].synchronize()
        except Exception as e:  # reported below
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    torch.cuda.synchronize()
    for b in bufs:
        for n in OVERLAP_NAMES:
            assert torch.equal(getattr(b, n), getattr(ref, n)), n


# Attention chunks: multiples of 64 tokens in calls of few workgroups, 8192 from three rounds on.  Grids
# of up to 512 workgroups are padded to the longest sequence and guide, larger ones compact.
ATTN_CASES = [
    ("unit-edges", 1, 8, 2, 128, [63, 64, 65, 129, 700, 1], [16, 3, 64, 9, 33, 1], True),
    ("even-cuts", 1, 8, 2, 64, [4097, 2333, 7681], [16, 80, 40], True),
    ("many-slots", 1, 2, 1, 128, [12000], [5], False),  # more chunks than the merge loads at once
    # compact grid: ten to one row groups a sequence, a guide longer than its sequence's chunks (first)
    ("ragged-compact", 2, 16, 2, 64, [3000, 130, 1200, 65, 2500], [300, 3, 40, 129, 1], True),
    ("ragged-compact-128", 2, 16, 2, 128, [2100, 64, 700], [40, 150, 1], False),
    ("usual-chunk", 12, 64, 64, 64, [90, 8193], [2, 1], True),  # > 768 workgroups
]


@pytest.mark.parametrize("case", ATTN_CASES, ids=[c[0] for c in ATTN_CASES])
def test_attention_chunks(gpu_lib, case):
    w, guide_keys = tga._workload(case), case[-1]
    (q, k, v, kg, vg), o_gpu, lse_gpu = tga._run_attention(w, guide_keys)
    for l in {0, w.L - 1}:
        for h in {0, w.Hkv - 1}:
            for b in range(w.batch):
                tga._check_rows(w, b, l, h, range(h * w.R, (h + 1) * w.R), o_gpu, lse_gpu, guide_keys)
    # the quantising instance: the same attention and every token's scale and codes
    d, bt = B.dims(w.L, w.Hq, w.Hkv, w.d), B.Batch(w.ctx_offsets(), w.guide_offsets())
    n = w.L * w.Hkv * w.n_tot
    out = torch.empty(o_gpu.size, device="cuda"), torch.empty(lse_gpu.size, device="cuda")
    got = torch.full((n,), -1.0, device="cuda"), torch.full((n * w.d,), 77, dtype=torch.uint8, device="cuda")
    ref = torch.empty(n, device="cuda"), torch.empty(n * w.d, dtype=torch.uint8, device="cuda")
    B.tp_guide_attention_quantize(d, bt, q, k, v, w.softmax_scale, 0, 8, *out, *got, k_guide=kg, v_guide=vg)
    B.tp_quantize_v_scales(d, bt, v, 0, 8, *ref)
    torch.cuda.synchronize()
    assert torch.equal(out[0].cpu(), torch.from_numpy(o_gpu.ravel()))
    assert torch.equal(out[1].cpu(), torch.from_numpy(lse_gpu.ravel()))
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
