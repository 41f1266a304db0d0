"""The launch rules that depend on sizes: each side of every line, on ragged and smallest shapes,
against the CPU oracle (the comparison rules are parity_util's)."""
import pytest

import synth

import test_gpu_parity as tgp

pytestmark = pytest.mark.gpu

# Score-pass chunks: multiples of 256 tokens, cut evenly per sequence; up to 768 workgroups pass 2
# merges the chunks' statistics itself, beyond that a kernel does.
CHUNK_CASES = [
    ("unit-edges", 1, 8, 2, 128, [255, 256, 257, 511, 513, 1], [16, 3, 64, 9, 33, 1], synth.DIST_NORMAL, 5),
    ("even-cuts", 1, 8, 2, 64, [4097, 2333, 7681], [16, 80, 40], synth.DIST_STUDENT_T3, 3),
    ("merge-kernel", 14, 32, 8, 64, [513, 70, 300], [64, 130, 5], synth.DIST_NORMAL, 5),  # > 768 workgroups
]


@pytest.mark.parametrize("guide_keys", [False, True])
@pytest.mark.parametrize("case", CHUNK_CASES, ids=[c[0] for c in CHUNK_CASES])
def test_score_pass_chunks(gpu_lib, case, guide_keys):
    tgp._guide_case(case, guide_keys)
