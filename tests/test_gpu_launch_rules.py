"""Shapes on the far side of the rules that choose a kernel by the size of the call, with lengths that end inside a tile: the small
parity cases of the other files take the kernels for few blocks only.  Checked as the full-size workloads are: the complete forward
of sampled heads and sampled rows of the gradients against the oracle, and identities of the gradients on every head."""
import pytest

from paper_2410_09397_amd import synth
from tests.test_gpu_fullsize import check_at_full_size

pytestmark = pytest.mark.gpu

RULES = [
    # large d, product tiles of 256 x 256 in both directions (144 tiles forward, 432 backward); three row blocks, the last with 8 rows
    synth.Workload("wide_products_d512", 81, 1, 24, 520, 512, "bf16"),
    # the same under the causal rule (270 and 810 tiles): tiles of one to nine row blocks, the last with 2 rows
    synth.Workload("wide_products_d512_causal", 82, 1, 15, 2050, 512, "bf16", causal=True),
    # 256 x 128 forward (72 tiles), 256 x 256 backward (216), four column tiles
    synth.Workload("wide_backward_d1024", 83, 1, 9, 300, 1024, "bf16"),
]


@pytest.mark.parametrize("w", RULES, ids=lambda w: w.name)
def test_large_calls_of_odd_length(w):
    check_at_full_size(w, w.index)
