"""Attention of prompts: groups of query rows with two key groups per workgroup, and the steps that need a mask or none."""
import numpy as np
import pytest

from paper_2512_09963_amd import synth
from tests.test_routes import attention_key_groups
from tests.test_verify_gpu import _run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,n_kv,hd,page,gamma,ctx,groups", [
    (64, 8, 64, 16, [511], [0], 2),                # 32 groups of 16 tokens, up to 16 steps, every group another odd or even number
    (64, 8, 64, 48, [300, 2, 230], [33, 700, 0], 2),      # pages of three tiles; a block of one group beside them
    (64, 8, 64, 16, [223, 223, 64], [0, 0, 0], 1),        # 7 steps
    (32, 8, 128, 32, [1000], [0], 2),
    (64, 64, 64, 16, [383, 127], [31, 600], 2),           # 128 tokens a group: every wave another limit
    (32, 16, 64, 64, [511, 500], [1, 40], 2),
])
def test_prompt_groups(heads, n_kv, hd, page, gamma, ctx, groups):
    """Against the float64 oracle within 2e-2 of the row scale (bfloat16 activations and pages)."""
    assert attention_key_groups(n_kv, heads // n_kv, gamma, ctx)[0] == groups
    ms = synth.ModelShape(1, 256, heads, n_kv, hd, 256, 512, 10000.0, dtype="bf16")
    _run_case(ms, 61 + page, np.array(gamma, np.int32), np.array(ctx, np.int32), page, 0.05)
