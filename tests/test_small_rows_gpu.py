"""Edges of the kernels that serve blocks of a few rows: the fp32 attention's chunks of 128 keys and its page sizes."""
import numpy as np
import pytest

from paper_2512_09963_amd import synth
from tests.test_verify_gpu import _run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,page,gamma,ctx", [
    (64, 16, [0, 1, 2, 0], [0, 126, 127, 128]),        # 1 key; the last row at, the first past a chunk of 128
    (64, 7, [3, 0, 5], [13, 255, 300]),                # pages that are no multiple of 4: scalar loads
    (128, 1, [2, 1], [3, 130]),
    (128, 12, [4, 6], [253, 40]),                      # a multiple of 4 but not of 16
    (128, 64, [1, 15], [512, 1]),
])
def test_f32_attention_chunks_and_page_sizes(hd, page, gamma, ctx):
    """Against the float64 oracle within 1e-4 of the row scale (float32 sums of at most a few hundred terms: about 1e-6)."""
    ms = synth.ModelShape(2, 4 * hd, 4, 2, hd, 384, 320, 10000.0, dtype="f32")
    _run_case(ms, 41 + page, np.array(gamma, np.int32), np.array(ctx, np.int32), page, 0.05)
