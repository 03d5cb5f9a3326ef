"""What a prefill leaves in the key / value cache behind its last token does not reach a later, shorter one: the rows up to the end
of the 32-token chunk are masked, and masked means exactly nothing also where an earlier call left NaN there (0 * NaN is NaN,
so zero probabilities alone are not enough: the value rows have to be overwritten)."""
import dataclasses

import numpy as np
import pytest

from paper_2510_26742_amd import synth
from tests.test_gpu_parity import Case, check_against_oracle

pytestmark = pytest.mark.gpu

# Three layers: the first one's keys and values of prompt tokens depend on no image, the last one's kernel takes two tiles per block.
EIGHT_HEADS = dataclasses.replace(synth.reduced_config(vocab=64), llm_layers=3, exp_layers=3)
# three query heads: 24 + 8 feature tiles of queries and keys in front of the values, which three feature tiles per block straddle
THREE_HEADS = dataclasses.replace(EIGHT_HEADS, vis_width=576, vis_heads=8, vis_mlp=100, llm_width=192, llm_mlp=320,
                                  llm_q_heads=3, exp_width=128, exp_mlp=192)


# lqkv=1: the register-staged QKV kernel, which the default schedule does not take
@pytest.mark.parametrize("cfg,precision,tune", [
    pytest.param(EIGHT_HEADS, "bf16", None, id="eight heads"), pytest.param(EIGHT_HEADS, "bf16", "lqkv=1", id="eight heads, register-staged"),
    pytest.param(EIGHT_HEADS, "mxfp8_prefix_mlp", None, id="eight heads, mxfp8"),
    pytest.param(THREE_HEADS, "bf16", None, id="three heads"), pytest.param(THREE_HEADS, "bf16", "lqkv=1", id="three heads, register-staged"),
])
def test_a_prefill_with_nan_leaves_nothing_behind(cfg, precision, tune):
    case = Case(cfg, tune=tune)
    try:
        case.m.pi0_set_precision(precision)
        for n_views, n_prompt in ((1, 7), (2, 21), (3, 15)):   # 263, 533, 783 tokens: nothing is a multiple of 32
            inputs = case.inputs(n_views, n_prompt)
            before = case.infer(*inputs)
            img, st, nz, ids = case.inputs(n_views, n_prompt // 32 * 32 + 32)   # to the end of the same chunk
            assert np.isnan(case.infer(np.full_like(img, np.nan), st, nz, ids)).all()
            np.testing.assert_array_equal(case.infer(*inputs), before)
    finally:
        case.close()


def test_blocks_of_queries_or_keys_and_values_where_chunks_are_whole():
    """800 tokens are whole chunks: there three feature tiles per block may still straddle the boundary between keys and values."""
    case = Case(THREE_HEADS)
    try:
        check_against_oracle(case, 3, 32, label="three heads, 800 tokens")
    finally:
        case.close()
