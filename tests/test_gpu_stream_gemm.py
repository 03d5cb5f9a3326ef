"""The mid-size GEMMs of the prefill (gemm_stream.hip) at the edges of what they take: k ranges that leave waves without
a step, feature counts that fill no tile, token counts that end inside a tile, heads across tiles, every tile of the choice, against the
CPU oracle through the whole pass (all per-layer taps)."""
import dataclasses

import pytest

from paper_2510_26742_amd import synth
from tests.test_gpu_parity import Case, check_against_oracle

pytestmark = pytest.mark.gpu

# k of 576 / 192 (36 and 12 steps over 8 waves: two waves have none), 100 -> 128 and 320 columns
NARROW = dataclasses.replace(synth.reduced_config(vocab=64), vis_width=576, vis_heads=8, vis_mlp=100, llm_width=192, llm_mlp=320,
                             llm_q_heads=3, exp_width=128, exp_mlp=192)
FULL_WIDTH = synth.reduced_config(vocab=64)
# heads of 76: 8 features straddle heads, and a block's feature tiles queries, keys and values; an odd number of column tiles
STRADDLING = dataclasses.replace(synth.reduced_config(vocab=64), vis_width=1216, vis_heads=16, vis_mlp=100, llm_width=320, llm_mlp=320,
                                 llm_q_heads=5, exp_width=128, exp_mlp=192)


@pytest.fixture(scope="module", params=["narrow", "full width", "straddling"])
def case(request):
    c = Case({"narrow": NARROW, "full width": FULL_WIDTH, "straddling": STRADDLING}[request.param])
    yield c
    c.close()


@pytest.mark.parametrize("n_views,n_prompt", [(1, 0), (1, 7), (1, 33), (2, 1), (2, 31), (3, 47)])
def test_prefill_gemms_match_the_oracle(case, n_views, n_prompt):
    check_against_oracle(case, n_views, n_prompt, seed_shift=7 * n_prompt, label=f"{case.cfg.llm_width} wide, {n_views} views + {n_prompt}")
