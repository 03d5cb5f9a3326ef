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


# the prefix's feed-forward tiles (gemm_tile.hip, contractions in multiples of 128): one and three turns of the operand ring
# (where the block column starts in it), five of the down projection, 257 and 289 tokens (statistics are read in pairs of
# rows), and 32 planes of statistics for 320 rows, more than LDS holds at once
@pytest.mark.parametrize("width,mlp,tune,n_views,n_prompt", [
    (128, 128, None, 1, 0), (128, 128, None, 1, 1), (384, 640, None, 1, 0), (384, 640, None, 1, 33), (384, 640, None, 2, 0),
    (384, 640, "fkl=1", 1, 1), (384, 640, "fkl=1", 3, 5), (2048, 16384, "fkl=1", 1, 7), (2048, 16384, "fkl=1", 2, 3),
])
def test_prefix_feed_forward_tiles_match_the_oracle(width, mlp, tune, n_views, n_prompt):
    cfg = FULL_WIDTH if width == 2048 else dataclasses.replace(FULL_WIDTH, llm_width=width, llm_mlp=mlp, llm_q_heads=width // 128 * 2 - 1)
    case = Case(cfg, tune=tune)
    try:
        check_against_oracle(case, n_views, n_prompt, seed_shift=3 * n_prompt, label=f"feed-forward {width} x {mlp}, {n_views} views + {n_prompt}, {tune}")
    finally:
        case.close()
