"""The prefix's gate||up and down through LDS (gemm_tile.hip) at the edges of what they take: a contraction of one turn of the loop, one
that splits into unequal ranges, feature counts that fill no tile, token counts around every tile height, against the
CPU oracle through the whole pass (all per-layer taps)."""
import dataclasses

import pytest

from paper_2510_26742_amd import synth
from tests.test_gpu_parity import Case, check_against_oracle

pytestmark = pytest.mark.gpu

# gate||up: k 128 (one turn), 1280 features; down: k 640 in ranges of 128 and 256, 128 features
ONE_TURN = dataclasses.replace(synth.reduced_config(vocab=64), llm_width=128, llm_mlp=640, llm_q_heads=3, exp_width=128, exp_mlp=192)
# gate||up: k 384, 1792 features; down: k 896, 384 features
ODD_TILES = dataclasses.replace(synth.reduced_config(vocab=64), llm_width=384, llm_mlp=896, llm_q_heads=3, exp_width=128, exp_mlp=192)


@pytest.fixture(scope="module", params=["one turn", "odd tiles"])
def case(request):
    c = Case({"one turn": ONE_TURN, "odd tiles": ODD_TILES}[request.param])
    yield c
    c.close()


@pytest.mark.parametrize("n_views,n_prompt", [(1, 0), (1, 1), (1, 48), (2, 0), (2, 1), (3, 0), (3, 48)])
def test_large_prefix_gemms_match_the_oracle(case, n_views, n_prompt):
    check_against_oracle(case, n_views, n_prompt, seed_shift=11 * n_prompt, label=f"{case.cfg.llm_width} wide, {n_views} views + {n_prompt}")


# Down over eight ranges, a die each: the last range shorter than the others (one turn of four stages, one of eight), and every tile that the rule picks at
# the full model's width (128 x 128 .. 320 x 128, 192 x 256), at both ends of the token counts that it picks it for
SHORT_RANGE = dataclasses.replace(synth.reduced_config(vocab=64), llm_width=256, llm_mlp=1920, llm_q_heads=3, exp_width=128, exp_mlp=192)   # ranges of 256, the last 128
SHORT_RANGE_8 = dataclasses.replace(SHORT_RANGE, llm_width=1024, llm_mlp=3840)                                                            # of 512, the last 256
FULL_WIDTH = dataclasses.replace(synth.reduced_config(vocab=64), max_prompt=255)


@pytest.mark.parametrize("cfg,shapes", [(SHORT_RANGE, ((1, 0), (1, 1), (2, 1))), (SHORT_RANGE_8, ((1, 0), (1, 1), (2, 1))),
                                        (FULL_WIDTH, ((1, 64), (1, 128), (1, 129), (2, 64), (2, 65), (2, 128), (2, 129)))],
                         ids=["short last range", "short last range, eight stages", "full width"])
def test_a_range_per_die_matches_the_oracle(cfg, shapes):
    case = Case(cfg)
    try:
        for n_views, n_prompt in shapes:
            check_against_oracle(case, n_views, n_prompt, seed_shift=13 * n_prompt, label=f"{cfg.llm_width} x {cfg.llm_mlp}, {n_views} views + {n_prompt}")
    finally:
        case.close()
