"""gate||up and down beyond 512 rows on tiles of seven and nine blocks of 32 rows, with a lower body for the rows that are left over
(gemm_cols_body): the token counts where the body or the number of tiles changes, a contraction of one turn of the loop, a last k range shorter than
the others, against the CPU oracle through the whole pass (all per-layer taps, which the launches leave).  That the persistent prefix gives the launches' bits is
test_gpu_prefix_loop's."""
import dataclasses

import pytest

from paper_2510_26742_amd import binding, build, synth
from tests.test_gpu_parity import Case, check_against_oracle
from tests.test_loop_code_size import code_objects, symbols

FULL_WIDTH = dataclasses.replace(synth.reduced_config(vocab=64), max_prompt=255)
ONE_TURN = dataclasses.replace(FULL_WIDTH, llm_width=256, llm_q_heads=3, exp_width=128, exp_mlp=192)   # gate||up: k 256
SHORT_RANGE = dataclasses.replace(FULL_WIDTH, llm_mlp=9728)                                           # down: ranges of 1280, the last 768


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,shapes", [(FULL_WIDTH, ((2, 1), (2, 32), (2, 33), (2, 64), (3, 1), (3, 32), (3, 33), (3, 64), (3, 65), (3, 96), (3, 128))),
                                        (ONE_TURN, ((2, 1), (2, 64), (3, 33), (3, 128))), (SHORT_RANGE, ((2, 33), (3, 48), (3, 128)))],
                         ids=["full width", "one turn", "short last range"])
def test_tall_tiles_match_the_oracle(cfg, shapes):
    case = Case(cfg)
    try:
        for n_views, n_prompt in shapes:
            check_against_oracle(case, n_views, n_prompt, seed_shift=17 * n_prompt, label=f"{cfg.llm_width} x {cfg.llm_mlp}, {n_views} views + {n_prompt}")
    finally:
        case.close()


@pytest.mark.parametrize("kernel", ["gemm_cols_kernelILi7ELi4EE", "gemm_cols_kernelILi9ELi4EE", "gemm_cols_kernelILi7ELi0EE", "prefix_loop_kernelILi5EE"])
def test_tall_tiles_spill_no_registers(kernel):
    binding.lib()
    with open(build.LIB, "rb") as f:
        library = f.read()
    found = {k: v for code in code_objects(library) for k, v in symbols(code).items() if kernel in k}
    (name, _), = [(k, v) for k, v in found.items() if "." not in k]
    assert found[name + ".private_seg_size"][0] == 0
