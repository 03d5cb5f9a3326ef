"""gate||up and down on MXFP8 operands (gemm_mx_kernel): every tile, one turn of the loop and several, eight steps in LDS and four, a k range for
each die and fewer, a last range shorter than the others, rows that end inside a tile or next to one, against the oracle that rounds the
same operands (all per-layer taps of the whole pass); graph replays give the same bits."""
import dataclasses

import numpy as np
import pytest

from paper_2510_26742_amd import binding, build, synth
from tests.test_gpu_parity import CACHE_TOL, DIRECT_LAUNCHES, MX_ACTION_TOL, MX_COS_MIN, MX_ROW_COS_MIN, Case, check_against_oracle
from tests.test_loop_code_size import code_objects, symbols

FULL_WIDTH = dataclasses.replace(synth.reduced_config(vocab=64), max_prompt=255)
NARROW = dataclasses.replace(FULL_WIDTH, llm_width=256, llm_q_heads=3, exp_width=128, exp_mlp=192)   # gate||up: k 256


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,shapes", [(FULL_WIDTH, ((1, 7), (1, 128), (2, 0), (2, 33), (3, 1))),
                                        (dataclasses.replace(NARROW, llm_mlp=256), ((1, 0), (2, 1))),                     # down: one range of one turn
                                        (dataclasses.replace(NARROW, llm_mlp=2304), ((1, 1), (3, 65))),                   # ranges of 512 and 256
                                        (dataclasses.replace(NARROW, llm_mlp=4096), ((1, 0), (1, 1), (1, 65), (2, 128)))],  # a range of 512 for each die
                         ids=["full width", "one range", "short last range", "range per die"])
def test_mxfp8_tiles_match_the_oracle(cfg, shapes):
    case = Case(cfg)
    try:
        case.m.pi0_set_precision("mxfp8_prefix_mlp")
        for n_views, n_prompt in shapes:
            act, _ = check_against_oracle(case, n_views, n_prompt, seed_shift=17 * n_prompt, label=f"mxfp8 {cfg.llm_width} x {cfg.llm_mlp}, {n_views} views + {n_prompt}", mxfp8=True,
                                          action_tol=MX_ACTION_TOL, cos_min=MX_COS_MIN, row_cos_min=MX_ROW_COS_MIN, cache_tol=2 * CACHE_TOL)
            inputs = case.inputs(n_views, n_prompt, 17 * n_prompt)
            for tune in ("pvl=0", "pvl=1"):   # enough kernels for a graph, and as a call comes
                case.m.pi0_tune(tune)
                assert tune == "pvl=1" or case.m.pi0_kernel_count(n_views, n_prompt) > DIRECT_LAUNCHES
                for _ in range(2):
                    np.testing.assert_array_equal(case.infer(*inputs), act)
    finally:
        case.close()


def test_mxfp8_tiles_spill_no_registers():
    binding.lib()
    with open(build.LIB, "rb") as f:
        library = f.read()
    found = {k: v for code in code_objects(library) for k, v in symbols(code).items() if "gemm_mx_kernel" in k and k.endswith(".private_seg_size")}
    assert len(found) == 13 and all(v[0] == 0 for v in found.values()), found
