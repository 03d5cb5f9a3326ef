"""The vision tower of pi0_infer and pi0_prefill runs as one persistent kernel with grid barriers; with pvl=0 its operations are launched one by one.  Both
add up every sum in the same order, so they agree bit for bit, whatever the number of views and whatever a replay before left in the
kernel's buffers.  (The launches are compared with the oracle in test_gpu_parity.py.)"""
import dataclasses

import numpy as np
import pytest

from paper_2510_26742_amd import binding, build, synth
from tests.test_gpu_parity import Case, say
from tests.test_loop_code_size import INSTRUCTION_CACHE, code_objects, symbols

CFG = dataclasses.replace(synth.reduced_config(vocab=64), vis_layers=3, max_views=4, max_prompt=0)   # a first, a middle and a last layer


@pytest.mark.gpu
@pytest.mark.parametrize("graphs", [True, False])
def test_infer_equals_prefill_and_denoise(graphs):
    case = Case(CFG)
    try:
        case.m.pi0_set_graph_mode(graphs)
        # 4 views: more than the kernel covers, launches in both; back and forth, so that every replay finds another call's buffers
        for n_views in (1, 3, 2, 4, 1, 2, 3):
            img, st, nz, ids = case.inputs(n_views, 0)
            say(f"[gpu] vision loop views={n_views} graphs={graphs}")
            want = case.by_launches(img, st, nz, ids)
            np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
            assert np.isnan(case.infer(np.full_like(img, np.nan), st, nz, ids)).all()
            for _ in range(3):
                np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
            np.testing.assert_array_equal(case.prefill_and_denoise(img, st, nz, ids), want)
            launches = case.m.pi0_kernel_count(n_views, 0)
            case.m.pi0_tune("pvl=0")
            np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
            # five operations a layer, and beyond 256 tokens a launch that adds up row statistics, become two launches in all
            assert case.m.pi0_kernel_count(n_views, 0) - launches == (0 if n_views > 3 else CFG.vis_layers * (5 + (n_views > 1)) - 2)
            case.m.pi0_tune("pvl=1")
        case.m.pi0_device_status(case.stream)   # raises if a bounded wait ran out
    finally:
        case.close()


# 216 blocks of the kernel run GEMM items; up needs, with the tiles that the launches choose as well: 216 of them (the most that fit),
# 224 and 228 (more than run items), 390 (more than the grid).  Where they do not fit pi0_infer launches the tower's operations.
@pytest.mark.gpu
@pytest.mark.parametrize("vis_mlp,views", [(5120, 1), (5376, 1), (4608, 2), (4864, 2), (4608, 3), (4864, 3), (8320, 3)])
def test_feed_forward_widths_around_one_round(vis_mlp, views):
    case = Case(dataclasses.replace(CFG, vis_mlp=vis_mlp))
    try:
        img, st, nz, ids = case.inputs(views, 0)
        say(f"[gpu] vision loop vis_mlp={vis_mlp} views={views}")
        want = case.by_launches(img, st, nz, ids)
        for _ in range(2):
            np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
        case.m.pi0_device_status(case.stream)
    finally:
        case.close()


@pytest.mark.parametrize("views", [1, 2, 3])
def test_vision_loop_fits_the_instruction_cache(views):
    """as test_loop_code_size.py for the denoise loop; nothing spilled"""
    binding.lib()
    with open(build.LIB, "rb") as f:
        library = f.read()
    found = {k: v for code in code_objects(library) for k, v in symbols(code).items() if f"vision_loop_kernelILi{views}EE" in k}
    (name, (_, size)), = [(k, v) for k, v in found.items() if "." not in k]
    assert 0 < size <= INSTRUCTION_CACHE, (name, size)
    assert found[name + ".private_seg_size"][0] == 0, "registers spilled"
