"""The prefix of pi0_infer and pi0_prefill runs as one persistent kernel with grid barriers; with ppl=0 its operations are launched one by one.  Both add up
every sum in the same order, so they agree bit for bit: at both ends of every range of prefix tokens that has a variant of its own, inside it
and next to it, and whatever a replay before left in the kernel's buffers.  (The launches are compared with the oracle in
test_gpu_parity.py.)"""
import dataclasses
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2510_26742_amd import binding, build, synth
from tests.test_gpu_parity import Case, say
from tests.test_loop_code_size import code_objects, symbols

CFG = dataclasses.replace(synth.reduced_config(vocab=64), llm_layers=4, exp_layers=4, max_prompt=48)   # three whole prefix layers


@pytest.mark.gpu
@pytest.mark.parametrize("graphs", [True, False])
def test_infer_equals_prefill_and_denoise(graphs):
    case = Case(CFG)
    try:
        case.m.pi0_set_graph_mode(graphs)
        for n_views, n_prompt in ((1, 0), (1, 1), (3, 48), (1, 48), (2, 0), (2, 31), (2, 1), (3, 0), (2, 48), (3, 1), (1, 7), (1, 0)):
            img, st, nz, ids = case.inputs(n_views, n_prompt)
            say(f"[gpu] prefix loop views={n_views} prompt={n_prompt} graphs={graphs}")
            want = case.by_launches(img, st, nz, ids)
            np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
            assert np.isnan(case.infer(np.full_like(img, np.nan), st, nz, ids)).all()
            for _ in range(2):
                np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
            np.testing.assert_array_equal(case.prefill_and_denoise(img, st, nz, ids), want)
            launches = case.m.pi0_kernel_count(n_views, n_prompt)
            case.m.pi0_tune("ppl=0")
            np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
            # five operations a whole layer, and beyond 256 tokens a launch that adds up row statistics, and the QKV projections between
            # them become two launches in all
            tokens, layers = 256 * n_views + n_prompt, CFG.llm_layers - 1
            assert case.m.pi0_kernel_count(n_views, n_prompt) - launches == (0 if tokens > 768 else layers * (5 + (tokens > 256)) + layers - 1 - 2)
            case.m.pi0_tune("ppl=1")
        case.m.pi0_device_status(case.stream)   # raises if a bounded wait ran out
    finally:
        case.close()


# The variants and where they end, with the full model's feed-forward: 193 .. 256, 257 .. 320, 385 .. 512, 513 .. 576, 641 .. 768 tokens
# (prefix_loop_tiles says which tiles, gemm_stream_tile and gemm_lds_tile where the launches choose the same ones).  What lies between runs
# as launches.  (views, prompt) of 256-token views, and of 64-token ones for fewer than 256.
RANGES = [(193, 256), (257, 320), (385, 512), (513, 576), (641, 768)]
WHOLE_VIEWS = dict(shapes=[(1, 0), (1, 64), (1, 65), (1, 128), (1, 129), (1, 135), (1, 191), (1, 255), (2, 1), (2, 32), (2, 33), (2, 64), (2, 65), (2, 128), (2, 129),
                           (2, 188), (2, 255), (3, 0), (3, 1)], max_prompt=255)
SMALL_VIEWS = dict(shapes=[(3, 0), (3, 1), (3, 8), (3, 31), (3, 33), (3, 63), (4, 0)], max_views=4, img_size=112, max_prompt=63)


@pytest.mark.gpu
@pytest.mark.parametrize("small", [False, True])
def test_ragged_lengths_of_every_variant(small):
    kw = dict(SMALL_VIEWS if small else WHOLE_VIEWS)
    shapes = kw.pop("shapes")
    case = Case(dataclasses.replace(CFG, **kw))
    try:
        for n_views, n_prompt in shapes:
            tokens = n_views * case.cfg.tokens_per_view + n_prompt
            say(f"[gpu] prefix loop, {tokens} tokens")
            img, st, nz, ids = case.inputs(n_views, n_prompt)
            want = case.by_launches(img, st, nz, ids)
            np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
            assert np.isnan(case.infer(np.full_like(img, np.nan), st, nz, ids)).all()
            np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
            launches = case.m.pi0_kernel_count(n_views, n_prompt)
            case.m.pi0_tune("ppl=0")
            assert (case.m.pi0_kernel_count(n_views, n_prompt) > launches) == any(a <= tokens <= b for a, b in RANGES)
            case.m.pi0_tune("ppl=1")
        case.m.pi0_device_status(case.stream)
    finally:
        case.close()


# A narrow feed-forward sends every prefix of up to 256 tokens to the first variant, however short
@pytest.mark.gpu
@pytest.mark.parametrize("llm_mlp", [2048, 4096])
def test_short_prefixes_of_a_narrow_feed_forward(llm_mlp):
    case = Case(dataclasses.replace(CFG, llm_mlp=llm_mlp, max_views=4, img_size=112, max_prompt=63))
    try:
        for n_views, n_prompt in ((1, 0), (1, 1), (1, 31), (2, 0), (2, 37), (3, 0), (4, 0)):
            say(f"[gpu] prefix loop, llm_mlp {llm_mlp}, {64 * n_views + n_prompt} tokens")
            img, st, nz, ids = case.inputs(n_views, n_prompt)
            want = case.by_launches(img, st, nz, ids)
            for _ in range(2):
                np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
            launches = case.m.pi0_kernel_count(n_views, n_prompt)
            case.m.pi0_tune("ppl=0")
            assert case.m.pi0_kernel_count(n_views, n_prompt) > launches
            case.m.pi0_tune("ppl=1")
        case.m.pi0_device_status(case.stream)
    finally:
        case.close()


# Half the full feed-forward: 513 .. 576 tokens have no use for gate||up's tiles of nine blocks of rows and are the fourth variant's
@pytest.mark.gpu
def test_a_narrower_feed_forward_beyond_512_tokens():
    case = Case(dataclasses.replace(CFG, llm_mlp=8192, max_prompt=64))
    try:
        for n_prompt in (1, 21, 32, 64):
            say(f"[gpu] prefix loop, llm_mlp 8192, {512 + n_prompt} tokens")
            img, st, nz, ids = case.inputs(2, n_prompt)
            want = case.by_launches(img, st, nz, ids)
            for _ in range(2):
                np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
            launches = case.m.pi0_kernel_count(2, n_prompt)
            case.m.pi0_tune("ppl=0")
            assert case.m.pi0_kernel_count(2, n_prompt) > launches
            case.m.pi0_tune("ppl=1")
        case.m.pi0_device_status(case.stream)
    finally:
        case.close()


@pytest.mark.parametrize("variant", range(6))
def test_prefix_loop_spills_no_registers(variant):
    binding.lib()
    with open(build.LIB, "rb") as f:
        library = f.read()
    found = {k: v for code in code_objects(library) for k, v in symbols(code).items() if f"prefix_loop_kernelILi{variant}EE" in k}
    (name, _), = [(k, v) for k, v in found.items() if "." not in k]
    assert found[name + ".private_seg_size"][0] == 0, "registers spilled"


OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
@pytest.mark.parametrize("variant", range(6))
def test_row_statistics_of_down_are_read_past_the_caches(variant, tmp_path):
    """An item of the reduction behind down leaves 64 bytes of a plane of row statistics, half a cache line, and the other half comes from
    another die.  A cached load of such a line could find the half that the reading die wrote and an older other one, which no parity
    test would show reliably: the QKV projection's eight loads of them (one per plane) have device scope.  Read from the code as built
    here; everything else that is read past the caches there goes 16 bytes at a time."""
    binding.lib()
    with open(build.LIB, "rb") as f:
        library = f.read()
    code, = [c for c in code_objects(library) if any(f"prefix_loop_kernelILi{variant}EE" in k for k in symbols(c))]
    at = tmp_path / "code.o"
    at.write_bytes(code)
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(at)], check=True, capture_output=True, text=True).stdout
    kernel, = [p for p in re.split(r"\n(?=[0-9a-f]+ <)", text) if f"prefix_loop_kernelILi{variant}EE" in p.split("\n", 1)[0]]
    assert len(re.findall(r"\bbuffer_load_dword(?:x2)? [^\n]*\bsc1\b", kernel)) == 8
