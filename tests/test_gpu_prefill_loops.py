"""pi0_prefill runs the vision tower and the prefix's layers as the persistent kernels of pi0_infer, which go on with the blocks that are resident:
the cache that it leaves gives the bits of the launches (pvl=0, ppl=0) with every number of blocks that takes part, at tile edges of every
variant, and beside a kernel of another context that holds the chip."""
import ctypes
import dataclasses

import numpy as np
import pytest
import torch

from paper_2510_26742_amd import binding, synth
from tests.test_gpu_parity import Case, say

CFG = dataclasses.replace(synth.reduced_config(vocab=64), vis_layers=2, llm_layers=3, exp_layers=3, max_prompt=64)
SHAPES = [(1, 0), (1, 7), (1, 64), (2, 0), (2, 21), (2, 64), (3, 0)]   # a shape of every variant, and its last one where that is ragged


@pytest.mark.gpu
@pytest.mark.parametrize("graphs", [True, False])
def test_any_number_of_blocks_gives_the_launches_bits(graphs):
    case = Case(CFG)
    try:
        case.m.pi0_set_graph_mode(graphs)
        for n_views, n_prompt in SHAPES:
            img, st, nz, ids = case.inputs(n_views, n_prompt)
            want = case.by_launches(img, st, nz, ids)
            for blocks in (256, 255, 216, 97, 1):
                say(f"[gpu] prefill loops, {n_views} views + {n_prompt}, {blocks} blocks, graphs={graphs}")
                case.m.pi0_tune(f"pmb={blocks}")
                np.testing.assert_array_equal(case.prefill_and_denoise(img, st, nz, ids), want)
                assert np.isnan(case.prefill_and_denoise(np.full_like(img, np.nan), st, nz, ids)).all()
                np.testing.assert_array_equal(case.prefill_and_denoise(img, st, nz, ids), want)
                np.testing.assert_array_equal(case.infer(img, st, nz, ids), want)
        case.m.pi0_device_status(case.stream)   # raises if a bounded wait ran out
    finally:
        case.close()


@pytest.mark.gpu
def test_every_turn_of_a_loop_that_does_not_get_the_chip():
    """Turns are four layers, and the eighth is all that are left: 38 layers of the tower and six of the prefix by fewer blocks than the grid has.  In front
    of each turn the blocks that take part are others: those that were left out before come ahead of some that took part."""
    case = Case(dataclasses.replace(CFG, vis_layers=38, llm_layers=7, exp_layers=7))
    try:
        for n_views, n_prompt in SHAPES:
            img, st, nz, ids = case.inputs(n_views, n_prompt)
            want = case.by_launches(img, st, nz, ids)
            for blocks in (255, 200, 33, 256):
                say(f"[gpu] turns, {n_views} views + {n_prompt}, {blocks} blocks")
                case.m.pi0_tune(f"pmb={blocks}")
                for _ in range(3):
                    np.testing.assert_array_equal(case.prefill_and_denoise(img, st, nz, ids), want)
        case.m.pi0_device_status(case.stream)
    finally:
        case.close()


@pytest.mark.gpu
def test_prefill_beside_another_contexts_denoise():
    """Both contexts' kernels ask for the whole chip.  The denoise waits for all of its blocks, the prefill's loops for none that does not come."""
    a, b = Case(CFG), Case(CFG, seed=1)
    try:
        ia, ib = a.inputs(1, 0), b.inputs(2, 21)
        want_a, want_b = a.prefill_and_denoise(*ia), b.prefill_and_denoise(*ib)
        d_img, d_st, d_nz, d_ids = b.to_dev(*ib)
        _, a_st, a_nz, _ = a.to_dev(*ia)
        act_a = [torch.empty((CFG.chunk, CFG.action_dim), device=a.dev) for _ in range(6)]
        for i in range(6):
            say(f"[gpu] prefill beside a denoise, pass {i}")
            a.m.pi0_denoise(a_st, a_nz, act_a[i], a.stream)
            b.m.pi0_prefill(d_img, 2, d_ids, 21, b.stream)
        a.stream.synchronize()
        b.stream.synchronize()
        act_b = torch.empty((CFG.chunk, CFG.action_dim), device=b.dev)
        b.m.pi0_denoise(d_st, d_nz, act_b, b.stream)
        b.stream.synchronize()
        for act in act_a:
            np.testing.assert_array_equal(act.cpu().numpy(), want_a)
        np.testing.assert_array_equal(act_b.cpu().numpy(), want_b)
        a.m.pi0_device_status(a.stream)
        b.m.pi0_device_status(b.stream)
    finally:
        a.close()
        b.close()


@pytest.mark.gpu
def test_two_contexts_prefill_at_once():
    """Neither gets all of the chip at its start; the blocks of each join its turns as the other's end."""
    cases = [Case(dataclasses.replace(CFG, vis_layers=18), seed=i) for i in range(2)]
    try:
        inputs = [c.inputs(*shape) for c, shape in zip(cases, ((1, 7), (2, 21)))]
        want = [c.by_launches(*i) for c, i in zip(cases, inputs)]
        dev = [c.to_dev(*i) for c, i in zip(cases, inputs)]
        for i in range(8):
            say(f"[gpu] two prefills at once, pass {i}")
            torch.cuda.synchronize()
            for c, (img, st, nz, ids), views in list(zip(cases, dev, (1, 2)))[:: 1 if i % 2 else -1]:
                c.m.pi0_prefill(img, views, ids, ids.numel(), c.stream)
            torch.cuda.synchronize()
            for c, (_, st, nz, _), w in zip(cases, inputs, want):
                np.testing.assert_array_equal(c.denoise_only(st, nz), w)
        for c in cases:
            c.m.pi0_device_status(c.stream)
    finally:
        for c in cases:
            c.close()


@pytest.mark.gpu
def test_prefill_after_frames():
    """While the denoise of a two-stream frame may be on its way on the other stream, a plain prefill is launches; once it is done, the persistent kernels again."""
    case = Case(dataclasses.replace(CFG, vis_layers=9))
    try:
        img, st, nz, ids = case.inputs(1, 7)
        want = case.prefill_and_denoise(img, st, nz, ids)
        before = min(timed(case, 1, (img, st, nz, ids)) for _ in range(5))
        side = torch.cuda.Stream(device=case.dev)
        d_img, d_st, d_nz, d_ids = case.to_dev(img, st, nz, ids)
        act = [torch.empty((CFG.chunk, CFG.action_dim), device=case.dev) for _ in range(3)]
        for i in range(3):
            case.m.pi0_stream_frame(d_img, 1, d_ids, 7, d_st, d_nz, act[i], case.stream, side)
            case.m.pi0_prefill(d_img, 1, d_ids, 7, case.stream)
        case.stream.synchronize()
        side.synchronize()
        for a in act:
            np.testing.assert_array_equal(a.cpu().numpy(), want)
        np.testing.assert_array_equal(case.prefill_and_denoise(img, st, nz, ids), want)
        after = min(timed(case, 1, (img, st, nz, ids)) for _ in range(5))
        case.m.pi0_tune("pvl=0,ppl=0")
        launches = min(timed(case, 1, (img, st, nz, ids)) for _ in range(5))
        case.m.pi0_tune("pvl=1,ppl=1")
        say(f"[gpu] pi0_prefill before frames {before:.3f} ms, after them {after:.3f}, as launches {launches:.3f}")
        assert after - before < 0.5 * (launches - before)
    finally:
        case.close()


def timed(case, n_views, inputs, calls=1):
    """ms that `calls` pi0_prefill take, the first begun on an idle device."""
    d_img, _, _, d_ids = case.to_dev(*inputs)
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    begin.record(case.stream)
    for _ in range(calls):
        case.m.pi0_prefill(d_img, n_views, d_ids, len(inputs[3]), case.stream)
    end.record(case.stream)
    end.synchronize()
    return begin.elapsed_time(end)


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["global", "thread local", "relaxed"])
def test_prefill_after_frames_leaves_another_streams_capture_alone(mode):
    """Whether a frame's denoise is under way is asked of an event, and such a question ends a capture in global mode, whosever it is."""
    hip = ctypes.CDLL("libamdhip64.so")
    case = Case(CFG)
    try:
        img, st, nz, ids = case.inputs(1, 7)
        want = case.prefill_and_denoise(img, st, nz, ids)
        side, captured = (torch.cuda.Stream(device=case.dev) for _ in range(2))
        d_img, d_st, d_nz, d_ids = case.to_dev(img, st, nz, ids)
        act = torch.empty((CFG.chunk, CFG.action_dim), device=case.dev)
        for _ in range(2):   # (its launches become a graph here, one for each copy of the cache)
            case.m.pi0_stream_frame(d_img, 1, d_ids, 7, d_st, d_nz, act, case.stream, side)
            case.m.pi0_prefill(d_img, 1, d_ids, 7, case.stream)
        torch.cuda.synchronize()
        for under_way in (False, True):
            say(f"[gpu] prefill beside a capture in {mode} mode, frame under way: {under_way}")
            case.m.pi0_stream_frame(d_img, 1, d_ids, 7, d_st, d_nz, act, case.stream, side)
            if not under_way:
                torch.cuda.synchronize()
            graph = ctypes.c_void_p()
            assert hip.hipStreamBeginCapture(ctypes.c_void_p(captured.cuda_stream), ["global", "thread local", "relaxed"].index(mode)) == 0
            case.m.pi0_prefill(d_img, 1, d_ids, 7, case.stream)
            assert hip.hipStreamEndCapture(ctypes.c_void_p(captured.cuda_stream), ctypes.byref(graph)) == 0
            assert hip.hipGraphDestroy(graph) == 0
            torch.cuda.synchronize()
            np.testing.assert_array_equal(act.cpu().numpy(), want)
            np.testing.assert_array_equal(case.denoise_only(st, nz), want)
    finally:
        case.close()


@pytest.mark.gpu
def test_prefill_after_a_wait_that_ran_out_is_quick_and_reported():
    """One poll is not enough for all blocks to come.  The error word stays raised until the weights are loaded again, and the blocks of a
    later prefill that find it raised end: with the work of all blocks for each of them, nine layers took some hundred times as long."""
    case = Case(dataclasses.replace(CFG, vis_layers=9))
    try:
        inputs = case.inputs(2, 21)
        want = case.by_launches(*inputs)
        np.testing.assert_array_equal(case.prefill_and_denoise(*inputs), want)
        whole = min(timed(case, 2, inputs) for _ in range(3))
        case.m.pi0_tune("spl=1")
        say("[gpu] prefill whose waits end at once")
        timed(case, 2, inputs)
        with pytest.raises(binding.Pi0Error):
            case.m.pi0_device_status(case.stream)
        case.m.pi0_tune("spl=1048576")
        say("[gpu] prefill with the error word raised")
        late = min(timed(case, 2, inputs) for _ in range(3))
        say(f"[gpu] {whole:.2f} ms before, {late:.2f} ms with the error word raised")
        assert late < 4 * whole
        with pytest.raises(binding.Pi0Error):
            case.m.pi0_device_status(case.stream)
        d_blob = torch.from_numpy(case.blob.view(np.int16)).to(case.dev)
        torch.cuda.synchronize()
        case.m.pi0_load_weights(d_blob, case.stream)
        np.testing.assert_array_equal(case.prefill_and_denoise(*inputs), want)
        case.m.pi0_device_status(case.stream)
    finally:
        case.close()


@pytest.mark.gpu
def test_a_chip_that_is_busy_for_a_moment_costs_prefill_no_more_than_a_turn():
    """Another context's denoise holds 224 compute units when pi0_prefill's tower begins, for a quarter of the time that 27 layers take on the
    other 32: the blocks that come when it is done join in front of the next turn."""
    b = Case(dataclasses.replace(CFG, vis_layers=27), seed=1)
    a = Case(dataclasses.replace(CFG, steps=32), tune="psb=224")
    try:
        ia, ib = a.inputs(1, 0), b.inputs(2, 21)
        alone = min(timed(b, 2, ib) for _ in range(3))
        want_a, want_b = a.prefill_and_denoise(*ia), b.by_launches(*ib)
        d_img, d_st, d_nz, _ = a.to_dev(*ia)
        b_img, _, _, b_ids = b.to_dev(*ib)
        act = torch.empty((CFG.chunk, CFG.action_dim), device=a.dev)
        side = torch.cuda.Stream(device=a.dev)
        frame, beside = [], []
        for i in range(4):   # the first one only warms up
            say(f"[gpu] prefill beside a frame that holds most of the chip, pass {i}")
            begin, end, done = (torch.cuda.Event(enable_timing=True) for _ in range(3))
            torch.cuda.synchronize()
            a.m.pi0_stream_frame(d_img, 1, None, 0, d_st, d_nz, act, a.stream, side)
            begin.record(b.stream)
            b.m.pi0_prefill(b_img, 2, b_ids, 21, b.stream)
            end.record(b.stream)
            done.record(side)
            torch.cuda.synchronize()
            frame.append(max(0.0, begin.elapsed_time(done)))
            beside.append(begin.elapsed_time(end))
            np.testing.assert_array_equal(act.cpu().numpy(), want_a)
            np.testing.assert_array_equal(b.denoise_only(ib[1], ib[2]), want_b)
        say(f"[gpu] pi0_prefill alone {alone:.2f} ms, beside the frames " + ", ".join(f"{t:.2f} (frame done after {f:.2f})" for t, f in zip(beside, frame)))
        assert min(beside[1:]) < max(frame[1:]) + 2 * alone   # measured 1.3; with the blocks of the start throughout 3.2
        a.m.pi0_device_status(a.stream)
        b.m.pi0_device_status(b.stream)
    finally:
        a.close()
        b.close()
