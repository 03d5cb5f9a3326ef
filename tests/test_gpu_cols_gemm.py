"""gate||up and down beyond 512 rows on tiles of seven and nine blocks of 32 rows, with a lower body for the rows that are left over
(gemm_cols_body): the token counts where the body or the number of tiles changes, a contraction of one turn of the loop, a last k range shorter than
the others, against the CPU oracle through the whole pass (all per-layer taps, which the launches leave).  That the persistent prefix gives the launches' bits is
test_gpu_prefix_loop's."""
import dataclasses
import os
import re
import subprocess

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


OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
WAIT_STATES = 20   # between a matrix product and another instruction that names the registers it writes, whatever its number of passes


def vector_registers(operands):
    return {r for a, b in re.findall(r"\bv\[(\d+):(\d+)\]", operands) for r in range(int(a), int(b) + 1)} | {int(r) for r in re.findall(r"\bv(\d+)\b", operands)}


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
@pytest.mark.parametrize("kernel", ["gemm_cols_kernelILi9ELi4EE", "prefix_loop_kernelILi5EE"])
def test_nothing_else_touches_the_ninth_block_behind_its_products(kernel, tmp_path):
    """The ninth block's products are assembly, behind which the compiler leaves no wait states: a copy or a spill of such an accumulator would find
    it unfinished, now and then.  In the code as built here, on every way on from such a product, only another product names its
    registers within the wait states that the hardware asks for (an instruction counts as one)."""
    binding.lib()
    with open(build.LIB, "rb") as f:
        library = f.read()
    code, = [c for c in code_objects(library) if any(kernel in k for k in symbols(c))]
    at = tmp_path / "code.o"
    at.write_bytes(code)
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(at)], check=True, capture_output=True, text=True).stdout
    body, = [p for p in re.split(r"\n(?=[0-9a-f]+ <)", text) if kernel in p.split("\n", 1)[0]]
    lines = re.findall(r"^\t(\S+)[ \t]*([^\n]*?)[ \t]*// ([0-9A-F]+):([^\n]*)$", body, re.M)
    start = int(lines[0][2], 16)
    index = {int(l[2], 16) - start: i for i, l in enumerate(lines)}
    assert len(lines) == len([l for l in body.strip().split("\n")[1:] if l.strip() != "..."])   # every line is understood (dots: zeros behind the end)

    def ways_on(i):
        op, _, _, rest = lines[i]
        out = [] if op in ("s_branch", "s_endpgm") else [i + 1]
        if "branch" in op:
            target = re.search(r"\+0x([0-9a-f]+)>", rest)
            out.append(index[int(target.group(1), 16) if target else 0])
        return out

    products = 0
    for i, (op, operands, _, _) in enumerate(lines):
        if not op.startswith("v_mfma") or not operands.startswith("v["):
            continue
        products += 1
        written = vector_registers(operands.split(",")[0])
        todo = [(j, 0) for j in ways_on(i)]
        while todo:
            j, states = todo.pop()
            if states >= WAIT_STATES:
                continue
            other, names, where, _ = lines[j]
            if vector_registers(names) & written:
                first, *_, last = [x.strip() for x in names.split(", ")]
                assert other.startswith("v_mfma") and vector_registers(first) == written == vector_registers(last), (lines[i], lines[j])
            todo += [(k, states + (int(names) + 1 if other == "s_nop" else 1)) for k in ways_on(j)]
    assert products == 64   # two bodies' worth: the loop's turn and the last one, 16 k steps x two feature tiles each
