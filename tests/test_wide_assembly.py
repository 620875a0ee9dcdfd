"""Where the wide fitness kernels' accumulators lie (no GPU).  Their K loops multiply by
inline assembly, whose latency the compiler does not track: a move of an accumulator that
the register allocator puts between two steps would read it before the multiply has written
it, with nothing to show for it but wrong losses now and then.  The kernels are compiled to
assembly and each such move is looked up: between one of these multiplies and a later read
or write of an accumulator there are the 24 wait states of mfma_acc_sync, in both
directions."""
import os
import re
import subprocess

import pytest

from paper_2501_03944_amd import build

ACC_SYNC = 24                 # wait states of mfma_acc_sync


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: [(instruction, whether it is inline assembly)]}, labels as "label:"."""
    out = tmp_path_factory.mktemp("asm") / "fit_wide.s"
    cmd = [build.hipcc(), *build.FLAGS, "--cuda-device-only", "-S",
           os.path.join(build.CSRC, "fit_wide.hip"), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    found = {}
    for m in re.finditer(r"^(_ZN5mgfwa3fit\w*k_fit_wide\w*):.*?\n(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S):
        code, inline = [], False
        for line in m.group(2).split("\n"):
            s = line.strip()
            if s.startswith(";;#ASMSTART") or s.startswith(";#ASMSTART"):
                inline = True
            elif s.startswith(";;#ASMEND") or s.startswith(";#ASMEND"):
                inline = False
            elif re.match(r"\.LBB\w+:", s):
                code.append((s.split(":")[0] + ":", False))
            elif s and s[0] not in ".;":
                code.append((s.split(";")[0].strip(), inline))
        found[m.group(1)] = code
    return found


def _blocks(code):
    """Basic blocks {name: (instructions, successors)}, in the order of the text."""
    blocks = {"entry": []}
    name = "entry"
    for ins, inline in code:
        if ins.endswith(":"):
            name = ins[:-1]
            blocks[name] = []
        else:
            blocks[name].append((ins, inline))
            if re.match(r"s_c?branch", ins):
                name = f"behind {name} {len(blocks)}"
                blocks[name] = []
    out, order = {}, list(blocks)
    for i, name in enumerate(order):
        last = blocks[name][-1][0] if blocks[name] else ""
        nxt = re.findall(r"^s_c?branch\w*\s+(\.LBB\w+)", last)
        if i + 1 < len(order) and not re.match(r"s_branch|s_endpgm|s_setpc", last):
            nxt.append(order[i + 1])
        out[name] = (blocks[name], nxt)
    return out


def _waits(ins):
    m = re.match(r"s_nop\s+(\d+)", ins)
    return int(m.group(1)) + 1 if m else 1


def _walk(blocks):
    """{instruction: (wait states since the last inline multiply, and since the last
    accumulator write by another instruction)}, the least over all paths."""
    far = (ACC_SYNC, ACC_SYNC)
    entry = {name: None for name in blocks}
    entry["entry"] = far
    todo = ["entry"]
    seen = {}
    while todo:
        name = todo.pop()
        mul, write = entry[name]
        body, nxt = blocks[name]
        for k, (ins, inline) in enumerate(body):
            at = seen.get((name, k))
            seen[name, k] = (min(mul, at[0]), min(write, at[1])) if at else (mul, write)
            n = _waits(ins)
            mul, write = min(ACC_SYNC, mul + n), min(ACC_SYNC, write + n)
            if ins.startswith("v_mfma") and inline:
                mul = 0
            elif ins.startswith("v_accvgpr_write"):
                write = 0
        for t in nxt:
            old = entry[t]
            new = (mul, write) if old is None else (min(mul, old[0]), min(write, old[1]))
            if new != old:
                entry[t] = new
                todo.append(t)
    return seen


def test_accumulators_are_not_moved_between_the_multiplies(kernels):
    assert len(kernels) == 16, sorted(kernels)      # 4 families x 4 activations
    for name, code in kernels.items():
        blocks = _blocks(code)
        seen = _walk(blocks)
        multiplies = moves = 0
        for (block, k), (mul, write) in seen.items():
            ins, inline = blocks[block][0][k]
            if ins.startswith("v_mfma") and inline:
                multiplies += 1
                # (a tile's first multiplies take no accumulator in)
                if not ins.endswith(", 0"):
                    assert write >= ACC_SYNC, (name, block, k, ins)
            elif re.search(r"\ba\[?\d", ins):
                moves += 1
                assert mul >= ACC_SYNC, (name, block, k, ins)
        assert multiplies >= 128 and moves >= 32, (name, multiplies, moves)


def test_no_register_is_spilled_to_memory(kernels):
    for name, code in kernels.items():
        assert not [ins for ins, _ in code if ins.startswith("scratch_") or "buffer_store_dword" in ins], name
