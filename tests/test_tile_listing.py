"""Wait states around the MFMAs that the wide tile kernels write as asm statements.

The compiler does not know what such a statement is and keeps no distance from it.  A 16 x 16 x 32 bf16 MFMA takes four passes;
whatever but another MFMA reads or writes its result has to come 8 wait states (instructions, or what s_nop says) behind
it, and a vector instruction's result 2 in front of an MFMA that reads it.  (The compiler's own distances on this target: a store right
behind the builtin gets s_nop 7.)  The listing of every instantiation is walked in its textual order; a loop's last statement
waits itself, so that no distance runs over a back edge."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_06295_amd import build

RESULT, OPERAND = 8, 2
REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def registers(text):
    return [(m[1], r) for m in REG.finditer(text)
            for r in (range(int(m[2]), int(m[3]) + 1) if m[2] else [int(m[4])])]


def faults(lines):
    """(line, register, distance) of every access that comes too early."""
    found, now = [], 0
    result, vector = {}, {}  # register -> when an MFMA / a vector instruction wrote it
    for n, line in enumerate(lines):
        ins = line.split(";")[0].strip()
        if not ins or ins.endswith(":") or ins.startswith((".", "#")):
            continue
        op, _, args = ins.partition(" ")
        now += 1 + (int(args, 0) if op == "s_nop" else 0)
        args = [registers(a) for a in re.split(r",(?![^\[]*\])", args)]
        if op.startswith("v_mfma"):
            for r in (r for a in args[1:] for r in a):
                if now - vector.get(r, -99) <= OPERAND:
                    found.append((n, r, now - vector[r]))
            for r in args[0]:
                result[r] = now
                vector.pop(r, None)
            continue
        for r in (r for a in args for r in a):
            if now - result.get(r, -99) <= RESULT:
                found.append((n, r, now - result[r]))
        if op.startswith("v_") and not op.startswith("v_cmp"):
            for r in args[0]:
                vector[r] = now
    return found


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    out = tmp_path_factory.mktemp("listing") / "kernels_gemm.s"
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "kernels_gemm.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    found, name = {}, None
    for line in out.read_text().splitlines():
        m = re.match(r"(_Z\w*k_gemm_(?:wide|tall)\w*):", line)
        if m:
            name = m[1]
            found[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name:
            found[name].append(line)
    return found


def test_no_access_comes_too_early(kernels):
    assert len(kernels) > 20
    for name, lines in kernels.items():
        assert sum("v_mfma" in l for l in lines) >= 24, name
        assert faults(lines) == [], name


def test_the_walk_finds_a_move_between_the_mfmas(kernels):
    for name, lines in kernels.items():
        at = [i for i, l in enumerate(lines) if "v_mfma" in l]
        dst = registers(lines[at[-1]].split(",")[0])[0][1]
        src = registers(lines[at[0]].split(",")[1])[0][1]
        assert faults(lines[:at[-1] + 1] + [f"\tv_accvgpr_read_b32 v0, a{dst}"] + lines[at[-1] + 1:]), name
        assert faults(lines[:at[0]] + [f"\tv_mov_b32_e32 v{src}, 0"] + lines[at[0]:]), name
