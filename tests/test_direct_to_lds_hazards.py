"""CPU check of the AMD assembly that hipcc makes of the kernels with direct-to-LDS
loads.  Those loads are inline asm, so the compiler's hazard recognizer does not see a
memory instruction and leaves out the wait states in front of it; the sources have to
provide them:
  * m0, the load's LDS address, is written by a scalar instruction: one wait state;
  * a scalar register that a vector instruction wrote (v_readfirstlane, v_readlane, v_cmp)
    and the load uses as base or through m0: five wait states.
An instruction is counted as one wait state, s_nop N as N + 1."""
import os
import re
import subprocess

import pytest

from paper_2606_15682_amd import build as libbuild

SOURCES = sorted(s for s in libbuild.SOURCES
                 if re.search(r"\bg2l(16|4)\(", open(os.path.join(libbuild.CSRC, s)).read()))


def _assembly(source, out):
    flags = [f for f in libbuild.HIPCC_FLAGS if f not in ("-shared", "-Wall")]
    subprocess.run([libbuild.hipcc(), *flags, "--cuda-device-only", "-S", os.path.join(libbuild.CSRC, source), "-o", out],
                   check=True, capture_output=True)
    with open(out) as f:
        return f.read()


def _sgprs(operand):
    """Numbers of the scalar registers an operand names ('m0' for that register)."""
    if operand == "m0":
        return {"m0"}
    m = re.fullmatch(r"s(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return set()
    lo, hi = (m[1], m[1]) if m[1] else (m[2], m[3])
    return set(range(int(lo), int(hi) + 1))


def hazards(text):
    """(direct-to-LDS loads, what is wrong with some of them)."""
    loads, bad, window = 0, [], []                        # window: (opcode, operands) so far, newest last
    for number, line in enumerate(text.splitlines(), 1):
        line = line.split(";")[0].strip()
        if re.fullmatch(r"_Z\w+:", line):
            window = []
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        op, _, rest = line.partition(" ") if " " in line else line.partition("\t")
        op, args = op.strip(), [a.strip() for a in re.split(r",(?![^\[]*\])", rest.strip())]
        if op.startswith("global_load_lds"):
            loads += 1
            base = _sgprs(args[1].split()[0]) if len(args) > 1 else set()
            if not base:
                bad.append("%d: no scalar base: %s" % (number, line))
            states, need = 0, base | {"m0"}
            for wop, wargs in reversed(window[-8:]):
                if wop == "s_nop":
                    states += int(wargs[0], 0) + 1
                    continue
                hit = bool(wargs) and _sgprs(wargs[0]) & need
                if hit and wop.startswith(("v_readfirstlane", "v_readlane", "v_cmp")) and states < 5:
                    bad.append("%d: %s, then %d wait states of 5: %s" % (number, wop, states, line))
                if hit and "m0" in hit and states < 1:
                    bad.append("%d: %s m0, then no wait state: %s" % (number, wop, line))
                states += 1
        window.append((op, args))
    return loads, bad


def test_the_check_itself():
    ok = "\ts_mov_b32 m0, s4\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v1, s[2:3]\n"
    assert hazards(ok) == (1, [])
    assert hazards(ok.replace("\ts_nop 0\n", "\tv_add_u32_e32 v2, v3, v4\n")) == (1, [])
    assert len(hazards(ok.replace("\ts_nop 0\n", ""))[1]) == 1
    assert len(hazards("\tv_readfirstlane_b32 s2, v9\n" + ok)[1]) == 1
    assert hazards("\tv_readfirstlane_b32 s2, v9\n\ts_nop 4\n" + ok)[1] == []
    assert len(hazards(ok.replace("s[2:3]", "v[2:3]"))[1]) == 1
    assert len(hazards("\tv_cmp_eq_u32_e64 s[2:3], v1, v2\n" + ok)[1]) == 1


def test_every_source_with_such_loads_is_listed():
    assert SOURCES == ["gemm_ksplit.hip", "gemm_tile256.hip", "gemm_w4a16_tile.hip"]


@pytest.mark.parametrize("source", SOURCES)
def test_wait_states(source, tmp_path):
    loads, bad = hazards(_assembly(source, str(tmp_path / "out.s")))
    assert loads > 0
    assert not bad, "%d of %d loads:\n%s" % (len(bad), loads, "\n".join(bad[:20]))
