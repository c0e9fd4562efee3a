"""Every kernel that loads from memory straight into LDS does so in inline
assembly, inside which the compiler checks no hazards and of which it knows
only what the statement declares. This test disassembles the gfx950 code of
every fast-path unit (all kernels with a global_load_lds) and checks what makes
those statements sound:

* the statement sets m0, the load's LDS address, and lists it as clobbered, a
  register the compiler reserves for itself: m0 appears nowhere else, and no
  instruction reads it implicitly (indexed register moves, messages, GWS,
  append/consume, LDS-DMA buffer loads, interpolation);
* a load to LDS needs one wait state after a scalar write of m0: at least one
  instruction stands between the two, in one run of code that no branch leaves
  or enters and no other load shares;
* the masked form also writes exec, which it cannot declare, and leaves every
  lane enabled: nothing else in those kernels writes exec, so every lane is
  enabled wherever a load stands;
* a memory instruction needs five wait states after a vector instruction
  (v_readfirstlane, the reload of a spilled scalar) writes a scalar it reads."""
import os
import re
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"
TARGET = "hipv4-amdgcn-amd-amdhsa--gfx950"
IMPLICIT_M0 = re.compile(r"^\s*(v_movrel|s_movrel|s_sendmsg|ds_gws|ds_append|ds_consume|v_interp|"
                         r"s_set_gpr_idx|buffer_load_\w+.*\blds\b)")
# writes of exec: as the (first) destination, or by the forms that always write it
WRITES_EXEC = re.compile(r"^(\w+\s+exec(_lo|_hi)?\b|v_cmpx_|\w+_saveexec_|\w+_wrexec_)")


def _units():
    from paper_1909_10616_amd import build
    return [u[0] for u in build._units() if u[1] == "gemm_inst.hip" and "-DGT_CPR=0" not in u[2]]


@pytest.fixture(scope="module")
def objects():
    from paper_1909_10616_amd import build
    paths = {u: os.path.join(build.BUILD, u + ".o") for u in _units()}
    if not all(os.path.exists(p) for p in paths.values()):
        build.build(incremental=True, verbose=False)
    return paths


def _kernels(obj, tmp_path):
    """Kernel → its instructions and which of them branches reach, of every
    kernel that loads into LDS."""
    fb, co = tmp_path / "fatbin", tmp_path / "device.co"
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fb}", obj], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fb}",
                    f"--targets={TARGET}", f"--output={co}"], check=True)
    out, body, at, start = {}, [], {}, 0
    for line in subprocess.run([f"{LLVM}/llvm-objdump", "-d", str(co)], check=True,
                               capture_output=True, text=True).stdout.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\w+)>:$", line)
        if m:
            start, body, at, targets = int(m.group(1), 16), [], {}, set()
            out[m.group(2)] = body, at, targets
        elif line.startswith("\t") and "//" in line:   # (not the "..." of padding)
            ins, _, note = line.partition("//")
            addr = int(re.match(r"\s*([0-9A-F]+):", note).group(1), 16) - start
            at[addr] = len(body)
            body.append(ins.strip())
            if re.match(r"s_c?branch", body[-1]):
                targets.add(int(re.search(r"<\w+(?:\+0x([0-9a-f]+))?>", note).group(1) or "0", 16))
    return {k: (v, {at[t] for t in targets if t in at}) for k, (v, at, targets) in out.items()
            if any(i.startswith("global_load_lds") for i in v)}


def _scalars(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    if m:
        return {int(m.group(1))}
    return {"vcc_lo": {"vl"}, "vcc_hi": {"vh"}, "vcc": {"vl", "vh"}}.get(operand, set())


def _split(ins):
    op, _, rest = ins.partition(" ")
    return op, [a.strip() for a in rest.split(",")] if rest else []


def _check_base(before, load):
    """The last writer of each scalar the load reads is scalar, or at least
    five wait states back."""
    need = _scalars(_split(load)[1][1])
    states = 0
    for ins in reversed(before):
        if not need or states >= 5:
            return
        op, args = _split(ins)
        wrote = _scalars(args[0]) & need if args else set()
        assert not (wrote and op.startswith("v_")), f"{ins} … {load}"
        need -= wrote
        states += int(args[0], 0) + 1 if op == "s_nop" else 1


@pytest.mark.parametrize("unit", _units())
def test_loads_into_lds_are_sound(objects, unit, tmp_path):
    kernels = _kernels(objects[unit], tmp_path)
    loads = 0
    for fn, (ins, targets) in kernels.items():
        assert targets, fn
        inside = set()   # instructions of the statements that write m0 or exec
        for at, i in enumerate(ins):
            where = f"{unit} {fn}: {ins[max(at - 12, 0):at + 2]}"
            assert not IMPLICIT_M0.match(i), where
            if not i.startswith("global_load_lds"):
                continue
            loads += 1
            assert i.startswith("global_load_lds_dwordx4 "), where
            m0 = next(a for a in range(at - 1, -1, -1) if re.search(r"\bm0\b", ins[a]))
            assert ins[m0].startswith("s_mov_b32 m0,") and m0 not in inside and at - m0 >= 2, where
            assert not any(re.match(r"s_c?branch|s_setpc|s_swappc|global_load_lds", x)
                           for x in ins[m0:at]), where
            assert not targets & set(range(m0 + 1, at + 1)), where
            inside.add(m0)
            if "exec" in ins[at - 1].split(",")[0]:      # the masked form
                assert ins[at - 1] == "s_cselect_b64 exec, -1, 0", where
                assert ins[at - 2].startswith("s_cmp_gt_i32 "), where
                assert at - m0 == 3 and ins[at + 1] == "s_mov_b64 exec, -1", where
                inside |= {at - 1, at + 1}
            _check_base(ins[max(at - 8, 0):at], i)
        for at, i in enumerate(ins):
            if at not in inside:
                assert not re.search(r"\bm0\b", i) and not WRITES_EXEC.match(i), f"{unit} {fn}: {i}"
    # every instantiation of the unit: 28 (TM, TN) pairs with 16×16 MFMA, 15
    # with 32×32, and in bf16 the evenly shared kernel beside the general one
    pairs = 28 if "_16_c" in unit else 15
    assert len(kernels) == pairs * (2 if "_bf16_" in unit else 1) and loads > len(kernels)
