"""Wait states in the device code of the built library, read from its assembly (CPU only).

A vector instruction that writes a scalar register has to be 5 wait states ahead of a memory instruction that reads that
register.  The compiler sees to it for its own loads but does not look into inline assembly, from which the direct loads to
LDS are written."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2310_02409_amd", "libdodo.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
NEEDED = 5

_KERNEL = re.compile(r"^[0-9a-f]+ <(.+)>:$")
_LINE = re.compile(r"^\s+([a-z][a-z0-9_]+)\s*(.*?)\s*// ([0-9A-F]+):(?:[^<]*<.*\+0x([0-9a-f]+)>)?")
_SCALAR = re.compile(r"(?<![a-z0-9_])(?:s(\d+)|s\[(\d+):(\d+)\]|(vcc))(?![a-z0-9_])")
_CARRY = re.compile(r"_co_|v_mad_[iu]64_|v_div_scale_")  # a second result, in scalar registers
_MEMORY = ("buffer_", "global_", "flat_", "scratch_")


def _scalars(text):
    out = set()
    for one, lo, hi, vcc in _SCALAR.findall(text):
        out |= {"vcc"} if vcc else set(range(int(one or lo), int(one or hi) + 1))
    return out


def _parse(text):
    """[(kernel, [(name, operands, address, address of a branch's target or None)])] of a disassembly."""
    kernels, start = [], 0
    for line in text.splitlines():
        head = _KERNEL.match(line)
        if head:
            kernels.append((head.group(1), []))
            start = None
            continue
        m = _LINE.match(line)
        if m and kernels:
            address = int(m.group(3), 16)
            start = address if start is None else start
            kernels[-1][1].append((m.group(1), m.group(2), address, None if m.group(4) is None else start + int(m.group(4), 16)))
    return kernels


def _too_close(code):
    """Memory instructions of a kernel that may read a scalar register fewer than NEEDED wait states after a vector
    instruction has written it, on any way through its branches."""
    index = {address: i for i, (_, _, address, _) in enumerate(code)}
    before = [None] * len(code)  # per instruction: registers written lately -> least wait states since
    todo, found = [(0, {})], set()
    while todo:
        i, state = todo.pop()
        while i < len(code):
            known = before[i]
            if known is not None:
                merged = {r: min(known.get(r, NEEDED), state.get(r, NEEDED)) for r in known.keys() | state.keys()}
                if merged == known:
                    break
                state = merged
            before[i] = dict(state)
            name, operands, address, target = code[i]
            if name.startswith(_MEMORY):
                found |= {(address, name, operands, r) for r in _scalars(operands) if r in state}
            passed = int(operands, 0) + 1 if name == "s_nop" else 1
            state = {r: n + passed for r, n in state.items() if n + passed < NEEDED}
            if name.startswith("v_"):
                parts = re.split(r",\s*(?![^\[]*\])", operands)
                written = _scalars(parts[0]) | (_scalars(parts[1]) if _CARRY.search(name) and len(parts) > 1 else set())
                state.update({r: 0 for r in written})
            if target is not None and name.startswith("s_") and target in index:
                todo.append((index[target], dict(state)))
            if name in ("s_branch", "s_endpgm", "s_setpc_b64"):
                break
            i += 1
    return sorted(found, key=str)


def _asm(*lines):
    return "\n".join(["0000000000000000 <k>:"] + [f"\t{l:60s} // {4 * i:012X}: 00000000 {t}" for i, (l, t) in enumerate(lines)])


def test_the_reader_sees_what_is_too_close():
    def sites(*lines):
        (_, code), = _parse(_asm(*[l if isinstance(l, tuple) else (l, "") for l in lines]))
        return sorted({s[0] // 4 for s in _too_close(code)})
    first, load, end = "v_readfirstlane_b32 s17, v1", "buffer_load_dwordx4 v2, s[16:19], 0 offen lds", "s_endpgm"
    assert sites(first, "s_mov_b32 m0, s3", "s_nop 0", load, end) == [3]
    assert sites(first, "s_mov_b32 m0, s3", "s_nop 3", load, end) == []
    assert sites(first, "s_mov_b32 m0, s3", "s_nop 2", load, end) == [3]
    assert sites("v_readfirstlane_b32 s20, v1", load, end) == []
    assert sites("v_cmp_lt_u32_e64 s[18:19], v1, v2", load, end) == [1]
    assert sites("v_add_co_u32_e64 v3, s[16:17], v1, v2", "v_add_f32_e32 v1, v1, v2", load, end) == [2]
    assert sites("global_load_dwordx4 v[4:7], v2, s[16:17]", first, ("s_cbranch_scc1 65533", "<k+0x0>"), "s_nop 4", end) == [0]
    assert sites(first, ("s_cbranch_scc1 1", "<k+0xc>"), "s_nop 4", load, end) == [3]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_memory_instructions_wait_for_their_scalar_registers(tmp_path):
    copy = shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", copy], check=True, capture_output=True, cwd=tmp_path)
    images = sorted(p for p in tmp_path.iterdir() if p.name.endswith("gfx950"))
    assert images
    direct, bad = 0, []
    for image in images:
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", image], check=True, capture_output=True, text=True).stdout
        for kernel, code in _parse(text):
            direct += sum(1 for name, operands, _, _ in code if name.startswith("global_load_lds") or operands.endswith(" lds"))
            bad += [(kernel,) + site for site in _too_close(code)]
    assert direct > 100
    assert not bad, f"{len(bad)} sites, e.g. {bad[:5]}"
