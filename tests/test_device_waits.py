"""The software wait states of the built device code.

gfx9-class processors leave some dependences between neighbouring instructions to software:
the compiler puts independent instructions or ``s_nop`` in between, but it neither looks into
inline asm nor knows what an asm block begins and ends with.  This reads the listing of every
kernel in the built library and holds each such pair to its distance, inside asm blocks and
across their edges (wait states are instructions in between; ``s_nop n`` counts n + 1):

* a scalar write of M0, then a load into LDS (which takes its address from M0): 1;
* a vector write of a VGPR, then an MFMA that reads it: 2 (3 behind a dot product);
* a vector write of an SGPR, then a memory instruction that reads it: 5;
* an MFMA, then anything but an accumulation on the same registers that touches its result:
  8 for the 16-bit 16x16x32, 10 for the fp32 16x16x4.

These are the distances that hipcc keeps between its own instructions on gfx950.
"""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
HORIZON = 20          # no rule reaches further

# wait states behind an MFMA until its result may be touched
MFMA_WAIT = {
    "v_mfma_f32_16x16x32_f16": 8, "v_mfma_f32_16x16x32_bf16": 8,
    "v_mfma_f32_16x16x4_f32": 10,
}
_REG = re.compile(r"(?<![\w.])([vas])(?:(\d+)|\[(\d+):(\d+)\])")
_SPECIAL = re.compile(r"(?<![\w.])(m0|vcc(?:_lo|_hi)?)(?!\w)")
_MEM = ("global_", "flat_", "buffer_", "scratch_")


def _regs(text):
    """The registers an operand list names, each by itself."""
    out = set()
    for kind, one, lo, hi in _REG.findall(text):
        out.update("%s%d" % (kind, n) for n in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    for name in _SPECIAL.findall(text):
        out.update(("vcc_lo", "vcc_hi") if name == "vcc" else (name,))
    return out


class _Instr:
    def __init__(self, line):
        code = line.split("//")[0].strip()
        self.text = code
        self.op, _, rest = code.partition(" ")
        ops = [x.strip() for x in re.split(r",(?![^\[]*\])", rest)] if rest else []
        op = self.op
        self.mfma = op.startswith("v_mfma") or op.startswith("v_smfma")
        self.valu = op.startswith("v_") and not self.mfma
        self.salu = op.startswith("s_")
        self.mem = op.startswith(_MEM)
        self.to_lds = (op.startswith("global_load_lds") or (op.startswith("buffer_load") and " lds" in code))
        self.wait = int(ops[0], 0) + 1 if op == "s_nop" else 1
        stores = self.mem and "load" not in op and "atomic" not in op or op.startswith("ds_write")
        n_dst = 0 if stores or self.to_lds or op.startswith("s_cmp") or op.startswith("s_bitcmp") else 1
        if "_swap" in op or "_co_" in op or op.startswith("v_div_scale"):
            n_dst = 2
        self.writes = _regs(",".join(ops[:n_dst]))
        self.reads = _regs(",".join(ops[n_dst:]))
        if "_swap" in op:
            self.reads |= self.writes
        if op.startswith("v_cmp") and op.endswith("_e32"):
            self.writes = {"vcc_lo", "vcc_hi"}
            self.reads = _regs(rest)
        if self.mfma:
            self.dst, self.src_c = ops[0], ops[3].split()[0]
            self.reads_ab = _regs(",".join(ops[1:3]))
        to = re.search(r"<[^>]*\+0x([0-9a-f]+)>", line) if op.startswith(("s_branch", "s_cbranch")) else None
        self.branch = int(to.group(1), 16) if to else 0 if re.search(r"<[^+>]+>$", line) and op.startswith(
            ("s_branch", "s_cbranch")) else None


def _step(pend, ins, found):
    """Holds `ins` to the pending waits and returns the waits pending behind it.  `pend` is a
    list of (rule, registers, wait states left, writer)."""
    for rule, regs, left, writer in pend:
        if rule == "m0":
            bad = ins.to_lds
        elif rule == "vgpr":
            bad = ins.mfma and ins.reads & regs
        elif rule == "sgpr":
            bad = ins.mem and ins.reads & regs
        else:
            touched = ins.reads | ins.writes
            if ins.mfma and ins.op == writer.op and ins.src_c == writer.dst:
                touched = ins.reads_ab      # the accumulator itself is forwarded; as an operand it is not
            bad = touched & regs
            # hipcc copies values that no path defines out of whatever register it likes; no kernel
            # takes a scalar from an accumulator
            bad = bad and ins.op != "v_readfirstlane_b32"
        if bad:
            found.append("%s: %s needs %d more wait states behind %s" % (rule, ins.text, left, writer.text))
    out = []
    for rule, regs, left, writer in pend:
        left -= ins.wait
        if ins.mfma or ins.valu:
            regs = regs - ins.writes if rule == "vgpr" else regs
        if left > 0 and (regs or rule == "m0"):
            out.append((rule, regs, left, writer))
    if ins.salu and "m0" in ins.writes:
        out.append(("m0", {"m0"}, 1, ins))
    if ins.valu:
        vec = {r for r in ins.writes if r[0] in "va" and r != "vcc_lo" and r != "vcc_hi"}
        if vec:
            out.append(("vgpr", vec, 3 if ins.op.startswith("v_dot") else 2, ins))
        if ins.writes - vec:
            out.append(("sgpr", ins.writes - vec, 5, ins))
    if ins.mfma:
        out.append(("mfma", ins.writes, MFMA_WAIT.get(ins.op, HORIZON), ins))
    return out


def scan(kernel):
    """The pairs of `kernel`, a list of (offset, _Instr), that are too close, on the straight
    line and behind each taken branch."""
    at = {off: i for i, (off, _) in enumerate(kernel)}
    found, pend = [], []
    for off, ins in kernel:
        pend = _step(pend, ins, found)
        if ins.branch is not None and pend and ins.branch in at:
            side, own = pend, {id(p[3]) for p in pend}
            for _, nxt in kernel[at[ins.branch]:at[ins.branch] + HORIZON]:
                side = [p for p in _step(side, nxt, found) if id(p[3]) in own]   # only what came along
                if not side:
                    break
        if ins.op in ("s_branch", "s_endpgm", "s_setpc_b64"):
            pend = []
    return found


def _parse(listing):
    kernels, name, base = {}, None, 0
    for line in listing.splitlines():
        head = re.match(r"([0-9a-f]{8,}) <([^>]+)>:$", line)
        if head:
            name, base = head.group(2), int(head.group(1), 16)
            kernels[name] = []
        elif name and line.startswith("\t") and "//" in line:
            off = int(line.split("//")[1].split(":")[0], 16) - base
            kernels[name].append((off, _Instr(line)))
    return kernels


def _listing(*lines):
    return [(8 * i, _Instr("\t" + s)) for i, s in enumerate(lines)]


@pytest.mark.parametrize("lines,n", [
    (("s_mov_b32 m0, s4", "global_load_lds_dwordx4 v1, s[2:3]"), 1),
    (("s_add_u32 m0, s4, 0x400", "s_nop 0", "global_load_lds_dwordx4 v1, s[2:3]"), 0),
    (("v_mov_b32_e32 v2, v9", "v_mfma_f32_16x16x32_f16 v[8:11], v[0:3], v[4:7], v[8:11]"), 1),
    (("v_mov_b32_e32 v2, v9", "ds_read_b128 v[12:15], v20", "s_nop 0",
      "v_mfma_f32_16x16x32_f16 v[8:11], v[0:3], v[4:7], v[8:11]"), 0),
    (("v_mfma_f32_16x16x32_f16 v[8:11], v[0:3], v[4:7], v[8:11]",
      "v_mfma_f32_16x16x32_f16 v[8:11], v[0:3], v[4:7], v[8:11]", "s_nop 7",
      "global_store_dwordx4 v12, v[8:11], s[2:3]"), 0),
    (("v_mfma_f32_16x16x32_f16 v[8:11], v[0:3], v[4:7], v[8:11]", "s_nop 6",
      "v_max_f32_e32 v1, v2, v9"), 1),
    (("v_mfma_f32_16x16x32_f16 v[8:11], v[0:3], v[4:7], v[8:11]",
      "v_mfma_f32_16x16x32_f16 v[16:19], v[8:11], v[4:7], v[16:19]"), 1),
    (("v_readfirstlane_b32 s2, v1", "s_nop 3", "global_load_dword v1, v2, s[2:3]"), 1),
    (("v_readfirstlane_b32 s2, v1", "s_nop 4", "global_load_dword v1, v2, s[2:3]"), 0),
])
def test_the_scan_finds_planted_pairs(lines, n):
    assert len(scan(_listing(*lines))) == n


def test_the_scan_follows_branches():
    head, tail = "\tv_mov_b32_e32 v12, v8", "\ts_cbranch_scc1 65533 // 000000000010: BF85FFFD <k>"
    near = [head, "\tv_mfma_f32_16x16x32_f16 v[8:11], v[0:3], v[4:7], v[8:11]", tail]
    far = [head, near[1], "\ts_nop 6", tail]
    for lines, n in ((near, 1), (far, 0)):
        assert len(scan([(8 * i, _Instr(s)) for i, s in enumerate(lines)])) == n


def test_built_kernels_keep_their_wait_states(tmp_path):
    from paper_2109_08008_amd import nt
    if not os.path.exists(nt.LIB_PATH):
        from paper_2109_08008_amd.build import build_library
        build_library()
    lib = shutil.copy(nt.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", os.path.basename(lib)], cwd=tmp_path, check=True, capture_output=True)
    images = sorted(f for f in os.listdir(tmp_path) if f.endswith("gfx950"))
    assert len(images) >= 7
    found, n_mfma, n_lds = {}, 0, 0
    for f in images:
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", f], cwd=tmp_path, check=True, capture_output=True,
                              text=True).stdout
        for name, kernel in _parse(text).items():
            n_mfma += sum(i.mfma for _, i in kernel)
            n_lds += sum(i.to_lds for _, i in kernel)
            assert {i.op for _, i in kernel if i.mfma} <= set(MFMA_WAIT), name
            bad = scan(kernel)
            if bad:
                found[name] = (len(bad), bad[:3])
    assert n_mfma > 1000 and n_lds > 1000     # the listing was read
    assert not found
