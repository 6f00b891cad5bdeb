"""Distances between matrix instructions and the vector instructions that use their results, in the built library.

gfx950 does not wait for a result of the matrix unit: a vector, LDS or memory instruction that reads or overwrites it has to
come passes + 4 wait states after a product of 4 passes or more.  The compiler fills them in, but it looks for the
instruction only 19 back, one short of what a 16-pass product needs, so a use exactly 19 behind by itself gets nothing;
pv_step (csrc/sage_attn_core.h) keeps its results clear of that.  Every instruction counts one, s_nop k counts k + 1; s_waitcnt
counts too (measured on the card: 4.5 cycles where s_nop 0 takes 4.06).  No GPU: this reads the disassembly of the library's own kernels."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


def _passes(op, text):
    if op == "v_mfma_f32_32x32x64_f8f6f4":       # FP6 / FP4 operands (formats 2 to 4) on both sides: half the passes
        fmts = [int(m.group(1)) if (m := re.search(name + r":(\d)", text)) else 0 for name in ("cbsz", "blgp")]
        return 8 if min(fmts) >= 2 else 16
    return {"v_mfma_i32_32x32x32_i8": 8, "v_mfma_i32_16x16x64_i8": 4}.get(op)      # (the FP32 and FP64 forms need less)


def _regs(token):
    m = re.match(r"([va])(?:\[(\d+):(\d+)\]|(\d+))$", token.strip().split(" ")[0])
    if not m:
        return set()
    lo, hi = (m.group(2), m.group(3)) if m.group(2) else (m.group(4), m.group(4))
    return {(m.group(1), i) for i in range(int(lo), int(hi) + 1)}


def _functions(listing):
    """name -> [(opcode, operand list, text, index of the branch target or None)]"""
    out, name = {}, None
    for line in listing.split("\n"):
        m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if m:
            name = m.group(1)
            out[name] = []
        elif name and line.startswith("\t") and "//" in line:          # (not the "..." of skipped padding)
            text, _, rest = line.strip().partition("//")
            text = text.strip()
            op = text.split(" ")[0]
            addr = int(rest.strip().split(":")[0], 16)
            target = re.search(r"<[^>]*?(?:\+0x([0-9a-f]+))?>\s*$", rest) if op.startswith(("s_cbranch", "s_branch")) else None
            out[name].append((op, [t for t in text[len(op):].split(",")], text, addr, int(target.group(1) or "0", 16) if target else None))
    for name, ins in out.items():
        at = {a: i for i, (_, _, _, a, _) in enumerate(ins)}
        base = ins[0][3] if ins else 0
        out[name] = [(op, ops, text, at.get(base + t) if t is not None else None) for op, ops, text, _, t in ins]
    return out


def violations(ins):
    """(distance, needed, matrix instruction, its user) for every use of a result that comes too early on some path."""
    found = []
    for k, (op, ops, text, _) in enumerate(ins):
        p = _passes(op, text)
        if p is None:
            continue
        need = p + 4
        paths, seen = [(k + 1, 0, frozenset(_regs(ops[0])))], set()
        while paths:
            i, n, live = paths.pop()
            while i < len(ins) and n < need and live and (i, n, live) not in seen:
                seen.add((i, n, live))
                o, args, t, target = ins[i]
                if o == "s_nop":
                    n += int(t.split(" ")[1], 0) + 1
                    i += 1
                    continue
                if o.startswith("v_mfma"):       # the accumulator operand is forwarded; a product in its place ends the watch
                    if any(_regs(a) & live for a in args[1:3]):
                        found.append((n, need, text, t))
                        break
                    live = live - _regs(args[0])
                elif not o.startswith("s_") and any(_regs(a) & live for a in args):
                    found.append((n, need, text, t))
                    break
                n += 1
                if o == "s_endpgm":
                    break
                if target is not None:
                    if o.startswith("s_cbranch"):
                        paths.append((target, n, live))
                    else:
                        i = target
                        continue
                i += 1
    return found


def test_results_of_the_matrix_unit_are_left_alone_long_enough(tmp_path):
    import paper_2411_10958_amd as pa
    if not os.path.exists(pa.lib_path()) or not os.path.exists(OBJDUMP):
        pytest.skip("needs the built library and llvm-objdump")
    lib = shutil.copy(pa.lib_path(), tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    bad, products = [], 0
    for f in sorted(tmp_path.glob("lib.so.*gfx950")):
        listing = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(f)], check=True, capture_output=True, text=True).stdout
        for name, ins in _functions(listing).items():
            products += sum(_passes(op, text) == 16 for op, _, text, _ in ins)
            bad += [f"{name}: {n} of {need} wait states: {a} | {b}" for n, need, a, b in violations(ins)]
    assert products > 1000                       # (the listing was understood)
    assert not bad, "\n".join(bad[:20])


def _listing(own, user, jump=False):
    """A 16-pass product, `own` wait states, the user of its result."""
    lines = ["v_mfma_f32_32x32x64_f8f6f4 v[2:17], v[20:27], v[30:37], v[2:17]"]
    lines += ["v_add_f32_e32 v40, v41, v42"] * (own - 12 - jump) + ["s_nop 10", "s_waitcnt lgkmcnt(0)"]
    if jump:
        lines += ["s_branch 0", user, "s_endpgm", user, "s_endpgm"]
    else:
        lines += [user, "s_endpgm"]
    out = ["0000000000001000 <k>:"]
    for i, t in enumerate(lines):
        to = f" <k+0x{4 * (len(lines) - 2):x}>" if t.startswith("s_branch") else ""
        out.append(f"\t{t} // {0x1000 + 4 * i:012X}: 00000000{to}")
    return "\n".join(out)


@pytest.mark.parametrize("user", ["v_mov_b64_e32 v[50:51], v[16:17]", "global_store_dwordx4 v0, v[14:17], s[0:1]", "v_mul_f32_e32 v17, v40, v41",
                                  "ds_write_b32 v1, v9", "v_mfma_f32_32x32x64_f8f6f4 v[50:65], v[10:17], v[30:37], v[50:65]"])
def test_a_use_one_wait_state_early_is_found(user):
    for jump in (False, True):
        assert [v[:2] for v in violations(_functions(_listing(19, user, jump))["k"])] == [(19, 20)]
        assert not violations(_functions(_listing(20, user, jump))["k"])
    assert not violations(_functions(_listing(16, "v_mfma_f32_32x32x64_f8f6f4 v[2:17], v[20:27], v[30:37], v[2:17]"))["k"])
