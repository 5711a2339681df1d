"""The matrix instructions and LDS reads that are written as inline assembly (`mfma_in_place`, `read_frag_asm`) take over
waits that the compiler inserts for its own: it does not know how long a result stays in flight, and would be free to copy
or overwrite a register too early.  Checked here, on the CPU, from the sources and from the built library:

* in the LLVM IR the sum of an inline product goes nowhere but into the next one and into the wait (`settle`), so that
  every later use depends on the wait, and the first product takes its start from a wait as well;
* in the built code no instruction touches the result of a matrix instruction, or the destination of an LDS read, before
  it has arrived (along every path through a kernel), and no matrix instruction reads what a vector instruction wrote
  less than two issue slots before.
"""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2603_18464_amd import binding, build

LLVM = "/opt/rocm/llvm/bin/"

# ---- the IR ----------------------------------------------------------------------------------------------------


def accumulator(product):
    return re.search(r"(\S+)\)[^)]*$", product).group(1)


def ir_faults(ir):
    """Uses of a product still in flight, and products that do not start from a settled value."""
    faults = []
    for func in re.split(r"\n(?=define )", ir)[1:]:
        defs, users = {}, {}
        for line in func.splitlines():
            m = re.match(r"\s*(?:(%[\w.]+) = )?(.*)", line)
            name, rhs = m.group(1), m.group(2).split(", !")[0]
            if name:
                defs[name] = rhs
            for used in set(re.findall(r"%[\w.]+", rhs)):
                users.setdefault(used, []).append((name, rhs))
        flying = [n for n, rhs in defs.items() if 'asm sideeffect "v_mfma' in rhs]
        seen = set(flying)
        while flying:                                    # products, what merges them at a loop's head, tuples of them
            n = flying.pop()
            for name, rhs in users.get(n, []):
                if rhs.startswith(("phi", "shufflevector")):
                    if name not in seen:
                        seen.add(name)
                        flying.append(name)
                elif not ('asm sideeffect "v_mfma' in rhs and accumulator(rhs) == n) and 'asm sideeffect "s_nop 15' not in rhs:
                    faults.append(f"{n} used by {rhs[:90]}")

        def settled(v, path=()):
            rhs = defs.get(v, "")
            if v in path or 'asm sideeffect "v_mfma' in rhs or 'asm sideeffect "s_nop 15' in rhs:
                return True
            if rhs.startswith("extractvalue"):
                return settled(re.findall(r"%[\w.]+", rhs)[-1], path + (v,))
            if rhs.startswith("shufflevector"):
                return all(settled(x, path + (v,)) for x in re.findall(r"%[\w.]+", rhs))
            if rhs.startswith("phi"):
                return all(settled(x, path + (v,)) for x in re.findall(r"\[ (\S+),", rhs))
            return False
        for n, rhs in defs.items():
            if 'asm sideeffect "v_mfma' in rhs:
                if not settled(accumulator(rhs)):
                    faults.append(f"{n} starts from {accumulator(rhs)}")
    return faults


@pytest.mark.parametrize("source", ["decode_gemm.hip", "gemm_f16.hip"])
def test_products_in_flight_only_reach_the_wait(source, tmp_path):
    out = str(tmp_path / "device.ll")
    subprocess.run(["/opt/rocm/bin/hipcc", *build.FLAGS, "--cuda-device-only", "-S", "-emit-llvm",
                    os.path.join(build.CSRC, source), "-o", out], check=True, capture_output=True)
    ir = open(out).read()
    assert ir.count('asm sideeffect "v_mfma') > 100
    assert not ir_faults(ir)[:5]


# ---- the built code --------------------------------------------------------------------------------------------
# Issue slots before anything but a product into the same sum may touch a result: passes + 4 (gfx950), + 2 without XDL.
SLOTS = {"v_mfma_f32_16x16x32_f16": 8, "v_mfma_f32_32x32x16_f16": 12, "v_mfma_f32_16x16x128_f8f6f4": 12,
         "v_mfma_f32_16x16x4_f32": 10}


def _regs(text):
    r = set()
    for kind, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", text):
        r.update((kind, i) for i in range(int(lo), int(hi) + 1))
    r.update((kind, int(i)) for kind, i in re.findall(r"\b([va])(\d+)\b", text))
    return frozenset(r)


def parse(listing):
    """{kernel: [(address, mnemonic, operand register sets, operand texts, branch target, encoded word)]}"""
    funcs, cur = {}, None
    for line in listing.splitlines():
        m = re.match(r"([0-9a-f]+) <(.*)>:", line)
        if m:
            start, cur = int(m.group(1), 16), funcs.setdefault(m.group(2), [])
            continue
        m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+): ([0-9A-F]+)(.*)", line)
        if m and cur is not None:
            ops = [o.strip() for o in re.split(r",(?![^\[]*\])", m.group(2))]
            t = re.search(r"<.*?(?:\+0x([0-9a-f]+))?>", m.group(5)) if m.group(1).startswith(("s_cbranch", "s_branch")) else None
            cur.append((int(m.group(3), 16), m.group(1), [_regs(o) for o in ops], ops,
                        start + int(t.group(1) or "0", 16) if t else None, int(m.group(4), 16)))
    return funcs


def run_block(code, i, state, heads, faults):
    """From instruction i to the end of its block.  A state says what may be in flight, over all paths here:
    flying {destination of a product: issue slots to go}, written {registers of a vector instruction: slots to go},
    lds {register an LDS read will write: LDS operations issued since}."""
    flying, written, lds = map(dict, state)
    while True:
        addr, op, regs, _, target, word = code[i]
        touched = frozenset().union(*regs)
        mfma = op.startswith("v_mfma")
        if not lds.keys().isdisjoint(touched):
            faults.add(f"{addr:x} {op} touches an LDS read in flight")
        for dst, left in flying.items():
            if mfma:
                if not dst.isdisjoint(regs[1] | regs[2]) or (regs[3] != dst and not dst.isdisjoint(regs[3]) and left > 1):
                    faults.add(f"{addr:x} {op} reads a product in flight")
            elif not dst.isdisjoint(touched):
                faults.add(f"{addr:x} {op} touches a product in flight")
        if mfma and any(not w.isdisjoint(regs[1] | regs[2] | regs[3]) for w in written):
            faults.add(f"{addr:x} {op} reads a register just written")
        slots = (word & 0xffff) + 1 if op == "s_nop" else 1
        flying = {d: n - slots for d, n in flying.items() if n > slots}
        written = {w: n - slots for w, n in written.items() if n > slots}
        if mfma:
            flying[regs[0]] = SLOTS[op.replace("_e64", "")]
        elif op.startswith("v_") and regs[0]:
            written[regs[0]] = 2
        elif op.startswith("ds_"):
            lds = {r: n + 1 for r, n in lds.items()}
            if op.startswith("ds_read"):
                lds.update((r, 0) for r in regs[0])
        elif op == "s_waitcnt":                                       # LDS operations return in order; scalar loads count
            n = word >> 8 & 15                                        # too, which can only make the wait longer
            lds = {r: k for r, k in lds.items() if k < n}
        out = (flying, written, lds)
        if op in ("s_endpgm", "s_branch"):
            return ([target] if op == "s_branch" else []), out
        if target is not None:
            return [target, code[i + 1][0]], out
        i += 1
        if code[i][0] in heads:
            return [code[i][0]], out


def join(a, b):
    """What may be in flight where two paths meet."""
    def worst(x, y, pick):
        return {k: pick(x[k], y[k]) if k in x and k in y else x.get(k, y.get(k)) for k in x.keys() | y.keys()}
    return worst(a[0], b[0], max), worst(a[1], b[1], max), worst(a[2], b[2], min)


def kernel_faults(code):
    at, heads, faults = {ins[0]: i for i, ins in enumerate(code)}, {ins[4] for ins in code}, set()
    states, work = {code[0][0]: ({}, {}, {})}, [code[0][0]]
    while work:
        addr = work.pop()
        successors, out = run_block(code, at[addr], states[addr], heads, faults)
        for s in successors:
            new = join(states[s], out) if s in states else out
            if s not in states or new != states[s]:
                states[s] = new
                if s not in work:
                    work.append(s)
    return faults


def _listing(lines):
    return "0000000000000000 <k>:\n" + "".join(f"\t{text} // {4 * i:012X}: {word:08X}\n" for i, (text, word) in enumerate(lines))


P = ("v_mfma_f32_32x32x16_f16 v[0:15], v[16:19], v[20:23], v[0:15]", 0xD3D50000)
READ = ("ds_read_b128 v[16:19], v30 offset:64", 0xD9FE0040)


@pytest.mark.parametrize("lines,bad", [
    ([P, P], False),                                                              # a chain in place
    ([P, ("v_mov_b32_e32 v40, v3", 0x7E500303)], True),                           # a copy right behind a product
    ([P, ("s_nop 15", 0xBF80000F), ("v_mov_b32_e32 v40, v3", 0x7E500303)], False),
    ([P, ("s_nop 9", 0xBF800009), ("v_mov_b32_e32 v40, v3", 0x7E500303)], True),  # ten slots are not enough
    ([("v_mov_b32_e32 v16, v3", 0x7E200303), P], True),                           # an operand written just before
    ([("v_mov_b32_e32 v16, v3", 0x7E200303), ("s_nop 1", 0xBF800001), P], False),
    ([READ, P], True),                                                            # an operand that has not arrived
    ([READ, ("s_waitcnt lgkmcnt(0)", 0xBF8CC07F), P], False),
    ([READ, ("ds_read_b128 v[24:27], v30", 0xD9FE0000), ("s_waitcnt lgkmcnt(1)", 0xBF8CC17F), P], False),
    ([READ, ("s_load_dword s4, s[0:1], 0x0", 0xC0020100), ("s_waitcnt lgkmcnt(1)", 0xBF8CC17F), P], True),
    ([P, ("s_nop 15", 0xBF80000F), ("v_mov_b32_e32 v40, v3", 0x7E500303), P,      # the copy is early on the way back only
      ("s_cbranch_scc1 65532", 0xBF85FFFC)], True),
])
def test_the_check_sees_early_uses(lines, bad):
    text = _listing(lines + [("s_endpgm", 0xBF810000)])
    text = text.replace("BF85FFFC", "BF85FFFC <k+0x8>")
    assert bool(kernel_faults(parse(text)["k"])) == bad


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    """{kernel: instructions} of the built library."""
    lib = str(tmp_path_factory.mktemp("code") / "libvla.so")
    shutil.copy(binding.library_path(), lib)
    subprocess.run([LLVM + "llvm-objdump", "--offloading", lib], check=True, capture_output=True)
    kernels = {}
    for obj in glob.glob(lib + ".*gfx950*"):
        kernels.update(parse(subprocess.run([LLVM + "llvm-objdump", "-d", obj], check=True, capture_output=True,
                                            text=True).stdout))
    return kernels


def test_built_code_waits_for_its_products_and_reads(built):
    assert sum(ins[1].startswith("v_mfma") for code in built.values() for ins in code) > 4000
    faults = [f"{name}: {f}" for name, code in built.items() for f in sorted(kernel_faults(code))]
    assert not faults[:5], len(faults)


def test_float32_rows_that_are_not_aligned_are_loaded_16_bytes_at_a_time(built):
    """Unlike the rest of this file about time, not values: an odd d_ffn must not cost a load per element."""
    odd = {n: [ins[1] for ins in code] for n, code in built.items() if "gemm_f32_kernelILi" in n and "ELb0E" in n.split("gemm_f32_kernel")[1][:9]}
    assert odd
    for name, ops in odd.items():
        assert ops.count("global_load_dwordx4") >= 12, name


def test_decode_attention_requests_only_rows_that_exist(built):
    """About time as well: rows past the context, clamped to its last row, made steps of short contexts up to 35 % longer where
    they are read as data that does not come again.  Loads bounded by a descriptor make no request for them."""
    kernels = {n: [ins[1] for ins in code] for n, code in built.items() if "decode_attention_kernelI" in n}
    assert len(kernels) == 8                                          # head size, low terms, read once
    for name, ops in kernels.items():
        assert ops.count("buffer_load_dwordx4") >= 24, name
        assert not {"global_load_dwordx2", "global_load_dwordx4", "flat_load_dwordx2", "flat_load_dwordx4"} & set(ops), name


def test_the_ceiling_probe_runs_the_instruction_of_the_prefill_gemm(built):
    """A ceiling measured with another instruction is no ceiling: 32x32x16 sustains less than 16x16x32."""
    def products(name, part):
        return {ins[1] for n, code in built.items() if name in n and part in n for ins in code if ins[1].startswith("v_mfma")}
    assert products("probe_mfma_kernel", "") == products("gemm_f16_kernel", "EpiSwigluELb0ELb0E") == {"v_mfma_f32_16x16x32_f16"}
