"""The prefill GEMMs load their operands into LDS ahead of use and wait for them by count: a wait for at most n loads in flight
stands for a certain slab only as long as the loads behind that slab's are really issued.  Loads into registers are ordinary
loads to the compiler, which may move them behind the wait or leave out those that nothing reads.  Checked here, on the CPU, from
the built code: along every path, each wave's share of slab b has landed when it reaches barrier b."""
import re

import pytest

from tests.test_device_code import _listing, built, parse  # noqa: F401 (built: the fixture)

LOOPS = 3                                                             # times a path goes back from one place


def events(code):
    """What a walk needs of a kernel: {first event of each kind at or behind an instruction}, as a list of nodes
    (kind, value, successors).  Kinds: load (True: into LDS), wait (loads that may stay in flight), barrier, and the end of the
    main loops, which is the first write into LDS by the waves themselves."""
    at = {ins[0]: i for i, ins in enumerate(code)}
    nodes = []
    for i, (_, op, _, ops, target, word) in enumerate(code):
        nxt = [] if op in ("s_endpgm", "s_branch") or i + 1 == len(code) else [i + 1]
        nxt += [at[target]] if target is not None else []
        if op.startswith(("buffer_load", "global_load", "flat_load", "scratch_load")):
            nodes.append(("load", "lds" in ops[-1].split(), nxt))
        elif op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            nodes.append(("load", False, nxt))                        # (stores and atomics count as well)
        elif op == "s_waitcnt":
            nodes.append(("wait", word & 15 | (word >> 14 & 3) << 4, nxt))
        elif op == "s_barrier":
            nodes.append(("barrier", None, nxt))
        elif op.startswith("ds_write") or op == "s_endpgm":
            nodes.append(("end", None, []))
        else:
            nodes.append((None, None, nxt))
    return nodes


def early_slabs(code, need):
    """Barriers b at which a path has loads of the first need(b) into LDS in flight, as (address, b, how many, path)."""
    nodes = events(code)
    useful = [kind == "barrier" for kind, _, _ in nodes]              # a barrier is still to come
    while True:
        more = [i for i in range(len(nodes)) if not useful[i] and any(useful[j] for j in nodes[i][2])]
        if not more:
            break
        for i in more:
            useful[i] = True
    found, ends = [], 0
    work = [(0, (), 0, 0, ())]                                        # where, in flight, loads into LDS, barriers, ways back
    while work:
        i, flying, issued, barriers, back = work.pop()
        flying = list(flying)
        while True:
            kind, value, nxt = nodes[i]
            if kind == "load":
                flying.append(issued if value else -1)
                issued += value
            elif kind == "wait":
                flying = flying[max(0, len(flying) - value):]         # they return in order
            elif kind == "barrier":
                late = sum(0 <= x < need(barriers) for x in flying)
                if late:
                    found.append((hex(code[i][0]), barriers, late, back))
                barriers += 1
            if kind == "end":
                ends += 1
                break
            nxt = [j for j in nxt if useful[j] or nodes[j][0] == "end" or not any(useful[k] for k in nxt)]
            if not nxt or not useful[i]:
                ends += 1
                break
            if len(nxt) == 1 and nxt[0] > i:
                i = nxt[0]
                continue
            for j in nxt:
                count = dict(back)
                if j <= i:
                    count[i] = count.get(i, 0) + 1
                    if count[i] > LOOPS:
                        continue
                work.append((j, tuple(flying), issued, barriers, tuple(sorted(count.items()))))
            break
    return found, ends


LDS, REG, BAR = ("buffer_load_dwordx4 v1, s[0:3], s5 offen lds", 0), ("buffer_load_dwordx4 v[4:7], v1, s[0:3], 0 offen", 0), ("s_barrier", 0)


def wait(n):
    return (f"s_waitcnt vmcnt({n})", 0xBF8C0F70 | n & 15 | (n >> 4) << 14)


@pytest.mark.parametrize("lines,late", [
    ([LDS, REG, REG, wait(2), BAR], 0),
    ([LDS, REG, wait(2), BAR, REG], 1),                               # a load that the count relies on, behind the barrier
    ([LDS, wait(0), BAR, LDS, REG, wait(1), BAR, LDS, REG, wait(2), BAR], 1),
    ([LDS, REG, wait(1), BAR, LDS, ("s_cbranch_scc0 1", 0xBF840001), REG, wait(1), BAR], 1),    # on one of two paths
])
def test_the_check_sees_a_wait_that_is_too_short(lines, late):
    text = _listing(lines + [("s_endpgm", 0xBF810000)]).replace("BF840001", "BF840001 <k+0x1c>")
    assert len(early_slabs(parse(text)["k"], lambda b: b + 1)[0]) == late


def arguments(name, kernel):
    """Numbers among a kernel's template arguments."""
    return [int(v) for v in re.findall(r"L[ib](\d+)E", name.split(kernel, 1)[1].split("EEvPK")[0] + "E")]


def test_few_row_products_wait_for_their_slabs(built):  # noqa: F811
    kernels = {n: code for n, code in built.items() if "gemm_few_kernelI" in n}
    assert len(kernels) == 14                                         # height, low terms
    for name, code in kernels.items():
        pieces = arguments(name, "gemm_few_kernel")[0]                # of a slab and wave
        found, paths = early_slabs(code, lambda b: (b + 1) * pieces)
        assert paths >= 4 and not found, (name, found[:3])


def test_tiled_products_wait_for_their_slabs(built):  # noqa: F811
    kernels = {n: code for n, code in built.items() if "gemm_f16_kernelI" in n}
    assert len(kernels) > 60
    for name, code in kernels.items():
        wgm, wgn, wm, wn = arguments(name, "gemm_f16_kernel")[:4]
        a, w = -(-wm // 8 // wgn), wn // 8 // wgm                     # pieces of a slab and wave; a third weight slab ahead is in
        # flight before the activations of the slab in front of it
        found, paths = early_slabs(code, lambda b: (b + 1) * (a + w))
        assert paths >= 2 and not found, (name, found[:3])
