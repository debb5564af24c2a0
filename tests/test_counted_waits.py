"""The kernels whose x slabs go from memory straight to LDS wait with counts: "at most N requests outstanding", where N requests were issued
behind the slab that is needed.  The slab requests are written in assembly, the weight requests among them are the compiler's, so
nothing in the source guarantees their number.  This test reads the assembly that the build produces and checks, along every
path to every such wait, that the last N requests before it hold no more slab requests than the slabs that may still be
under way: were a weight request dropped, merged or moved behind the wait, one of the needed slab's would be among them."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2510_11696_amd import build

VMEM = re.compile(r"\s+(global|buffer|scratch|flat)_\w+")
SLAB = re.compile(r"\s+global_load_lds_dwordx4")
WAIT = re.compile(r"\s+s_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)$")


def _panel(nt, kw, rt):
    xi, xb = nt * kw // 2, 4 if kw == 2 or nt <= 2 else 3 if nt == 3 else 2
    return {(xb - 2) * xi + (xb - 1) * 2 * rt: (xb - 2) * xi}


# kernel (mangled name) -> {N of the loop's wait: slab requests that may still be under way}
LOOPS = {f"panel_kernelILi{nt}ELi{kw}ELi{rt}ELb{direct}EE": _panel(nt, kw, rt)
         for direct in (0, 1) for nt, kw, rt in [(1, 4, 1), (2, 4, 1), (1, 4, 2), (2, 4, 2), (3, 4, 2), (4, 4, 2), (2, 2, 2), (3, 2, 2), (4, 2, 2)]}
LOOPS["prefill_kernelILi4ELi2ELi4EE"] = {4 + 8: 4}
LOOPS["mx_gemm_kernel"] = {4 + 8: 4}
SOURCES = ("linear_panel.hip", "linear_prefill.hip", "mx.hip")


def _blocks(lines):
    """Basic blocks of one function: (lines, indices of the blocks before it)."""
    blocks, names = [[]], {}
    for line in lines:
        if m := re.match(r"(\.?\w+):", line):
            if blocks[-1]:
                blocks.append([])
            names[m.group(1)] = len(blocks) - 1
        else:
            blocks[-1].append(line)
            if re.match(r"\s+(s_c?branch|s_endpgm)", line):
                blocks.append([])
    before, target = [set() for _ in blocks], {}
    for i, b in enumerate(blocks):
        ops = [x.split() for x in b if x.strip() and not x.strip().startswith((";", "."))]
        last = ops[-1] if ops else [""]
        if last[0].startswith(("s_branch", "s_cbranch")):
            target[i] = names[last[1]]
            before[target[i]].add(i)
        if last[0] not in ("s_branch", "s_endpgm") and i + 1 < len(blocks):
            before[i + 1].add(i)
    # The two arms of a request (inside K, across its end) come one behind the other: the first falls into a test of its own
    # flag that skips the second.
    slabs = [any(SLAB.match(x) for x in b) for b in blocks]
    for c in range(1, len(blocks) - 2):
        if target.get(c) == c + 2 and slabs[c - 1] and slabs[c + 1] and not any(VMEM.match(x) for x in blocks[c]) and c - 1 in before[c] and \
                any(re.match(r"\s+s_cbranch_vcc", x) for x in blocks[c]):
            before[c].discard(c - 1)
            before[c + 2].add(c - 1)
    return blocks, before


def _slabs_in_the_last(blocks, before, block, at, n):
    """The most slab requests among the last n requests before line `at` of `block`, over all paths."""
    most, seen, todo = 0, set(), [(block, at, n, 0)]
    while todo:
        b, end, left, slabs = todo.pop()
        for line in reversed(blocks[b][:end]):
            if left == 0:
                break
            if VMEM.match(line):
                left -= 1
                slabs += bool(SLAB.match(line))
        most = max(most, slabs)
        if left:
            for p in before[b]:
                if (p, left, slabs) not in seen:
                    seen.add((p, left, slabs))
                    todo.append((p, len(blocks[p]), left, slabs))
    return most


def _functions(text):
    found = {}
    for m in re.finditer(r"^(_ZN4qerl\w+):.*?^\.Lfunc_end", text, re.S | re.M):
        for name, loops in LOOPS.items():
            if name in m.group(1):
                found[name] = (m.group(0).split("\n")[1:-1], loops)
    return found


def _violations(lines, loops):
    """(waits of the loop found, those with a slab request too many behind the needed slab)"""
    blocks, before = _blocks(lines)
    waits, bad = 0, []
    for b, block in enumerate(blocks):
        for i, line in enumerate(block):
            m = WAIT.match(line)
            if m and int(m.group(1)) in loops and "s_barrier" in block[i + 1]:
                waits += 1
                n = int(m.group(1))
                if (got := _slabs_in_the_last(blocks, before, b, i, n)) > loops[n]:
                    bad.append((n, got, loops[n]))
    return waits, bad


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not found")
    out = tmp_path_factory.mktemp("asm")

    def assembly(src):
        s = str(out / (src + ".asm"))
        cmd = ["hipcc", *build.COMMON, *build.PER_FILE.get(src, []), "-S", "--cuda-device-only", os.path.join(build.CSRC, src), "-o", s]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return _functions(open(s).read())

    with ThreadPoolExecutor(max_workers=3) as ex:
        return {k: v for d in ex.map(assembly, SOURCES) for k, v in d.items()}


@pytest.mark.timeout(600)
def test_no_slab_is_read_before_it_has_arrived(functions):
    assert set(functions) == set(LOOPS)
    for name, (lines, loops) in functions.items():
        waits, bad = _violations(lines, loops)
        assert waits >= 2 and not bad, (name, waits, bad)


def test_missing_weight_requests_are_noticed(functions):
    for name, (lines, loops) in functions.items():
        load = [i for i, x in enumerate(lines) if VMEM.match(x) and not SLAB.match(x) and "load" in x and "scratch" not in x]
        ends = [i for i, x in enumerate(lines) if (m := WAIT.match(x)) and int(m.group(1)) in loops]
        # the loop's last weight request before a counted wait, taken out of the text; the MX kernel requests more than it counts
        drop = set(load) if name == "mx_gemm_kernel" else {max(i for i in load if i < ends[-1])}
        assert _violations([x for i, x in enumerate(lines) if i not in drop], loops)[1], name
