"""CPU tests of the device code itself: the built library is disassembled and the waits that the
instruction set asks of the program, not of the hardware, are looked for on every path.

The compiler puts them in between its own instructions, but not around inline code: it sees neither
what that reads nor what it loads.  No GPU is involved."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_02599_amd import build as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# wait states between a matrix instruction of four passes and a vector or memory instruction that
# reads its result, and between a vector instruction that writes a scalar register and a memory
# instruction that takes its address from there
MFMA_WAIT = {"v_mfma_f32_16x16x32_bf16": 8}
SGPR_WAIT = 5
LINE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]+): (?:[0-9A-F]{8} ?)+(?:<(\S+)\+0x([0-9a-f]+)>)?")
REG = re.compile(r"\b([vas])(?:(\d+)|\[(\d+):(\d+)\])")


def _regs(text):
    out = set()
    for kind, one, lo, hi in REG.findall(text):
        out.update((kind, i) for i in (range(int(lo), int(hi) + 1) if lo else [int(one)]))
    return out


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    """[(name, [(mnemonic, [operands], index of the branch target or None)])] of every kernel."""
    if not os.path.exists(OBJDUMP) or not os.path.exists(B.LIB):
        pytest.skip("no disassembler, or the library is not built")
    d = tmp_path_factory.mktemp("image")
    lib = shutil.copy(B.LIB, d / "librap.so")
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=d, stdout=subprocess.DEVNULL, check=True)
    out = []
    for image in sorted(p for p in os.listdir(d) if p.endswith("gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(d / image)], stdout=subprocess.PIPE, text=True, check=True).stdout
        for part in re.split(r"^(?=[0-9a-f]{16} <)", text, flags=re.M)[1:]:
            head = re.match(r"([0-9a-f]{16}) <(.+)>:", part)
            start, code, at, jumps = int(head.group(1), 16), [], {}, []
            for line in part.splitlines()[1:]:
                m = LINE.match(line)
                if not m:
                    continue
                at[int(m.group(3), 16)] = len(code)
                to = None
                if m.group(1).startswith(("s_branch", "s_cbranch")):
                    assert m.group(4) == head.group(2) or m.group(5) is None, line
                    to = start + int(m.group(5) or "0", 16)
                    jumps.append(len(code))
                code.append([m.group(1), [x.strip() for x in m.group(2).split(",")], to])
            for i in jumps:
                code[i][2] = at[code[i][2]]
            out.append((head.group(2), code))
    assert sum(len(c) for _, c in out) > 100000
    return out


def _after(code, i, wait):
    """Instructions that can run fewer than `wait` wait states after instruction i, on any path."""
    todo, best = [(i + 1, 0)], {}
    while todo:
        j, d = todo.pop()
        while j < len(code) and d < wait and best.get(j, wait) > d:
            best[j] = d
            op, args, to = code[j]
            yield op, args
            d += int(args[0], 0) + 1 if op == "s_nop" else 1
            if op == "s_endpgm":
                break
            if to is not None:
                if op != "s_branch":
                    todo.append((j + 1, d))
                j = to
            else:
                j += 1


def _is_memory(op):
    return op.startswith(("global_", "buffer_", "flat_", "scratch_", "ds_"))


def _read(op, args):
    also_first = op.startswith(("v_fmac", "v_mac", "v_swap")) or "_swap" in op or "store" in op or "write" in op
    return _regs(",".join(args if also_first else args[1:]))


def test_matrix_results_are_not_read_too_early(functions):
    """Eight wait states from a matrix instruction to a vector or memory instruction that reads its
    result (matrix instructions themselves are interlocked or waited for by their own rule)."""
    n, bad = 0, []
    for name, code in functions:
        for i, (op, args, _) in enumerate(code):
            if not op.startswith(("v_mfma", "v_smfma")):
                continue
            n += 1
            dst = _regs(args[0])
            for op2, args2 in _after(code, i, MFMA_WAIT[op]):
                if (op2.startswith("v_") and not op2.startswith("v_mfma") or _is_memory(op2)) and _read(op2, args2) & dst:
                    bad.append("%s: %s %s ... %s %s" % (name, op, args[0], op2, ", ".join(args2)))
                    break
    assert n > 5000
    assert not bad, "%d of %d, first: %s" % (len(bad), n, bad[0])


def test_load_addresses_are_not_read_too_early(functions):
    """Five wait states from a vector instruction that writes a scalar register to a memory
    instruction that reads it; the hand-written load into LDS keeps them within itself, whatever the
    compiler puts in front of it."""
    bad, loads = [], 0
    for name, code in functions:
        for i, (op, args, _) in enumerate(code):
            if op.startswith(("v_readlane", "v_readfirstlane")):
                dst = _regs(args[0])
                bad += ["%s: %s %s ... %s %s" % (name, op, args[0], op2, args2) for op2, args2 in _after(code, i, SGPR_WAIT)
                        if _is_memory(op2) and _regs(",".join(args2)) & dst]
            if op == "global_load_lds_dwordx4":
                loads += 1
                before = code[i - 1]
                waits = int(before[1][0], 0) + 1 if before[0] == "s_nop" else 0
                if waits < SGPR_WAIT:
                    bad.append("%s: %d wait states of its own before %s %s" % (name, waits, op, args))
    assert loads > 100
    assert not bad, "%d, first: %s" % (len(bad), bad[0])


PROBE = r"""
#include "%s/rap_prefill_kernel.h"
namespace rap { namespace {
typedef __attribute__((address_space(1))) const void* gp;
typedef __attribute__((address_space(3))) void* lp;
__global__ void probe(const unsigned char* p, uint32_t slot, float* out) {
  __shared__ unsigned char area[4096];
  __builtin_amdgcn_global_load_lds((gp)p, (lp)area, 4, 0, 0);
  load_to_lds(p, 16 * threadIdx.x, slot);
  __builtin_amdgcn_global_load_lds((gp)(p + 64), (lp)area, 4, 0, 0);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  out[threadIdx.x] = area[threadIdx.x];
}
} }
void launch() { hipLaunchKernelGGL(rap::probe, dim3(1), dim3(64), 0, 0, nullptr, 0, nullptr); }
"""


def test_hand_written_load_declares_m0(tmp_path):
    """A load into LDS by the compiler's own form on either side of the hand-written one: m0 has to be
    set again for the second (compiled only, never run)."""
    if not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not available")
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE % B.CSRC)
    subprocess.run([B.hipcc(), *B.FLAGS, "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True,
                   stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=120)
    steps = re.findall(r"s_mov_b32 m0|global_load_lds_dword\w*", asm.read_text())
    assert steps == ["s_mov_b32 m0", "global_load_lds_dword", "s_mov_b32 m0", "global_load_lds_dwordx4",
                     "s_mov_b32 m0", "global_load_lds_dword"], steps


def _loops(code):
    """Sets of instructions that can reach each other: the loops of a function (iterative Tarjan)."""
    index, low, on, stack, out, n = {}, {}, set(), [], [], 0
    follow = [([to] if to is not None else []) + ([] if op in ("s_branch", "s_endpgm") or i + 1 == len(code) else [i + 1])
              for i, (op, _, to) in enumerate(code)]
    for root in range(len(code)):
        if root in index:
            continue
        work = [(root, iter(follow[root]))]
        index[root] = low[root] = n
        n += 1
        stack.append(root)
        on.add(root)
        while work:
            v, nexts = work[-1]
            for w in nexts:
                if w not in index:
                    index[w] = low[w] = n
                    n += 1
                    stack.append(w)
                    on.add(w)
                    work.append((w, iter(follow[w])))
                    break
                if w in on:
                    low[v] = min(low[v], index[w])
            else:
                work.pop()
                if work:
                    low[work[-1][0]] = min(low[work[-1][0]], low[v])
                if low[v] == index[v]:
                    part = set()
                    while True:
                        w = stack.pop()
                        on.discard(w)
                        part.add(w)
                        if w == v:
                            break
                    if len(part) > 1:
                        out.append(part)
    return out


def test_tile_in_flight_is_not_waited_for(functions):
    """Decode kernels for long ranges of dense caches: the loop over whole tiles has no wait for all loads between
    those of the next tile and the first matrix instruction, which works on the tile before it."""
    n, bad = 0, []
    for name, code in functions:
        form = re.search(r"decode_mfma_kernelILi(\d+)ELi(\d+)ELb\dELb(\d)ELb(\d)ELb\dELi(\d+)ELi(\d)E", name)
        if not form or form.group(3) == "1" or form.group(6) == "0":
            continue
        k, nt, q8, mx4 = (int(form.group(i)) for i in (1, 2, 4, 5))
        tile = 2 + (mx4 + 1) // 2 if mx4 else k + nt // 2 if q8 else 2 * k + nt
        for part in _loops(code):
            loads = [i for i in part if code[i][0] == "global_load_dwordx4" and code[i][1][-1].endswith(" nt")]
            # the loop over the last tiles has loads for parts of a tile beside those of a whole one
            if not 0 < len(loads) <= tile + 1 or not any(code[i][0].startswith("v_mfma") for i in part):
                continue
            n += 1
            todo, seen = [i + 1 for i in loads], set()
            while todo:
                j = todo.pop()
                while j in part and j not in seen:
                    seen.add(j)
                    op, args, to = code[j]
                    if op.startswith("v_mfma"):
                        break
                    if op == "s_waitcnt" and "vmcnt(0)" in ",".join(args):
                        bad.append("%s at %d" % (name, j))
                        break
                    if to is not None:
                        todo.append(to)
                    if op in ("s_branch", "s_endpgm"):
                        break
                    j += 1
    assert n > 150
    assert not bad, "%d, first: %s" % (len(bad), bad[0])


def _short_forms(functions):
    """(score steps, channel tiles, paired, paged) -> (code, its loop over tiles) of the bf16 decode kernels for short ranges."""
    out = {}
    for name, code in functions:
        form = re.search(r"decode_mfma_kernelILi(\d+)ELi(\d+)ELb(\d)ELb(\d)ELb0ELb\dELi0ELi0E", name)
        loops = [part for part in _loops(code) if any(code[i][0].startswith("v_mfma") for i in part)] if form else []
        if loops:
            assert len(loops) == 1, name
            out[tuple(int(x) for x in form.groups())] = code, loops[0]
    assert len(out) == 96
    return out


def test_short_ranges_spill_few_scalars(functions):
    """Scalars that did not fit are read back from vector registers 28 to 45 times in these kernels, and were 82 times where
    the order of the arguments made the compiler load them in other groups (1 x 24831 rows, d = 128, 33.0 -> 33.25 us)."""
    reads = {k: sum(op == "v_readlane_b32" for op, _, _ in code) for k, (code, _) in _short_forms(functions).items()}
    assert max(reads.values()) <= 50, {k: n for k, n in reads.items() if n > 50}


def test_short_ranges_of_pages_wait_no_more_than_dense_ones(functions):
    """The loop over tiles of a paged kernel has about as many waits as that of the dense one; it had up to 20 more where reads
    from LDS were waited for one by one (2 x 3780 rows, d = 106, 11.65 -> 11.9 us).  Three score steps with eight channel
    tiles spill, and wait for that too."""
    forms = _short_forms(functions)
    waits = {k: sum(code[i][0] == "s_waitcnt" for i in loop) for k, (code, loop) in forms.items()}
    over = {k: (n, waits[k[:3] + (0,)]) for k, n in waits.items() if k[3] and k[:2] != (3, 8) and n > waits[k[:3] + (0,)] + 6}
    assert not over, over
