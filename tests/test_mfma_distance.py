"""The kernels' own AMD assembly, checked on the CPU: distances that the hardware does not keep by itself.

A vector instruction that reads (or writes) a register too soon behind the MFMA that writes it gets the old contents.  The
compiler keeps the distance by filling in s_nop, counting wait states backwards from each use; where paths of different
length meet in one block on the way, it counts that block along one of them only, so the shorter path can come out short
(`SHARED_BLOCK` below is such a kernel: 11 wait states on one of its paths where straight code gets 12).  Which
source patterns are hit depends on the block order, so every kernel with MFMAs is walked along all its paths here.

The fragment reads from LDS are inline assembly whose results the compiler takes to be there at once: no path may touch
the registers of such a read before a wait that covers it."""
import functools
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2409_15241_amd import build as B

needs_compiler = pytest.mark.skipif(not shutil.which(B.hipcc()), reason="needs the ROCm compiler")
NEED = {"32x32x16": 12, "16x16x32": 8}          # wait states to the first use, as straight code gets them (checked below)

STRAIGHT = """
__global__ void straight32(const bf16x8* a, const bf16x8* b, float* o) {
  f32x16 c; for (int v = 0; v < 16; ++v) c[v] = 0;
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[threadIdx.x], b[threadIdx.x], c, 0, 0, 0);
  for (int v = 0; v < 16; ++v) o[threadIdx.x * 16 + v] = __builtin_amdgcn_exp2f(c[v]);
}
__global__ void straight16(const bf16x8* a, const bf16x8* b, float* o) {
  f32x4 c; for (int v = 0; v < 4; ++v) c[v] = 0;
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[threadIdx.x], b[threadIdx.x], c, 0, 0, 0);
  for (int v = 0; v < 4; ++v) o[threadIdx.x * 4 + v] = __builtin_amdgcn_exp2f(c[v]);
}
"""
# what the compiler (ROCm 7.2) makes of: product; if (m) { long; if (n) x; else y; } else if (n) z; use of the product
# (its scalar code cut down to the blocks and the distances that matter)
SHARED_BLOCK = """
_Z12shared_blockv:
\tv_mfma_f32_32x32x16_bf16 v[2:17], v[2:5], v[6:9], 0
\ts_cmp_eq_u32 s10, 0
\ts_cbranch_scc1 .L5
\ts_sleep 2
\ts_sleep 2
\ts_branch .L8
.L5:
\ts_cmp_eq_u32 s11, 0
\ts_cbranch_scc1 .L8
\ts_sleep 11
.L8:
\ts_nop 6
\tv_exp_f32_e32 v2, v2
\ts_endpgm
.Lfunc_end0:
"""
EARLY_READ = """
_Z10early_readv:
\tds_read_b128 v[0:3], v8
\tds_read_b128 v[4:7], v8 offset:2048
\ts_cbranch_scc1 .L1
\ts_waitcnt lgkmcnt(1)
.L1:
\tv_mov_b32_e32 v9, v3
\ts_waitcnt lgkmcnt(0)
\tv_mov_b32_e32 v10, v4
\ts_endpgm
.Lfunc_end0:
"""


def registers(text):
    out = set()
    for kind, one, lo, hi in re.findall(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])", text):
        out.update((kind, i) for i in (range(int(one), int(one) + 1) if one else range(int(lo), int(hi) + 1)))
    return frozenset(out)


class Kernel:
    """Instructions of one function: (opcode, operands, registers of each operand), and the successors of each."""

    def __init__(self, name, lines):
        self.name, self.code, labels = name, [], {}
        for line in lines:
            s = line.split(";")[0].strip()
            m = re.match(r"^([.\w$]+):$", s)
            if m:
                labels[m.group(1)] = len(self.code)
            elif s and not s.startswith("."):
                op, _, rest = s.partition("\t") if "\t" in s else s.partition(" ")
                operands = [x.strip() for x in re.split(r",(?![^\[]*\])", rest)] if rest.strip() else []
                self.code.append((op, operands, [registers(x) for x in operands]))
        self.next = []
        for i, (op, operands, _) in enumerate(self.code):
            assert not op.startswith(("s_setpc", "s_swappc", "s_call")), f"{name}: a call, whose paths are not followed"
            if op == "s_branch":
                self.next.append([labels[operands[0]]])
            elif op.startswith("s_cbranch"):
                self.next.append([i + 1, labels[operands[0]]])
            else:
                self.next.append([] if op == "s_endpgm" or i + 1 == len(self.code) else [i + 1])

    def walk(self, start, step):
        """Visits what can follow instruction `start`, each instruction once per smaller count: step(i, count) gives the
        count behind instruction i, or None where the walk ends."""
        seen, todo = {}, [(0, i) for i in self.next[start]]
        while todo:
            count, i = todo.pop()
            if seen.get(i, 1 << 30) <= count:
                continue
            seen[i] = count
            behind = step(i, count)
            if behind is not None:
                todo += [(behind, k) for k in self.next[i]]

    def touches(self, i, regs):
        op, _, rs = self.code[i]
        return op.startswith(("v_", "ds_", "buffer_", "global_", "flat_", "scratch_")) and any(r & regs for r in rs)

    def early_uses(self):
        """(MFMA, instruction, wait states between them) for every use of an MFMA's result that comes too soon."""
        found = []
        for i, (op, _, rs) in enumerate(self.code):
            if not op.startswith("v_mfma"):
                continue
            need = next(n for shape, n in NEED.items() if shape in op)
            dst = rs[0]

            def step(k, count):
                o, operands, r = self.code[k]
                if count >= need:
                    return None
                if o.startswith("v_mfma"):
                    # the next MFMA takes the sums of the one before without a gap; as a factor, or in part, they must be there
                    if (r[1] | r[2]) & dst or (len(r) > 3 and r[3] & dst and r[3] != dst):
                        found.append((i, k, count))
                elif o.startswith("v_") and self.touches(k, dst):
                    found.append((i, k, count))
                elif not o.startswith("ds_read") and self.touches(k, dst):      # a store; an LDS read arrives long after
                    found.append((i, k, count))
                return count + (int(operands[0], 0) + 1 if o == "s_nop" else 1)

            self.walk(i, step)
        return found

    def fresh_operands(self):
        """(vector instruction, MFMA, wait states between them) for every MFMA that reads a register less than two wait
        states behind the vector instruction that writes it: the compiler keeps them for its own MFMAs, not in inline assembly."""
        found = []
        for i, (op, _, rs) in enumerate(self.code):
            if not op.startswith("v_") or op.startswith(("v_mfma", "v_cmp")) or not rs:
                continue

            def step(k, count):
                o, operands, r = self.code[k]
                if count >= 2:
                    return None
                if o.startswith("v_mfma") and any(x & rs[0] for x in r[1:]):
                    found.append((i, k, count))
                return count + (int(operands[0], 0) + 1 if o == "s_nop" else 1)

            self.walk(i, step)
        return found

    def unwaited_reads(self):
        """(LDS read, instruction) for every instruction that touches a read's registers before a wait that covers it."""
        found = []
        for i, (op, _, rs) in enumerate(self.code):
            if not op.startswith("ds_read"):
                continue

            def step(k, later):                      # later: LDS operations behind the read (they complete in order)
                o, operands, _ = self.code[k]
                if o == "s_waitcnt":
                    m = re.search(r"lgkmcnt\((\d+)\)", " ".join(operands))
                    if m and int(m.group(1)) <= later:
                        return None
                if self.touches(k, rs[0]):
                    found.append((i, k))
                    return None
                return min(later + o.startswith("ds_"), 16)

            self.walk(i, step)
        return found


def kernels(text):
    name, lines = None, []
    for line in text.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            name, lines = m.group(1), []
        elif name and line.startswith(".Lfunc_end"):
            yield Kernel(name, lines)
            name = None
        elif name:
            lines.append(line)


def assembly(source, out):
    flags = [f for f in B.FLAGS if f != "-fPIC"]
    r = subprocess.run([B.hipcc(), *flags, "-S", "--cuda-device-only", source, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    with open(out) as f:
        return f.read()


@functools.lru_cache(maxsize=None)
def built(tmp):
    names = ("attention.hip", "gemm.hip")
    with ThreadPoolExecutor(2) as ex:
        texts = list(ex.map(lambda n: assembly(os.path.join(B.CSRC, n), os.path.join(tmp, n + ".s")), names))
    return {n: list(kernels(t)) for n, t in zip(names, texts)}


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    return built(str(tmp_path_factory.mktemp("asm")))


def test_the_walk_finds_planted_mistakes():
    (k,) = kernels(SHARED_BLOCK)
    assert [(k.code[b][0], n) for _, b, n in k.early_uses()] == [("v_exp_f32_e32", 11)]
    (k,) = kernels(SHARED_BLOCK.replace("s_nop 6", "s_nop 7"))
    assert not k.early_uses()
    (k,) = kernels(EARLY_READ)
    assert [k.code[b][1] for _, b in k.unwaited_reads()] == [["v9", "v3"]]


FRESH_OPERAND = """
_Z13fresh_operandv:
\tv_cvt_pk_bf16_f32 v3, v10, v11
\ts_nop 0
\tv_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[0:3], a[0:15]
\ts_endpgm
.Lfunc_end0:
"""


@needs_compiler
@pytest.mark.parametrize("source", ["attention.hip", "gemm.hip"])
def test_no_mfma_reads_an_operand_that_the_vector_alu_has_just_written(library, source):
    (k,) = kernels(FRESH_OPERAND)
    assert [n for _, _, n in k.fresh_operands()] == [1]
    (k,) = kernels(FRESH_OPERAND.replace("s_nop 0", "s_nop 1"))
    assert not k.fresh_operands()
    for k in library[source]:
        show = lambda i: " ".join([k.code[i][0], ", ".join(k.code[i][1])])
        assert not [(show(a), show(b), n) for a, b, n in k.fresh_operands()][:5], k.name


@needs_compiler
def test_straight_code_gets_the_distances_that_are_asked_for(tmp_path):
    src = tmp_path / "straight.hip"
    src.write_text('#include "' + os.path.join(B.CSRC, "common.h") + '"\n' + STRAIGHT)
    for k in kernels(assembly(str(src), str(tmp_path / "straight.s"))):
        (m,) = [i for i, c in enumerate(k.code) if c[0].startswith("v_mfma")]
        need = next(n for shape, n in NEED.items() if shape in k.code[m][0])
        assert k.code[m + 1][0] == "s_nop" and int(k.code[m + 1][1][0], 0) + 1 == need, k.name
        assert not k.early_uses()


@needs_compiler
@pytest.mark.parametrize("source,least", [("attention.hip", 12), ("gemm.hip", 48)])
def test_no_path_uses_a_product_or_a_fragment_too_early(library, source, least):
    with_products = [k for k in library[source] if any(c[0].startswith("v_mfma") for c in k.code)]
    assert len(with_products) >= least
    for k in with_products:
        show = lambda i: " ".join([k.code[i][0], ", ".join(k.code[i][1])])
        assert not [(show(a), show(b), n) for a, b, n in k.early_uses()][:5], k.name
        assert sum(c[0].startswith("ds_read") for c in k.code) > 8
        assert not [(show(a), show(b)) for a, b in k.unwaited_reads()][:5], k.name
