"""What the built library's own gfx950 code must keep to where the compiler does not see an instruction (inline assembly)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2101_07706_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
WIDE_STORE = re.compile(r"(global|flat|scratch|buffer)_store_(dwordx[34]|b96|b128)$")
REG = re.compile(r"^([va])(?:(\d+)|\[(\d+):(\d+)\])$")


def _code_objects():
    """The gfx950 ELF images of the bundles inside the shared library."""
    with open(build.LIB, "rb") as f:
        blob = f.read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at, out = blob.find(magic), []
    while at >= 0:
        p = at + len(magic)
        n, = struct.unpack_from("<Q", blob, p)
        p += 8
        for _ in range(n):
            off, size, id_len = struct.unpack_from("<QQQ", blob, p)
            p += 24
            if b"gfx950" in blob[p:p + id_len] and size:
                out.append(blob[at + off:at + off + size])
            p += id_len
        at = blob.find(magic, at + 1)
    return out


def _regs(operand):
    m = REG.match(operand.strip())
    if not m:
        return set()
    lo = int(m.group(2) or m.group(3))
    return {(m.group(1), r) for r in range(lo, int(m.group(2) or m.group(4)) + 1)}


def _functions(obj_path):
    """(name, [(address, mnemonic, operands, branch target or None)]) of every function."""
    text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", obj_path], stdout=subprocess.PIPE, text=True, check=True).stdout
    name, ins = None, []
    for line in text.splitlines():
        head = re.match(r"^([0-9a-f]+) <(.*)>:$", line)
        if head:
            if ins:
                yield name, ins
            name, start, ins = head.group(2), int(head.group(1), 16), []
            continue
        body, _, tail = line.partition("//")
        f = body.split(None, 1)
        addr = re.match(r"\s*([0-9A-Fa-f]+):", tail)
        if not f or not addr:
            continue
        target = re.search(r"<.*\+0x([0-9a-f]+)>\s*$", tail)
        ins.append((int(addr.group(1), 16), f[0], f[1] if len(f) > 1 else "", start + int(target.group(1), 16) if target else None))
    if ins:
        yield name, ins


def _within_two_wait_states(ins, i, is_hit):
    """The first instruction less than two wait states after instruction i that is_hit(op, args), on any way through the code."""
    at = {a: k for k, (a, _, _, _) in enumerate(ins)}
    todo = [(i + 1, 0)]
    while todo:
        k, passed = todo.pop()
        if k >= len(ins) or passed >= 2:
            continue
        _, op, args, target = ins[k]
        if is_hit(op, args):
            return f"{op} {args.strip()}"
        if op == "s_endpgm":
            continue
        step = int(args.split()[0], 0) + 1 if op == "s_nop" else 1
        if op.startswith(("s_branch", "s_cbranch")) and target in at:
            todo.append((at[target], passed + step))
        if op != "s_branch":
            todo.append((k + 1, passed + step))
    return None


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    if not os.path.exists(build.LIB):
        build.build_library()
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    objects = _code_objects()
    assert len(objects) == len(build.SOURCES)
    out = []
    for j, obj in enumerate(objects):
        path = tmp_path_factory.mktemp("code") / f"{j}.elf"
        path.write_bytes(obj)
        out += list(_functions(str(path)))
    return out


# A store of more than 64 bits reads its data registers late: a vector instruction may write them two wait states after it
# at the earliest.  The compiler sees to that for its own stores, not for those written as inline assembly.
def test_wide_stores_keep_their_data(functions):
    n_stores, bad = 0, []
    for name, ins in functions:
        for i, (addr, op, args, _) in enumerate(ins):
            if not WIDE_STORE.match(op):
                continue
            n_stores += 1
            data = _regs(args.split(",")[0 if op.startswith("buffer") else 1])
            assert data, f"{name}: {op} {args}"
            hit = _within_two_wait_states(ins, i, lambda o, a: o.startswith("v_") and _regs(a.split(",")[0]) & data)
            if hit:
                bad.append(f"{name} {addr:#x}: {op} {args.strip()} -> {hit}")
    assert n_stores > 100
    assert not bad, f"{len(bad)} stores lose their data registers:\n" + "\n".join(bad[:20])


# VCC written by a vector instruction may be read by one two wait states later at the earliest (the carry of a 64-bit
# addition, a select); a register may be read through a lane exchange (DPP) that far behind its writing.
def test_carries_and_lane_exchanges_wait(functions):
    n_carries, bad = 0, []
    for name, ins in functions:
        for i, (addr, op, args, _) in enumerate(ins):
            if not op.startswith("v_") or op == "v_nop":
                continue
            dst = args.split(",")[:2]
            writes_vcc = "vcc" in [d.strip() for d in (dst if "_co_" in op or op.startswith("v_div_scale") else dst[:1])]
            n_carries += writes_vcc
            if not writes_vcc and not any("_dpp" in o for _, o, _, _ in ins[i + 1:i + 3]):
                continue
            regs = _regs(dst[0])

            def hit(o, a):
                if not o.startswith("v_"):
                    return False
                f = [x.strip() for x in a.split(",")]
                reads_vcc = any(re.match(r"vcc\b", x) for x in f[2 if "_co_" in o or o.startswith("v_div_scale") else 1:])
                return (writes_vcc and reads_vcc) or ("_dpp" in o and any(_regs(x.split()[0]) & regs for x in f[1:]))
            h = _within_two_wait_states(ins, i, hit)
            if h:
                bad.append(f"{name} {addr:#x}: {op} {args.strip()} -> {h}")
    assert n_carries > 100
    assert not bad, f"{len(bad)} reads too early:\n" + "\n".join(bad[:20])


# Aggregations with one or two features a lane and 32 or 64 lanes a row: the registers leave room for the blocks that the LDS
# holds (a block puts one wavefront on each of a compute unit's four units; 512 registers a lane in pieces of 8, 160 KB of LDS).
def test_narrow_aggregations_fill_the_lds(functions, tmp_path):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    seen = 0
    for j, obj in enumerate(_code_objects()):
        path = tmp_path / f"{j}.elf"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
        for kernel in re.split(r"\n  - \.", notes):
            name = re.search(r"\.name: +(\S+)", kernel)
            if not name or not re.search(r"11aggregate_kI[ft]Li[12]ELi(32|64)E", name.group(1)):
                continue
            lds, regs = (int(re.search(rf"\.{key}: +(\d+)", kernel).group(1)) for key in ("group_segment_fixed_size", "vgpr_count"))
            seen += 1
            assert 512 // (-(-regs // 8) * 8) >= (160 << 10) // lds, f"{name.group(1)}: {regs} registers, {lds} bytes of LDS"
    assert seen == 16


# Rows that start on any element: what the compiler is told of a piece's address is the alignment of an element and no more,
# in every load and store of a feature row (a typedef's own alignment, for one, is lost where it is a template argument).
ROW_PIECES = """
#include "aggregate_tile.hpp"
using namespace csgs;
template <typename T, int V>
__device__ inline void row(const T *x, float *out)
{
    const Vec<V> v = load_row<T, V>(x + threadIdx.x);
    for (int i = 0; i < V; ++i) out[i * 64 + threadIdx.x] = v.x[i];
}
#define ROW(T, V) extern "C" __global__ void row_##T##_##V(const T *x, float *out) { row<T, V>(x, out); }
ROW(float, 1) ROW(float, 2) ROW(float, 4) ROW(float, 8)
ROW(uint16_t, 1) ROW(uint16_t, 2) ROW(uint16_t, 4) ROW(uint16_t, 8)
extern "C" __global__ void piece_uint16_t(const char *x, char *out)
{
    store_global<u32x4, 2>(out + 2 * threadIdx.x, load_global<u32x4, 2>(x + 2 * threadIdx.x));
}
"""


def test_rows_claim_no_more_than_an_element(tmp_path):
    src = tmp_path / "pieces.hip"
    src.write_text(ROW_PIECES)
    ir = subprocess.run(["hipcc", "--offload-arch=gfx950", "--cuda-device-only", "-O3", "-std=c++17", "-S", "-emit-llvm", "-o", "-",
                         "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, str(src)], stdout=subprocess.PIPE, text=True, check=True).stdout
    seen = {}
    for name, body in re.findall(r"^define [^\n]*@((?:row|piece)_\w+)\([^\n]*\{\n(.*?)^\}", ir, re.M | re.S):
        element = 4 if "float" in name else 2
        loads = [(line.strip(), int(align)) for line, align in re.findall(r"(= load (?:<|i|float|half)[^\n]*addrspace\(1\)[^\n]*?align (\d+)[^\n]*)", body)]
        stores = [(line.strip(), int(align)) for line, align in re.findall(r"(store <[^\n]*addrspace\(1\)[^\n]*?align (\d+)[^\n]*)", body)]
        assert loads, name
        assert name[0] == "r" or stores, name
        for line, align in loads + stores:
            assert align <= element, f"{name}: {line}"
        seen[name] = len(loads)
    assert len(seen) == 9, seen


# The wide weight scan copies its sorted entries out of LDS two at a time, 16 bytes: the array says that it lies on such a piece, and does not
# leave that to where the compiler happens to put it.
def test_sorted_entries_are_aligned_for_their_copy():
    ir = subprocess.run(["hipcc", "--offload-arch=gfx950", "--cuda-device-only", "-O3", "-std=c++17", "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes", "-o", "-",
                         "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, os.path.join(build.CSRC, "probs.hip")],
                        stdout=subprocess.PIPE, text=True, check=True).stdout
    align = re.findall(r"^@_ZZN4csgs9scan_wideILb[01]E\w+E1u = [^\n]*addrspace\(3\)[^\n]*align (\d+)", ir, re.M)
    assert len(align) == 2 and min(map(int, align)) >= 16, align


# Four call sequences may be in flight on a device, and the one-pass adjacency launches a quarter of as many blocks as the source says a compute unit
# holds, which wait for each other: by its registers (512 a lane on each of four units, in pieces of 8) and its LDS (160 KB) a unit holds them.
def test_waiting_blocks_fit_together(tmp_path):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    with open(os.path.join(build.CSRC, "sample.hip")) as f:
        src = f.read()
    blocks = int(re.search(r"constexpr int ADJ_ONCE_BLOCKS = (\d+);", src).group(1))
    assert "blocks(resident_grid(ADJ_ONCE_BLOCKS) / CALL_SEQUENCES, 1)" in src
    seen = 0
    for j, obj in enumerate(_code_objects()):
        path = tmp_path / f"{j}.elf"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
        for kernel in re.split(r"\n  - \.", notes):
            name = re.search(r"\.name: +(\S+)", kernel)
            if not name or "8adj_once" not in name.group(1):
                continue
            lds, regs = (int(re.search(rf"\.{key}: +(\d+)", kernel).group(1)) for key in ("group_segment_fixed_size", "vgpr_count"))
            seen += 1
            assert 512 // (-(-regs // 8) * 8) >= blocks, f"{regs} registers"
            assert blocks * lds <= 160 << 10, f"{lds} bytes of LDS"
    assert seen == 1
