"""What the compiler made of the kernels, read from the library's own code object: properties that the kernels' speed
rests on, that no result shows, and that a change of source or compiler can silently lose."""
import re
import struct
import subprocess

import pytest

import paper_2602_01469_amd as pe
from paper_2602_01469_amd.binding import lib_path

LLVM = "/opt/rocm/llvm/bin/"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects inside the built library, one file each."""
    pe.load_library()
    data = open(lib_path(), "rb").read()
    out, at = [], data.find(BUNDLE)
    while at >= 0:
        pos = at + len(BUNDLE)
        (n,) = struct.unpack_from("<Q", data, pos)
        pos += 8
        for _ in range(n):
            off, size, name_len = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + name_len]
            pos += 24 + name_len
            if b"gfx950" in name and size:
                path = tmp_path_factory.mktemp("co") / f"{len(out)}.co"
                path.write_bytes(data[at + off:at + off + size])
                out.append(str(path))
        at = data.find(BUNDLE, at + 1)
    assert out
    return out


def _tool(name, *args):
    return subprocess.run([LLVM + name, *args], check=True, stdout=subprocess.PIPE, text=True).stdout


def _matrix_stretches(disassembly):
    """(kernel, instructions up to the last matrix instruction) of every stretch without a branch or barrier that holds at
    least 32 matrix instructions."""
    kernel, stretch = "", []
    for line in disassembly.splitlines() + ["<end>:"]:
        label = re.match(r"^[0-9a-f]* ?<(\S+)>:", line)
        if label or re.match(r"\s+s_(c?branch|barrier)", line):
            mfma = [i for i, s in enumerate(stretch) if s.startswith("v_mfma")]
            if len(mfma) >= 32:
                yield kernel, stretch[:mfma[-1]]
            stretch = []
            kernel = label.group(1) if label else kernel
        elif line.startswith("\t"):
            stretch.append(line.strip())


def test_full_row_tiles_of_dkdv_wait_for_no_load(code_objects):
    """The D = 64 dK/dV items, in their own kernel and in one grid with dQ, compute a row tile while the next one is copied to
    LDS: a stretch of matrix instructions that
    loads no register (the full row tiles, with the copies between their matrix instructions or issued before) must not wait
    for vector memory, which would be the next tile's copies."""
    riding, quiet = {}, {}
    for co in code_objects:
        for kernel, s in _matrix_stretches(_tool("llvm-objdump", "-d", "--no-show-raw-insn", co)):
            rows = re.search(r"(dkdv|bwd)_kernelILi64ELi(\d)ELb(\d)E", kernel)
            if not rows or any(re.match(r"(global|flat|scratch|buffer)_load(?!_lds)", x) for x in s):
                continue
            seen = riding if any("_load_lds" in x for x in s) else quiet
            seen[rows.groups()] = seen.get(rows.groups(), 0) + 1
            assert not any("vmcnt" in x for x in s), kernel
    # with and without the shared vector: an unmasked body that copies in every form but the dense far one (1), and a masked
    # one (far: also the unmasked one) that does not; listed ones (2, 4) mask by the start of a sequence as well
    forms = [(kernel, rows, sv) for kernel in ("dkdv", "bwd") for rows in "01234" for sv in "01"]
    assert riding == {f: 1 for f in forms if f[1] != "1"}
    assert quiet == {f: 1 if f[1] in "03" else 2 for f in forms}


def _tile_loops(disassembly):
    """(kernel, instructions) of every innermost loop that holds at least 16 matrix instructions."""
    kernel, start, code = "", 0, []
    for line in disassembly.splitlines() + ["0 <end>:"]:
        label = re.match(r"^([0-9a-f]+) <(\S+)>:", line)
        if label:
            back = set()
            for at, text, target in code:
                to = re.search(r"<\S+?\+0x([0-9a-f]+)>", target) if re.match(r"s_c?branch", text) else None
                if to and start + int(to.group(1), 16) <= at:
                    back.add((start + int(to.group(1), 16), at))
            inner = []
            for lo, hi in sorted(back, key=lambda r: r[1] - r[0]):
                body = [text for at, text, _ in code if lo <= at <= hi]
                if sum(x.startswith("v_mfma") for x in body) < 16 or any(lo <= a and b <= hi for a, b in inner):
                    continue
                inner.append((lo, hi))
                yield kernel, body
            start, kernel, code = int(label.group(1), 16), label.group(2), []
        else:
            m = re.match(r"\t(.*?)\s*// ([0-9A-F]+):?(.*)$", line)
            if m:
                code.append((int(m.group(2), 16), m.group(1), m.group(3)))


def test_no_loop_over_tiles_loads_a_parameter(code_objects):
    """Where one of two parameters is chosen, the compiler may choose between their addresses and load the result at each
    use.  A scalar load in the loop over tiles makes the wait for it a wait for every LDS read in flight."""
    seen = set()
    for co in code_objects:
        for kernel, body in _tile_loops(_tool("llvm-objdump", "-d", "--no-show-raw-insn", co)):
            seen.add(kernel)
            assert not [x for x in body if x.startswith("s_load")], kernel
    for name in ("fwd_kernel", "dq_kernel", "dq_pipe_kernel", "dkdv_kernel", "bwd_kernel", "draft_decode_kernel"):
        assert any(name in k for k in seen), name


def test_full_tiles_copy_no_bitmask(code_objects):
    """The forward and the pipelined dQ kernel run a list's full tiles in a loop that copies whole K / V tiles (16 bytes a
    lane; at least two tiles' or both forms' copies) and neither tests for nor copies a bitmask (4 bytes a lane)."""
    seen = {}
    for co in code_objects:
        for kernel, body in _tile_loops(_tool("llvm-objdump", "-d", "--no-show-raw-insn", co)):
            wide, narrow = (sum(x.startswith(f"global_load_lds_dword{w} ") for x in body) for w in ("x4", ""))
            if re.search("fwd_kernel|dq_pipe_kernel", kernel) and wide >= 16 and sum(x.startswith("v_mfma") for x in body) >= 32:
                seen[kernel] = seen.get(kernel, 0) + narrow
    assert len(seen) == 10 and not any(seen.values()), seen  # (nine forwards, one dQ)


def test_the_workgroups_that_a_launch_bound_means_fit_a_cu(code_objects):
    """256 threads are one wave for each of a CU's four SIMDs, so that n workgroups of them share 512 registers a lane and 160 KB of
    LDS.  The row-stationary kernels rest on the number that their launch bound names: short lists are covered by the other
    workgroups of the CU."""
    per_cu = {r"fwd_kernelILi64ELi\dELb\dELi(\d)E": None, r"fwd_kernelILi128ELi\dELb\dELi(\d)E": None, r"dq_kernelILi64E": 3,
              r"dq_kernelILi128E": 2, r"dq_pipe_kernelILi64E": 2, r"(?:dkdv|bwd)_kernelILi64E": 2}
    seen = set()
    for co in code_objects:
        notes = _tool("llvm-readobj", "--notes", co)
        for lds, name, vgprs in re.findall(r"\.group_segment_fixed_size:\s+(\d+).*?\.name:\s+(\S+).*?\.vgpr_count:\s+(\d+)", notes, re.S):
            for kernel, n in per_cu.items():
                m = re.search(kernel, name)
                if m:
                    n = n or int(m.group(1))
                    seen.add((kernel, n))
                    assert int(lds) * n <= 160 * 1024 and int(vgprs) * n <= 512, (name, lds, vgprs)
    assert {n for k, n in seen if k.startswith("fwd_kernelILi64")} == {2, 3, 4} and len({k for k, _ in seen}) == len(per_cu), seen


def test_no_kernel_spills(code_objects):
    """No kernel keeps registers in scratch memory: a reload inside a loop waits for the copies issued before it."""
    spilling, seen = {}, 0
    for co in code_objects:
        notes = _tool("llvm-readobj", "--notes", co)
        for name, size in re.findall(r"\.name:\s+(\S+).*?\.private_segment_fixed_size:\s+(\d+)", notes, re.S):
            seen += 1
            if int(size):
                spilling[name] = int(size)
    assert seen >= 30 and not spilling


def test_how_many_loads_the_sum_of_partials_has_on_their_way(code_objects):
    """16-byte loads between two waits: one head's (with rotary embedding two) in the form for long sums of one set of partials,
    four heads' (eight) in the others."""
    most = {}
    for co in code_objects:
        kernel, run = "", 0
        for line in _tool("llvm-objdump", "-d", "--no-show-raw-insn", co).splitlines():
            label = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
            if label:
                kernel, run = label.group(1), 0
            sets = re.search(r"reduce_partials_kernelILi(\d+)ELi(\d)ELi(\d)E", kernel)
            if not sets:
                continue
            run = 0 if "vmcnt" in line else run + ("global_load_dwordx4" in line)
            most[sets.groups()] = max(most.get(sets.groups(), 0), run)
    assert most == {(d, *form): loads for d in ("64", "128") for form, loads in ((("1", "1"), 2), (("1", "4"), 8), (("4", "4"), 8))}
