"""What the built code has to show of three kernels.  The grouped GEMM's k-steps with two slots of weights wait for the copy of the
activations and leave the weights requested after it in flight: the loads between the two are exactly as many as the wait leaves
out.  The decode kernels request a rank step while another is on its way, and their copies to LDS have arrived at every barrier.  The
tiled gate's products follow each other without branches."""
import math
import os
import re
import struct
import subprocess

import paper_2512_17073_amd as amd
from paper_2512_17073_amd import build, binding

LLVM = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build._hipcc()))), "llvm", "bin")


def _functions(tmp_path, kernel):
    """(name, instructions) of the kernel's instantiations in the built library."""
    co = tmp_path / "kernel.co"
    co.write_bytes(_gfx950_code(tmp_path, kernel))
    text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", str(co)], capture_output=True, text=True, check=True).stdout
    for name, body in re.findall(r"^[0-9a-f]+ <(\S*%s\S*)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)" % kernel, text, re.S | re.M):
        yield name, [ln.split("//")[0].strip() for ln in body.splitlines()]


def _gfx950_code(tmp_path, kernel):
    amd.lib()                                             # (raises if the library is not built)
    fat = str(tmp_path / "fat")
    subprocess.run([os.path.join(LLVM, "llvm-objcopy"), "--dump-section", ".hip_fatbin=" + fat, binding.LIB_PATH, str(tmp_path / "copy")], check=True)
    data = open(fat, "rb").read()
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):       # one bundle per translation unit
        at = m.start() + 32
        for _ in range(struct.unpack_from("<Q", data, m.start() + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, at)
            code = data[m.start() + off:m.start() + off + size]
            if b"gfx950" in data[at + 24:at + 24 + n] and kernel.encode() in code:
                return code
            at += 24 + n
    raise AssertionError(f"no gfx950 code with {kernel} in the library")


def test_waits_leave_exactly_the_next_weights_in_flight(tmp_path):
    found = {}
    for name, lines in _functions(tmp_path, "qgemm_tile_kernel"):
        loads = None                                      # weight loads since the last copy to LDS (None: not known)
        for i, ln in enumerate(lines):
            wait = re.fullmatch(r"s_waitcnt vmcnt\((\d+)\)", ln)
            if re.match(r"buffer_load_.*\blds$", ln):
                loads = 0
            elif loads is not None and re.match(r"(buffer|global|flat|scratch)_", ln):
                loads += 1
            elif wait and int(wait[1]) > 0 and any(x.startswith("s_barrier") for x in lines[i + 1:i + 3]):
                assert loads == int(wait[1]), (name, ln, loads)
                found[name] = found.get(name, 0) + 1
    # 2, 3 and 4 bits; W1|W3, W2 in two and in four n-tiles; with and without 3-bit factor pairs
    assert len(found) == 18 and min(found.values()) >= 2, found


def _decode_functions(tmp_path):
    """(name, bits, dual, q3, instructions) of the 24 decode kernels."""
    found = list(_functions(tmp_path, "qgemm_decode_kernel"))
    assert len(found) == 24, [n for n, _ in found]
    for name, lines in found:
        bits, dual, q3, _ = re.search(r"qgemm_decode_kernelILi(\d)ELb(\d)ELb(\d)ELb(\d)", name).groups()
        yield name, int(bits), int(dual), int(q3), lines


def test_decode_kernels_refill_a_slot_while_the_other_rank_step_is_on_its_way(tmp_path):
    # Between two barriers (the k-steps have 16 products a row tile and more): a loop that multiplies a slot's step of two streams and
    # requests the next into it, for either slot, then the last turn's products.  A request anywhere else is one whose product
    # comes next, with nothing else in flight.
    for name, bits, dual, q3, lines in _decode_functions(tmp_path):
        events = ""
        for ln in lines:
            if ln.startswith("s_barrier"):
                events += "B"
            elif ln.startswith("buffer_load_dwordx4") and not ln.endswith("lds"):
                events += "L"
            elif ln.startswith("v_mfma_f32_16x16x32"):
                events += "P"
        parts = [part for part in events.split("B") if part.strip("L") and part.count("P") < 32]
        assert sorted(part.count("P") for part in parts) == [8, 16], (name, parts)         # one row tile, two
        assert all(part.count("L") == 4 and "LLL" not in part for part in parts), (name, parts)


def _blocks(tmp_path, kernel):
    """(name, basic blocks) of the kernel's instantiations: lists of instructions and of the blocks that can follow."""
    co = tmp_path / "kernel.co"
    co.write_bytes(_gfx950_code(tmp_path, kernel))
    text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", str(co)], capture_output=True, text=True, check=True).stdout
    for start, name, body in re.findall(r"^([0-9a-f]+) <(\S*%s\S*)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)" % kernel, text, re.S | re.M):
        code = [(int(at, 16), ln.strip(), target and int(start, 16) + int(target, 16))
                for ln, at, target in re.findall(r"^\s+(\S.*?)\s*// ([0-9A-F]+):[^<\n]*(?:<[^+\n]*\+0x([0-9a-f]+)>)?", body, re.M)]
        heads = {code[0][0]} | {t for _, _, t in code if t} | {code[i + 1][0] for i, c in enumerate(code[:-1]) if c[2] or c[1] == "s_endpgm"}
        blocks, at = {}, None
        for i, (addr, ln, target) in enumerate(code):
            if addr in heads:
                at = addr
                blocks[at] = ([], [])
            blocks[at][0].append(ln)
            if target:
                blocks[at][1].append(target)
            last = i + 1 == len(code)
            if not last and code[i + 1][0] in heads and not ln.startswith(("s_branch", "s_endpgm")):
                blocks[at][1].append(code[i + 1][0])
        yield name, blocks


def _copies_left_at_barriers(blocks):
    """Barriers that a path reaches with copies to LDS of its wavefront in flight.  Along a path: the least number of loads requested since the
    last copy that no wait was for (inf: none); a wait that leaves no more than these in flight was for the copy."""
    state, todo, left = {min(blocks): math.inf}, [min(blocks)], {}
    while todo:
        at = todo.pop()
        since = state[at]
        for i, ln in enumerate(blocks[at][0]):
            wait = re.match(r"s_waitcnt .*vmcnt\((\d+)\)", ln)
            if re.match(r"global_load_lds|buffer_load_.*\blds$", ln):
                since = 0
            elif re.match(r"(buffer|global|flat|scratch)_load", ln):
                since += 1
            elif wait and since >= int(wait[1]):
                since = math.inf
            elif ln.startswith("s_barrier") and since < math.inf:
                left[at, i] = since
        for to in blocks[at][1]:
            if to not in state or since < state[to]:
                state[to] = since
                todo.append(to)
    return left


def test_copies_of_the_decode_kernels_have_arrived_at_every_barrier(tmp_path):
    # A pass's first wait leaves the first turn of the ring in flight (two loads of either stream's slot, three at 3 and 4 bits) and
    # one load a row tile of the rows' exponents: neither fewer, nor so many that a copy is among them.
    found = 0
    for name, blocks in _blocks(tmp_path, "qgemm_decode_kernel"):
        bits = int(re.search(r"qgemm_decode_kernelILi(\d)", name)[1])
        waits = [(at, i, int(ln[len("s_waitcnt vmcnt("):].split(")")[0])) for at, (code, _) in blocks.items() for i, ln in enumerate(code[:-1])
                 if ln.startswith("s_waitcnt vmcnt(") and not ln.startswith("s_waitcnt vmcnt(0)") and code[i + 1].startswith("s_barrier")]
        ring = 8 if bits == 2 else 12
        assert sorted(n for _, _, n in waits) == [ring + 1, ring + 2], (name, waits)       # one row tile, two
        assert not _copies_left_at_barriers(blocks), (name, _copies_left_at_barriers(blocks))
        # and what it would look like otherwise: a wait that leaves one more load in flight
        for at, i, n in waits:
            code = list(blocks[at][0])
            code[i] = "s_waitcnt vmcnt(%d)" % (n + 1)
            assert _copies_left_at_barriers({**blocks, at: (code, blocks[at][1])}), (name, at, n)
        found += 1
    assert found == 24


def test_products_of_the_tiled_gate_between_branches(tmp_path):
    found = 0
    for name, lines in _functions(tmp_path, "gate_logits_kernel"):
        runs, run = [], 0                                 # matrix instructions between two branches
        for ln in lines:
            if ln.startswith("v_mfma"):
                run += 1
            elif ln.startswith(("s_cbranch", "s_branch")):
                runs.append(run)
                run = 0
        runs = [r for r in runs + [run] if r > 0]
        # one 16 x 16 tile: a batch of four 16-byte chunks; four tiles: a pair of values
        assert runs and min(runs) >= (32 if "ILi8ELi1EE" in name else 8), (name, runs)
        found += 1
    assert found == 2
