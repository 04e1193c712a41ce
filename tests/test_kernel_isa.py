"""Static checks on the code hipcc generates for the persistent GEMM kernel (CPU only: cross-compilation).

The kernel names its accumulator registers itself (a[0:255], see csrc/gemm_common.h) instead of handing 64
values to the register allocator.  That is only sound if nothing else in the kernel touches an AGPR, if the
kernel really allocates all 256 of them, and if nothing is spilled to scratch memory; the copy statements
rely on M0 being written and consumed inside one asm statement; and the MFMA statements get no hazard
handling from the compiler.  All of that is a property of the generated
code, so it is checked on the generated code.
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_01193_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("isa") / "gemm_persistent.s")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "hip", "--cuda-device-only",
           "-S", os.path.join(CSRC, "gemm_persistent.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    text = open(out).read()
    # one entry per kernel: (name, instruction lines, trailer with the resource summary)
    parts = re.split(r"^(_ZN5lobra22gemm_persistent_kernel\w+):", text, flags=re.M)
    ks = []
    for i in range(1, len(parts), 2):
        body = parts[i + 1]
        end = body.index(".end_amdhsa_kernel")
        code = [l.split(";")[0].strip() for l in body[:body.rindex("s_endpgm", 0, end) + 8].split("\n")]
        code = [l for l in code if l and not l.startswith(".")]
        tail = body[end:end + 3000]
        ks.append((parts[i], code, tail))
    assert len(ks) == 2, [k[0] for k in ks]      # forward and backward instantiation
    return ks


def test_only_the_named_statements_touch_agprs(kernels):
    mfma = re.compile(r"v_mfma_f32_16x16x32_bf16 a\[\w+:\w+\], v\[\d+:\d+\], v\[\d+:\d+\], (a\[\w+:\w+\]|0)$")
    rd = re.compile(r"v_accvgpr_read_b32 v\d+, a\[\w+\]$")
    for name, code, _ in kernels:
        users = [l for l in code if re.search(r"\ba(\[|\d)", l)]
        assert len(users) > 300, name
        bad = [l for l in users if not (mfma.match(l) or rd.match(l))]
        assert not bad, (name, bad[:5])
        # an MFMA updates its accumulator in place (or starts it from zero)
        for l in users:
            m = re.match(r"v_mfma_f32_16x16x32_bf16 (a\[\w+:\w+\]), .*, (a\[\w+:\w+\]|0)$", l)
            if m:
                assert m.group(2) in ("0", m.group(1)), l


def test_all_agprs_allocated_and_nothing_spilled(kernels):
    for name, code, tail in kernels:
        assert re.search(r"; NumAgprs: 256\b", tail), (name, tail[:800])
        assert re.search(r"; ScratchSize: 0\b", tail), (name, tail[:800])
        assert not [l for l in code if l.startswith("scratch_")], name
        assert re.search(r"; Occupancy: 1\b", tail), name


def test_m0_is_written_and_consumed_inside_one_statement(kernels):
    for name, code, _ in kernels:
        writes = [i for i, l in enumerate(code) if re.match(r"s_mov_b32 m0,", l)]
        copies = [i for i, l in enumerate(code) if l.startswith("global_load_lds_dwordx4")]
        assert len(copies) >= 48 and len(writes) == len(copies), (name, len(writes), len(copies))
        for w, c in zip(writes, copies):
            assert 0 < c - w <= 2, (name, code[w:c + 1])         # at most the MFMA / s_nop of the statement between
        # nothing else writes M0
        assert not [l for l in code if re.search(r"\bm0\b", l) and not l.startswith(("s_mov_b32 m0,", "global_load_lds"))], name


def _vregs(tok):
    m = re.match(r"v\[(\d+):(\d+)\]$", tok)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.match(r"v(\d+)$", tok)
    return {int(m.group(1))} if m else set()


def test_no_mfma_reads_a_register_a_vector_alu_instruction_has_just_written(kernels):
    """The MFMAs are asm statements and the compiler's hazard pass does not look into those: an MFMA needs two
    wait states between a vector ALU write of one of its operand registers and its own read of it (operands that
    come from LDS or memory are covered by the waitcnt the compiler does insert)."""
    for name, code, _ in kernels:
        for i, l in enumerate(code):
            if not l.startswith("v_mfma"):
                continue
            ops = [t.strip() for t in l.split(None, 1)[1].split(",")]
            src = _vregs(ops[1]) | _vregs(ops[2])
            states, k = 0, i - 1
            while states < 2 and k >= 0:
                pl = code[k]
                if pl.startswith("v_") and not pl.startswith(("v_mfma", "v_accvgpr")):
                    dst = pl.split(None, 1)[1].split(",")[0].strip()
                    assert not (_vregs(dst) & src), (name, code[k:i + 1])
                m = re.match(r"s_nop (\d+)$", pl)
                states += int(m.group(1)) + 1 if m else 1
                k -= 1


def test_main_loop_has_no_instruction_clumps(kernels):
    """A wave issues one instruction per four cycles and an MFMA holds its pipe for 16: more than a dozen other
    instructions between two MFMAs of the main loop drain the matrix pipe."""
    for name, code, _ in kernels:
        idx = [i for i, l in enumerate(code) if l.startswith("v_mfma")]
        # the longest run of MFMAs at most 13 instructions apart must cover a whole K tile (128 MFMAs) and more
        best = run = 1
        for a, b in zip(idx, idx[1:]):
            run = run + 1 if b - a <= 13 else 1
            best = max(best, run)
        assert best >= 128, (name, best)


@pytest.fixture(scope="module")
def ktail_kernels(tmp_path_factory):
    """The same kernel for K that is no multiple of 128 (compiled from the same source as kernels of another name)."""
    out = str(tmp_path_factory.mktemp("isa") / "gemm_persistent_ktail.s")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "hip", "--cuda-device-only",
           "-S", os.path.join(CSRC, "gemm_persistent_ktail.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    parts = re.split(r"^(_ZN5lobra28gemm_persistent_ktail_kernel\w+):", open(out).read(), flags=re.M)
    ks = []
    for i in range(1, len(parts), 2):
        body = parts[i + 1]
        end = body.index(".end_amdhsa_kernel")
        code = [l.split(";")[0].strip() for l in body[:body.rindex("s_endpgm", 0, end) + 8].split("\n")]
        ks.append((parts[i], [l for l in code if l and not l.startswith(".")], body[end:end + 3000]))
    assert len(ks) == 2, [k[0] for k in ks]
    return ks


@pytest.mark.parametrize("check", [test_only_the_named_statements_touch_agprs, test_all_agprs_allocated_and_nothing_spilled,
                                   test_m0_is_written_and_consumed_inside_one_statement,
                                   test_no_mfma_reads_a_register_a_vector_alu_instruction_has_just_written,
                                   test_main_loop_has_no_instruction_clumps], ids=lambda f: f.__name__)
def test_ktail_kernels(ktail_kernels, check):
    check(ktail_kernels)


# ---------------------------------------------------------------------------------------------------------
# The K-sliced rank-r kernel keeps several items' copies in flight and waits for them by count.  That only
# works if the compiler adds no wait of its own that drains them: its tables must be read with scalar loads
# (which the vector-memory counter does not see), the item barrier must come without a fence, and the copies
# must be the direct-to-LDS kind with M0 written right in front of each.
# ---------------------------------------------------------------------------------------------------------
@pytest.fixture(scope="module")
def sliced_kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("isa") / "skinny_mfma.s")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "hip", "--cuda-device-only",
           "-S", os.path.join(CSRC, "skinny_mfma.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    text = open(out).read()
    parts = re.split(r"^(_ZN5lobra20shrink_sliced_kernel\w+):", text, flags=re.M)
    ks = []
    for i in range(1, len(parts), 2):
        body = parts[i + 1]
        end = body.index(".end_amdhsa_kernel")
        code = [l.split(";")[0].strip() for l in body[:end].split("\n")]
        code = [l for l in code if l and not l.startswith(".")]
        ks.append((parts[i], code, body[end:end + 3000]))
    assert len(ks) == 1, [k[0] for k in ks]      # projection with dB
    return ks


def test_sliced_kernel_waits_for_its_copies_by_count(sliced_kernels):
    for name, code, tail in sliced_kernels:
        assert re.search(r"; ScratchSize: 0\b", tail), name
        copies = [i for i, l in enumerate(code) if l.startswith("global_load_lds_dwordx4")]
        assert len(copies) >= 16, (name, len(copies))
        for c in copies:            # M0 is written inside the copy's own asm statement
            assert any(re.match(r"s_mov_b32 m0,", code[k]) for k in range(max(0, c - 2), c)), (name, code[c - 3:c + 1])
        # the steady-state wait leaves the copies of three younger items in flight (wave 0 has a fifth copy per item), the
        # drain at the end counts down
        waits = {int(m.group(1)) for l in code for m in [re.match(r"s_waitcnt vmcnt\((\d+)\)$", l)] if m}
        assert {12, 8, 4} <= waits, (name, sorted(waits))
        assert {15, 10, 5} <= waits, (name, sorted(waits))
        # ordinary vector loads: only the adapter rows (16 bytes per lane), never the tables
        plain = [l for l in code if re.match(r"global_load_(dword|dwordx2|dwordx3|ubyte|ushort|sbyte|sshort)\b", l)]
        assert not plain, (name, plain[:4])
        assert [l for l in code if l.startswith("s_load_dwordx4") or l.startswith("s_load_dwordx2")], name
        # no barrier drags a full vector-memory wait along (what a fenced barrier would do)
        for i, l in enumerate(code):
            if l == "s_barrier":
                assert not any(re.match(r"s_waitcnt.*vmcnt\(0\)", code[k]) for k in range(max(0, i - 3), i)), (name, code[i - 4:i + 1])


# ---------------------------------------------------------------------------------------------------------
# The kernels with hand-placed barriers: the barrier instruction does not wait for LDS, so whatever a wave has written there
# for others must be waited for in front of it, on every path.
# ---------------------------------------------------------------------------------------------------------
def _lds_writes_pending_at_a_barrier(lines):
    """Follows every path through a kernel's assembly; returns the barriers (as the lines in front of them) at which a wave
    may arrive with an LDS write of its own in flight.  LDS operations of a wave end in order, so `lgkmcnt(n)` covers a write
    behind which n or more have been issued; the youngest write is the one to follow, and of two paths that meet, the one with fewer
    operations behind it."""
    labels = {l[:-1]: i for i, l in enumerate(lines) if l.endswith(":")}
    none = 1 << 30                                   # no write in flight
    best, todo, bad = {}, [(0, none)], set()
    while todo:
        i, behind = todo.pop()
        while i < len(lines) and behind < best.get(i, none + 1):
            best[i] = behind
            l = lines[i]
            if l.startswith("ds_write"):
                behind = 0
            elif l.startswith("ds_") and behind < none:
                behind += 1
            m = re.match(r"s_waitcnt\b.*lgkmcnt\((\d+)\)", l)
            if m and behind >= int(m.group(1)):
                behind = none
            if l.startswith("s_barrier") and behind < none:
                bad.add(i)
            if l.startswith("s_endpgm"):
                break
            m = re.match(r"s_c?branch\w*\s+(\S+)$", l)
            if m:
                todo.append((labels[m.group(1)], behind))
                if l.startswith("s_branch"):
                    break
            i += 1
    return [lines[max(0, i - 6):i + 1] for i in sorted(bad)]


def test_the_barrier_check_itself():
    wait, nowait = "s_waitcnt vmcnt(0) lgkmcnt(0)", "s_waitcnt vmcnt(0)"
    assert not _lds_writes_pending_at_a_barrier(["ds_write_b32 v0, v1", wait, "s_barrier", "s_endpgm"])
    assert _lds_writes_pending_at_a_barrier(["ds_write_b32 v0, v1", nowait, "s_barrier", "s_endpgm"])
    # covered by count only if that many operations lie behind the write
    assert not _lds_writes_pending_at_a_barrier(["ds_write_b32 v0, v1", "ds_read_b32 v2, v3", "s_waitcnt lgkmcnt(1)", "s_barrier", "s_endpgm"])
    assert _lds_writes_pending_at_a_barrier(["ds_write_b32 v0, v1", "s_waitcnt lgkmcnt(1)", "s_barrier", "s_endpgm"])
    # one of two paths waits
    assert _lds_writes_pending_at_a_barrier(["ds_write_b32 v0, v1", "s_cbranch_scc0 .L", wait, ".L:", "s_barrier", "s_endpgm"])
    # a write at a loop's end, a barrier at its head
    assert _lds_writes_pending_at_a_barrier([".L:", "s_barrier", "ds_write_b32 v0, v1", "s_cbranch_scc0 .L", "s_endpgm"])


@pytest.mark.parametrize("source,least", [("gemm_tile.hip", 8), ("gemm_persistent.hip", 2), ("gemm_persistent_ktail.hip", 2),
                                          ("skinny_mfma.hip", 10), ("fp32_mfma.hip", 12), ("gemm_staged.hip", 2)])
def test_lds_writes_are_waited_for_in_front_of_every_barrier(tmp_path, source, least):
    out = str(tmp_path / "k.s")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "hip", "--cuda-device-only",
           "-S", os.path.join(CSRC, source), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    parts = re.split(r"^(_ZN5lobra\w+):", open(out).read(), flags=re.M)
    kernels = barriers = 0
    for name, body in zip(parts[1::2], parts[2::2]):
        if ".end_amdhsa_kernel" not in body:
            continue
        lines = [l.split(";")[0].strip() for l in body[:body.index(".end_amdhsa_kernel")].split("\n")]
        lines = [l for l in lines if l and (not l.startswith(".") or l.endswith(":"))]
        kernels += 1
        barriers += sum(l.startswith("s_barrier") for l in lines)
        assert not _lds_writes_pending_at_a_barrier(lines), (name, _lds_writes_pending_at_a_barrier(lines)[0])
    assert kernels >= least and barriers >= kernels, (kernels, barriers)


def test_lds_writes_of_the_ring_projection_are_waited_for(tmp_path):
    test_lds_writes_are_waited_for_in_front_of_every_barrier(tmp_path, "shrink_ring.hip", 6)


@pytest.mark.parametrize("source,least", [("fp32_mfma.hip", 30), ("gemm_tile.hip", 8), ("shrink_ring.hip", 6), ("kernels_plain.hip", 8)])
def test_no_kernel_takes_scratch_memory(tmp_path, source, least):
    """Registers that do not fit go to scratch memory, whose loads the counted waits of the copies would wait for as well."""
    out = str(tmp_path / "k.s")
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "hip", "--cuda-device-only",
           "-S", os.path.join(CSRC, source), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    parts = re.split(r"^\s*\.amdhsa_kernel (\w+)$", open(out).read(), flags=re.M)
    sizes = {name: int(re.search(r"; ScratchSize: (\d+)", body).group(1)) for name, body in zip(parts[1::2], parts[2::2])}
    assert len(sizes) >= least, (source, len(sizes))
    assert not {k: v for k, v in sizes.items() if v}
