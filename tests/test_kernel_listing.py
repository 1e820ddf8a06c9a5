"""What the hand-scheduled product kernels rely on and the compiler does not know, read off the listing of the built library:
loads that are requested in one place and collected in another by a hand-written wait, and DMA requests whose LDS target
travels in a register (m0) that an earlier statement wrote."""
import os
import re
import struct
import subprocess
import tempfile

import pytest

import paper_2210_03052_amd as pkg

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def code_objects(path):
    """The gfx950 code objects of a shared library (uncompressed offload bundles)."""
    data, at, out = open(path, "rb").read(), 0, []
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                out.append(data[at + off:at + off + size])
            p += 24 + length
        at += 24
    return out


@pytest.fixture(scope="module")
def kernels():
    """{mangled name: [instruction, ...]} of every kernel of the library; labels are kept as 'name:'."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(pkg.LIB_PATH):
        from paper_2210_03052_amd.build import build_library
        build_library(verbose=False)
    found = {}
    for code in code_objects(pkg.LIB_PATH):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(code)
            f.flush()
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", "--symbolize-operands", f.name],
                                  check=True, capture_output=True, text=True).stdout
        body = None
        for line in text.splitlines():
            m = re.match(r"<(\S+)>:", line)
            if m and re.fullmatch(r"L\d+", m.group(1)) and body is not None:
                body.append(m.group(1) + ":")
            elif m:
                body = found.setdefault(m.group(1), [])
            elif body is not None and line.strip():
                body.append(line.split("//")[0].strip())
    assert found
    return found


def registers(text):
    """Vector registers named in an instruction or operand."""
    out = set()
    for m in re.finditer(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        lo = int(m.group(2) or m.group(4))
        out |= {m.group(1) + str(r) for r in range(lo, int(m.group(3) or lo) + 1)}
    return out


def dma_faults(body):
    """DMA requests into LDS without a target of their own: m0 has to be written for each of them, in the same run of
    instructions, with another instruction in between (the wait state between the write and its use)."""
    bad, written = [], None
    for i, ins in enumerate(body):
        if ins.endswith(":") or re.match(r"s_(c?branch|setpc|swappc|call|endpgm)", ins):
            written = None
        elif ins.startswith("global_load_lds"):
            if written is None or i - written < 2:
                bad.append((i, ins))
            written = None
        elif re.match(r"\S+ m0\b", ins):
            if written is not None:
                bad.append((written, body[written]))
            written = i
    return bad


def in_flight(body):
    """(instructions that touch the destination of a row-sum request before the wait that collects it, MFMAs issued
    between the first run of requests and that wait)."""
    first = next(i for i, ins in enumerate(body) if ins.startswith("global_load_dwordx2"))
    pending, touched, mfmas = set(), [], 0
    for ins in body[first:]:
        if ins.startswith("s_waitcnt") and "vmcnt(0)" in ins:
            return touched, mfmas
        if ins.startswith("global_load_dwordx2"):
            dest, addr = ins.split(",", 1)
            if registers(addr) & pending:
                touched.append(ins)
            pending |= registers(dest)
        elif registers(ins) & pending:
            touched.append(ins)
        mfmas += ins.startswith("v_mfma")
    raise AssertionError("no wait behind the requests")


def test_in_flight_finds_a_touched_register():
    run = ["global_load_dwordx2 v[2:3], v[8:9], off", "v_mfma_f32_16x16x32_f16 a[0:3], v[10:13], v[14:17], a[0:3]",
           "s_waitcnt vmcnt(0)"]
    assert in_flight(run) == ([], 1)
    assert in_flight(run[:1] + ["v_mov_b32_e32 v5, v3"] + run[1:])[0] == ["v_mov_b32_e32 v5, v3"]
    assert in_flight(run[:1] + ["global_load_dwordx2 v[4:5], v[2:3], off"] + run[1:])[0]


def test_folded_wide_row_sums_are_requested_ahead_of_the_last_slabs(kernels):
    """EPI_FOLD of the wide tiles: the row sums travel under at least one slab of MFMAs (2 k-steps of MI x NI), and nothing
    touches the registers they arrive in before the wait."""
    names = [n for n in kernels if re.search(r"gemm_wide_kernelILi\d+ELi128ELi\dELi1E", n)]
    assert len(names) == 15  # 256, 192, 128 rows; three shape classes without activation and two activations
    for n in names:
        rows = int(re.search(r"ILi(\d+)E", n).group(1))
        touched, mfmas = in_flight(kernels[n])
        assert not touched, (n, touched[:4])
        assert mfmas >= 2 * (rows // 32) * 4, (n, mfmas)


def test_dma_faults_finds_lost_and_hasty_targets():
    to, load, mfma = "s_add_u32 m0, s4, 0x400", "global_load_lds_dwordx4 v2, s[2:3]", "v_mfma_f32_16x16x32_f16 a[0:3], v[10:13], v[14:17], a[0:3]"
    assert dma_faults([to, mfma, load, to, "s_nop 0", load]) == []
    assert dma_faults([to, load])                                      # no wait state
    assert dma_faults([to, mfma, load, mfma, load])                    # second request without a target
    assert dma_faults([to, "s_mov_b32 m0, s9", mfma, load])            # something else wrote m0 in between
    assert dma_faults([to, "L3:", mfma, load])                         # another way into the request


def test_every_dma_request_has_its_own_target(kernels):
    """The hand-scheduled loop writes m0 in one statement and requests in another, with an MFMA between them that the
    compiler could move: in the built library every pair is whole."""
    seen = 0
    for name, body in kernels.items():
        assert not dma_faults(body), (name, dma_faults(body)[:3])
        seen += sum(ins.startswith("global_load_lds") for ins in body)
    assert seen > 1000


def test_layernorm_rows_are_one_memory_round_trip(kernels):
    """Packed rows up to 1024 wide: all five operands of a row (x, residual, gamma, beta, bias) are requested before the
    first wait for any of them."""
    for cpl in (1, 2):
        body, = (b for n, b in kernels.items() if f"bias_residual_ln_kernelILi{cpl}ELb0ELb0ELb0E" in n)
        first = next(i for i, ins in enumerate(body) if ins.startswith("global_load_dwordx4"))
        wait = next(i for i, ins in enumerate(body) if i > first and ins.startswith("s_waitcnt") and "vmcnt" in ins)
        assert sum(ins.startswith("global_load_dwordx4") for ins in body[first:wait]) == 5 * cpl, cpl


def test_mask_total_is_reported_behind_every_workgroup(kernels):
    """The kernel with a workgroup per 4 096 mask entries may tell the host the total only when all of them have read theirs, since
    the host is free to refill the mask then: the workgroup that reports is the one whose counter increment came back complete."""
    bodies = {n: b for n, b in kernels.items() if "offsets_mask_chunks_kernel" in n}
    assert bodies
    for name, body in bodies.items():
        counted = [i for i, t in enumerate(body) if t.startswith("global_atomic_add_x2") and "sc0" in t]  # sc0: returns the old value
        reported = [i for i, t in enumerate(body) if re.match(r"(global|flat)_store_dword\b", t) and "sc0 sc1" in t]  # system scope
        one_workgroup = "ILb1E" in name
        assert reported and len(counted) == (0 if one_workgroup else 1), name
        assert one_workgroup or min(reported) > counted[0], name
