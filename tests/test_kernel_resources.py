"""Every gfx950 kernel of the library must run without scratch memory and without reading the
dispatch packet: both were measured to cost far more than the short decode kernels themselves
(a private array that the compiler failed to keep in registers, or a by-value argument struct
indexed at run time, each silently add microseconds per workgroup).  Checked on the compiler's
assembly output; needs hipcc, not a GPU."""
import functools
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_2501_04052_amd import build

ALLOWED_SCRATCH = {}      # kernel-name substring -> bytes (none at present)


@functools.lru_cache(maxsize=None)
def _asm(src):
    cmd = [build.hipcc()] + [f for f in build.HIPCC_FLAGS if f != "-fPIC"] + \
          ["--cuda-device-only", "-S", os.path.join(build.CSRC, src), "-o", "-"]
    return subprocess.run(cmd, check=True, capture_output=True, text=True).stdout


def test_encoder_keeps_its_waves():
    """The block encoder is bound by vector issue and by waiting waves; its rare paths (near ties, non-finite blocks) are
    compiled into the same kernels and must not take the registers that four waves per SIMD (five for 16-bit elements in
    blocks of 16) leave: 512 / 4, and 512 / 5 in steps of 8."""
    text = _asm("razer_quantize.hip")
    regs = {m.group(1): int(re.search(r"\.amdhsa_next_free_vgpr (\d+)", m.group(2)).group(1))
            for m in re.finditer(r"\.amdhsa_kernel (\S*encode_kernel\S*)(.*?)\.end_amdhsa_kernel", text, re.S)}
    assert len(regs) == 18
    for name, n in regs.items():
        single = "kernelIt" in name and "ELi1EEv" in name        # element type; last template argument: runs per block
        assert n <= (96 if single else 128), (name, n)


def _vector_registers(operands):
    out = set()
    for kind, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", operands):
        out |= {(kind, i) for i in range(int(lo), int(hi) + 1)}
    return out | {(kind, int(i)) for kind, i in re.findall(r"\b([va])(\d+)\b", operands)}


def _uses_before_wait(lines):
    """Instructions that touch a register which an LDS read may still be writing, on any path through the kernel.  LDS
    reads return in order, so s_waitcnt lgkmcnt(n) leaves the newest n in flight; a scalar load among them (None below)
    may return out of order, then only lgkmcnt(0) tells anything.  The counter has four bits: with 15 in flight the next
    one waits."""
    code, labels = [], {}
    for line in lines:
        label = re.match(r"(\.L\w+):", line)
        if label:
            labels[label.group(1)] = len(code)
        line = line.split(";")[0].strip()
        if line and not line.startswith(".") and not line.endswith(":"):
            op, _, operands = line.partition(" ")
            code.append((op, operands, _vector_registers(operands)))
    targets = set(labels.values())
    found, seen, work = set(), set(), [(0, ())]
    while work:
        pc, flying = work.pop()
        while pc < len(code):
            if pc in targets:
                if (pc, flying) in seen:
                    break
                seen.add((pc, flying))
            op, operands, regs = code[pc]
            if op == "s_endpgm":
                break
            if op == "s_waitcnt":
                n = re.search(r"lgkmcnt\((\d+)\)", operands)
                if n and (n.group(1) == "0" or None not in flying):
                    flying = flying[len(flying) - min(len(flying), int(n.group(1))):]
            else:
                if regs and any(r and regs & r for r in flying):
                    found.add("%s %s" % (op, operands))
                if op.startswith("ds_"):
                    returns = re.match(r"ds_(read|bpermute|permute|swizzle|\w+_rtn)", op)
                    flying += (frozenset(_vector_registers(operands.split(",")[0])) if returns else frozenset(),)
                elif re.match(r"s_(buffer_)?load|s_mem", op):
                    flying += (None,)
                flying = flying[-16:]
            if op.startswith(("s_branch", "s_cbranch")):
                work.append((labels[operands.strip()], flying))
                if op == "s_branch":
                    break
            pc += 1
    return found


def test_registers_of_lds_reads_are_left_alone_until_their_wait():
    """The GEMM and small-batch kernels read LDS in inline assembly and place the waits by hand.  To the compiler such a
    register is written at once and free after its last use: where a wait does not name the registers it guards, only
    the order of the generated code keeps their users behind it."""
    kernels = checked = 0
    for src in ("razer_gemm.hip", "razer_skinny.hip"):
        for m in re.finditer(r"^(_ZN5razer\S*):[^\n]*\n(.*?)^\.Lfunc_end", _asm(src), re.S | re.M):
            kernels += 1
            checked += m.group(2).count("ds_read")
            bad = _uses_before_wait(m.group(2).split("\n"))
            assert not bad, (m.group(1), sorted(bad)[:4])
    assert kernels >= 100 and checked >= 1000
    # the check itself: a use ahead of the wait, one behind it, a wait that leaves the read in flight, a loop's back edge
    read, use = "ds_read_b128 v[0:3], v9", "v_mov_b32_e32 v2, 0"
    assert _uses_before_wait([read, use, "s_waitcnt lgkmcnt(0)", "s_endpgm"]) == {"v_mov_b32_e32 v2, 0"}
    assert not _uses_before_wait([read, "s_waitcnt lgkmcnt(0)", use, "s_endpgm"])
    assert _uses_before_wait([read, "ds_read_b32 v5, v9", "s_waitcnt lgkmcnt(1)", "v_add_f32 v1, v5, v6", "s_endpgm"]) == {"v_add_f32 v1, v5, v6"}
    assert _uses_before_wait([".LBB0_1:", use, read, "s_cbranch_scc1 .LBB0_1", "s_waitcnt lgkmcnt(0)", "s_endpgm"]) == {use, read}


def _copies_before_counted_wait(lines):
    """What stands between a full wait for copies and the next counted one, in the order of issue: a = 16-byte copy, s =
    scale copy (1 or 2 bytes), p = 4-byte copy (a prefetch), | = branch.  A full wait with no copy between it and the counted
    one is the one in its place when nothing follows."""
    seq, before, found = "", "", []
    for line in lines:
        op = line.split(";")[0].strip()
        if op.startswith("global_load_lds"):
            seq += {"x4": "a", "rd": "p"}.get(op.split()[0][-2:], "s")
        elif op.startswith(("s_cbranch", "s_branch")):
            seq += "" if seq.endswith("|") else "|"
        elif op.startswith("s_waitcnt") and "vmcnt" in op:
            n = int(re.search(r"vmcnt\((\d+)\)", op).group(1))
            if n:
                found.append((n, seq if seq.strip("|") else before))
            else:
                before, seq = (seq if seq.strip("|") else before), ""
    return found


def test_small_batch_kernel_counts_the_copies_it_may_leave():
    """With activations in halves the wait ahead of the second half leaves the newest 2 G copies in flight (G where the
    workgroup staged the scales).  Copies land in the order of their issue, so these must be the next step's G codes and G
    scales and every activation copy must stand before them."""
    kernels = {"": 0, "staged_": 0, "sliced_": 0}
    for m in re.finditer(r"^(_ZN5razer\d\d(|staged_|sliced_)ring_kernelILi(\d+)ELi(\d)ELb[01]ELi[01]ELi(\d+)ELb[01]EE\S*):[^\n]*\n(.*?)^\.Lfunc_end", _asm("razer_skinny.hip"), re.S | re.M):
        kind, na, g, waves = m.group(2), int(m.group(3)), int(m.group(4)), int(m.group(5))
        if not (na == 16 or (na == 4 and waves == 16)):              # (whole steps)
            continue
        kernels[kind] += 1
        left = "a" * g + ("" if kind == "staged_" else "s" * g)
        assert _copies_before_counted_wait(m.group(6).split("\n")) == [(len(left), "a" * (na // 2) + "|" + left + "|")], m.group(1)
    assert kernels == {"": 17, "staged_": 17, "sliced_": 4}
    # the check itself: an activation copy behind the codes
    copy, scale, wait = "global_load_lds_dwordx4 v1, s[0:1]", "global_load_lds_ushort v1, s[0:1]", "s_waitcnt vmcnt(2)"
    full = ["s_waitcnt vmcnt(0)", copy, copy, "s_cbranch_scc1 .L1", copy, scale, ".L1:", "s_cbranch_scc1 .L2", "s_waitcnt vmcnt(0)", "s_cbranch_scc1 .L3", wait]
    assert _copies_before_counted_wait(full) == [(2, "aa|as|")]
    assert _copies_before_counted_wait(full[:2] + full[3:5] + [copy] + full[5:]) == [(2, "a|aas|")]


def test_wide_gemm_counts_the_copies_it_may_leave():
    """64 weight rows per wave.  The wait for K-tile kt + 1 leaves the newest 12 copies in flight, which must be those of tile
    kt + 2 (eight of activations, two of codes, two of scales); with two K groups the newest one, which must be the
    prefetch.  Each loop has one such wait: whole K-tiles, and the last ones of a row that ends inside a K-tile."""
    kernels = 0
    for m in re.finditer(r"^(_ZN5razer\d\dgemm_(halves|wide)\S*):[^\n]*\n(.*?)^\.Lfunc_end", _asm("razer_gemm.hip"), re.S | re.M):
        kernels += 1
        found = _copies_before_counted_wait(m.group(3).split("\n"))
        assert [n for n, _ in found] == [1, 1] + [12, 12] * (m.group(2) == "wide"), (m.group(1), found)
        for n, seq in found:
            assert re.search(r"a{8}p$" if n == 1 else r"a{10}ss$", seq), (m.group(1), n, seq)
    assert kernels == 8


def test_no_scratch_no_dispatch_packet():
    with ThreadPoolExecutor(max_workers=6) as ex:
        outs = list(ex.map(_asm, build.SOURCES))
    seen = 0
    for src, text in zip(build.SOURCES, outs):
        for m in re.finditer(r"\.amdhsa_kernel (\S+)(.*?)\.end_amdhsa_kernel", text, re.S):
            name, body = m.group(1), m.group(2)
            seen += 1
            scratch = int(re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", body).group(1))
            allowed = max([v for k, v in ALLOWED_SCRATCH.items() if k in name] + [0])
            assert scratch <= allowed, "%s: %s uses %d bytes of scratch" % (src, name, scratch)
            disp = re.search(r"\.amdhsa_user_sgpr_dispatch_ptr (\d+)", body)
            assert disp is None or disp.group(1) == "0", "%s: %s reads the dispatch packet" % (src, name)
    assert seen >= 20
