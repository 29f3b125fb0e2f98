"""CPU check of the generated device code (no GPU needed: hipcc cross-compiles to assembly).

The weight-streaming loops of the GEMM phases only reach HBM speed if every wait in them leaves the other
seven weight loads of the wavefront in flight (`s_waitcnt vmcnt(7)`).  Whether the compiler emits that
depends on details far from the loop - e.g. an activation-panel address it can no longer prove to be LDS
becomes a flat load, and then every wait in the loop waits for all loads - so the property is checked on the
assembly of the instantiation the bf16 workloads run."""
import os
import re
import subprocess

import pytest

from paper_2410_05589_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _assembly(tmp_path_factory, source, defines=()):
    out = str(tmp_path_factory.mktemp("asm") / (source + ".s"))
    cmd = [build.hipcc_path(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fno-gpu-rdc", "-fvisibility=hidden",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-mllvm", "-instcombine-max-copied-from-constant-users=10000",
           "-I", os.path.join(ROOT, "include"), "-I", build.CSRC, *defines,
           "--cuda-device-only", "-S", "-o", out, os.path.join(build.CSRC, source + ".hip")]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-2000:]
    return open(out).read()


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    return _assembly(tmp_path_factory, "ps_inst", ("-DPS_INST_NAME=bf16_d128", "-DPS_INST_BF16=1", "-DPS_INST_D=128"))


def _streaming_loops(text):
    """(kernel, label, mfma count, vmcnt values, scratch accesses) of every basic block that branches back to itself
    and holds 8 weight loads and at least 16 MFMAs."""
    found = []
    kernel, label, lines = None, None, []

    def close():
        if kernel and label:
            n_mfma = sum("v_mfma" in l for l in lines)
            n_load = sum("global_load_dwordx4" in l for l in lines)
            loops = any(re.search(r"s_cbranch\w+\s+%s\b" % re.escape(label), l) for l in lines)
            if loops and n_mfma >= 16 and n_load == 8:
                found.append((kernel, label, n_mfma, [int(m.group(1)) for l in lines for m in [re.search(r"vmcnt\((\d+)\)", l)] if m],
                              sum("scratch_" in l for l in lines)))

    for line in text.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            close()
            kernel, label, lines = m.group(1), None, []
            continue
        m = re.match(r"^(\.LBB\d+_\d+):", line)
        if m:
            close()
            label, lines = m.group(1), []
            continue
        lines.append(line)
    close()
    return found


def test_streaming_loops_keep_seven_weight_loads_in_flight(asm):
    loops = _streaming_loops(asm)
    fused = [l for l in loops if "fused_kernel" in l[0]]
    # the persistent kernel: four variants (1..4 column tiles of rows) x five GEMM phases
    assert len(fused) == 20, [(l[0], l[1]) for l in fused]
    for kernel, label, n_mfma, waits, scratch in loops:
        assert waits and all(w == 7 for w in waits) and scratch == 0, (kernel, label, waits, scratch)


def test_no_flat_loads_and_few_spills_in_the_persistent_kernel(asm):
    """Nothing spilled for up to three column tiles of rows; four (49 to 64 rows) may spill a handful of values that live through
    the step (at present none, see below), none of them inside a streaming loop (see above)."""
    assert "flat_load" not in asm
    meta = re.findall(r"\.name:\s+(\S+)\n(?:.*\n)*?\s+\.vgpr_spill_count:\s+(\d+)", asm)
    spills = {n: int(v) for n, v in meta}
    fused = {n: v for n, v in spills.items() if "fused_kernel" in n}
    assert len(fused) == 4, fused
    for n, v in fused.items():
        assert v <= (11 if "ELi4EEv" in n else 0), (n, v)
    for lds, scratch, vgpr, spill in _resources(asm, "fused_kernel"):
        assert vgpr <= 256 and scratch <= 60


def test_the_persistent_kernel_spills_nothing(asm):
    """All four variants keep their values in registers: seven spilled ones cost a step of 49 to 64 rows 1 to 2.5 %."""
    found = _resources(asm, "fused_kernel")
    assert len(found) == 4 and all(spill == 0 for lds, scratch, vgpr, spill in found), found


def test_attention_loop_keeps_the_next_key_groups_in_flight(asm):
    """bf16 attention: while a wavefront works on two groups of keys, the K and V rows of the next two (16 loads)
    must stay in flight: every wait inside the loop over key groups leaves at least 8 loads outstanding.  (Requests
    under a condition would make the compiler wait for all of them.)"""
    text = asm[asm.index("_Z12attn2_kernel"):]
    text = text[:text.index("s_endpgm")]
    loops = {}          # header label -> lines of all the blocks of that (inner) loop
    cur = None
    for line in text.splitlines():
        m = re.match(r"^\.L(BB\d+_\d+):\s*(;.*)?$", line)
        if m:
            note = m.group(2) or ""
            h = re.search(r"in Loop: Header=(BB\d+_\d+) Depth=2", note)
            cur = h.group(1) if h else (m.group(1) if "Parent Loop" in note and "Depth=1" in note else None)
            continue
        if cur:
            loops.setdefault(cur, []).append(line)
    found = []
    for header, body in loops.items():
        n_mfma = sum("v_mfma" in l for l in body)
        n_load = sum("global_load_dwordx4" in l for l in body)
        if n_mfma >= 40 and n_load >= 16:
            found.append((header, [int(m.group(1)) for l in body for m in [re.search(r"vmcnt\((\d+)\)", l)] if m]))
    assert len(found) == 1, found
    assert found[0][1] and min(found[0][1]) >= 8, found


@pytest.fixture(scope="module")
def train_asm(tmp_path_factory):
    return _assembly(tmp_path_factory, "ps_train")


def _resources(text, kernel):
    """(bytes of LDS, bytes of scratch, vector registers, spilled ones) of the kernel's instances."""
    found = re.findall(r"\.group_segment_fixed_size:\s+(\d+)\n(?:.*\n)*?\s+\.name:\s+(\S+)\n(?:.*\n)*?\s+\.private_segment_fixed_size:\s+(\d+)\n"
                       r"(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)\n\s+\.vgpr_spill_count:\s+(\d+)", text)
    return [tuple(int(x) for x in (m[0], m[2], m[3], m[4])) for m in found if kernel in m[1]]


def test_training_attention_kernel_fits_four_workgroups_per_compute_unit(train_asm):
    """The 16-row bf16 kernel of the training attention runs four workgroups (16 wavefronts) per compute unit: at most
    128 vector registers per lane and 40 KiB of LDS per workgroup, no flat loads (LDS addresses stay LDS addresses), and
    only a handful of spilled registers (loop-invariant values)."""
    assert "flat_load" not in train_asm
    found = _resources(train_asm, "ga_attn_bf16_kernel")
    assert len(found) == 2        # head_dim 64 and 128
    for lds, scratch, vgpr, spill in found:
        assert vgpr <= 128 and lds <= 40 * 1024 and spill <= 4, found


def test_training_attention_wide_and_float32_kernels_fit_the_compute_units_places(train_asm):
    """The wide bf16 kernel runs two workgroups of four wavefronts per compute unit (256 vector registers per lane); the float32
    kernel four of four (head_dim 64) or two of eight (128 registers both), the one of short calls two of eight (head_dim
    64) or one (256): in a quarter, half or all of a compute unit's 160 KiB of LDS each, with nothing spilled.  (Eight
    spilled registers cost the wide kernel 3 % of a short call.  The scratch memory is that of the call that looks at rows
    which are not finite.)"""
    for kernel, d, regs, per_cu in (("ga_attn_wide_kernel", 64, 256, 2), ("ga_attn_wide_kernel", 128, 256, 2),
                                    ("ga_attn_f32_kernel", 64, 128, 4), ("ga_attn_f32_kernel", 128, 128, 2),
                                    ("ga_attn_f32_short_kernel", 64, 128, 2), ("ga_attn_f32_short_kernel", 128, 256, 1)):
        found = _resources(train_asm, "%sILi%dE" % (kernel, d))
        assert len(found) == 1, (kernel, d, found)
        lds, scratch, vgpr, spill = found[0]
        assert lds <= 160 * 1024 // per_cu and vgpr <= regs and spill == 0 and scratch <= 32, (kernel, d, found)


def test_training_attention_main_loops(train_asm):
    """The loops over the real tokens' keys hold the MFMAs of one tile and no scratch accesses: 2 products x 2 parts of the
    bf16 split x head_dim / 16 steps (wide kernel), 2 x head_dim / 4 (float32, both kernels)."""
    for kernel, mfma, counts in (("ga_attn_wide_kernel", "v_mfma_f32_32x32x16_bf16", {64: 16, 128: 32}),
                                 ("ga_attn_f32_kernel", "v_mfma_f32_16x16x4_f32", {64: 32, 128: 64}),
                                 ("ga_attn_f32_short_kernel", "v_mfma_f32_16x16x4_f32", {64: 32, 128: 64})):
        for d, n in counts.items():
            text = train_asm[re.search(r"^_Z\w*%sILi%d\w*:" % (kernel, d), train_asm, flags=re.M).end():]
            text = text[:text.index(".Lfunc_end")]
            loops, label = {}, None
            for line in text.splitlines():
                m = re.match(r"^\.L(BB\d+_\d+):\s*(;.*)?$", line)
                if m:
                    note = m.group(2) or ""
                    h = re.search(r"in Loop: Header=(BB\d+_\d+) Depth=1", note)
                    label = h.group(1) if h else (m.group(1) if "Loop Header: Depth=1" in note else None)
                    continue
                if label:
                    loops.setdefault(label, []).append(line)
            found = [(sum(mfma in l for l in body), sum("scratch_" in l for l in body)) for body in loops.values()]
            assert (n, 0) in found, (kernel, d, found)


def test_the_walk_kernels_hold_their_rows_in_registers(tmp_path_factory):
    """The walk's workgroups are 16 wavefronts (at most 128 vector registers per lane) that keep the residual and the drafter's row
    in registers, with nothing in scratch memory and no flat loads."""
    text = _assembly(tmp_path_factory, "ps_verify")
    assert "flat_load" not in text
    for kernel, n in (("verify_walk_reg_kernel", 2), ("verify_walk_kernel", 3)):
        found = _resources(text, kernel)
        assert len(found) == n, (kernel, found)
        for lds, scratch, vgpr, spill in found:
            assert vgpr <= 128 and spill == 0 and scratch == 0 and lds <= 64 * 1024, (kernel, found)
