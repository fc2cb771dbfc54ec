"""What the compiler reported for the kernels of the library as built (paper_2510_26692_amd/libkda.resources.json,
written by every build): the kernels of the bench workloads must not touch scratch memory.  In the one-kernel
prefill a scratch access waits behind the write-through slot stores in the same queue (a chunk took 22 instead of
14 microseconds with a handful of spilled registers), and an array indexed by the wave number, which the compiler
places in scratch, cost the 2^20-token workload 5 % before it was noticed."""
import json
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
REPORT = os.path.join(ROOT, "paper_2510_26692_amd", "libkda.resources.json")


@pytest.fixture(scope="module")
def resources():
    if not os.path.exists(REPORT):
        pytest.skip("no resource report: build the library first (python -m paper_2510_26692_amd.build)")
    with open(REPORT) as f:
        return json.load(f)


def _kernels(resources, *fragments):
    return {k: v for k, v in resources.items() if all(f in k for f in fragments)}


def test_report_covers_the_kernels_of_the_hot_path(resources):
    assert len(_kernels(resources, "kda_prefill_kernel")) == 10          # raw x bf16-out x gate, scalar x bf16-out
    assert _kernels(resources, "kda_step_kernel") and _kernels(resources, "kda_fused_fill_kernel")


def test_prefill_kernels_use_no_scratch_outside_the_gated_variants(resources):
    # template arguments <kRaw, kScalar, kOutBf16, kGate>
    every = _kernels(resources, "kda_prefill_kernel")
    for name, r in every.items():
        gate = name.endswith("Lb1EEEvNS0_9FusedArgsE")
        assert r["VGPRs"] <= 256 and r["Occupancy [waves/SIMD]"] >= 2, (name, r)
        if not gate:
            assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, (name, r)
        else:
            # (the gated variants keep a few dwords outside the scan loop)
            assert r["VGPRs Spill"] <= 16, (name, r)


def test_decode_kernels_use_no_scratch(resources):
    for name, r in _kernels(resources, "kda_step_kernel").items():
        assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, (name, r)


def test_fp32_kernels_use_no_scratch_beyond_a_few_dwords_of_the_gradients_kernel(resources):
    # The walks are chains of steps, and the per-chunk kernel is short: neither has anything to hide a reload behind.  The
    # gradients kernel keeps two workgroups a compute unit (256 registers); at d 128 a few values wait in scratch between
    # its two halves.
    walks = _kernels(resources, "kda_f32_forward_walk") | _kernels(resources, "kda_f32_forward_roles") | \
        _kernels(resources, "kda_f32_both_walks")
    prep, gradients = _kernels(resources, "kda_f32_prep_kernel"), _kernels(resources, "kda_bwd_gradients_kernel")
    halves = _kernels(resources, "kda_bwd_half_gradients_kernel")
    assert len(walks) == 10 + 4 + 21 and len(prep) == 8 and len(gradients) == 6 and len(halves) == 3
    for name, r in (walks | prep | halves).items():          # (a half has one channel tile a wave, and registers to spare)
        assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, (name, r)
    for name, r in (walks | halves).items():                 # the dispatch counts on two workgroups a compute unit
        assert r["Occupancy [waves/SIMD]"] >= 2, (name, r)
    for name, r in prep.items():
        assert r["Occupancy [waves/SIMD]"] >= 3, (name, r)
    for name, r in gradients.items():
        assert r["Occupancy [waves/SIMD]"] >= 2 and r["VGPRs Spill"] <= (8 if "Li128E" in name else 0), (name, r)


_OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _kernel_code(lib, folder, fragment):
    """{kernel name: [instruction, ..]} of the kernels of `lib` whose name holds `fragment`, as the compiler left them."""
    here = os.path.join(str(folder), "lib.so")
    os.symlink(lib, here)                                    # (the code objects are written beside the file)
    subprocess.run([_OBJDUMP, "--offloading", here], check=True, capture_output=True, cwd=str(folder))
    code = {}
    for name in os.listdir(str(folder)):
        path = os.path.join(str(folder), name)
        if "gfx950" not in name or fragment.encode() not in open(path, "rb").read():
            continue
        text = subprocess.run([_OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", path], check=True, capture_output=True, text=True).stdout
        kernel = None
        for ln in text.splitlines():
            m = re.match(r"(?:[0-9a-f]+ )?<(\w+)>:", ln)
            if m:
                kernel = code.setdefault(m.group(1), []) if fragment in m.group(1) else None
            elif kernel is not None and ln.strip():
                kernel.append(ln.split("//")[0].strip())
    return code


@pytest.mark.skipif(not os.path.exists(_OBJDUMP), reason="needs llvm-objdump")
def test_no_prefill_kernel_waits_for_each_load_of_a_state_before_the_next(tmp_path):
    """A scan workgroup starts from 64 loads a lane.  Asked one by one whether there is a state to load, two of the kernels waited for
    each (4 pairs of 4023 tokens, gate and bf16 output: 156 instead of 140 us).  The longest run of loads with a wait for all memory
    between any two and no store and no product: the copy of a range's final state, which waits for each, stores each."""
    lib = os.path.join(ROOT, "paper_2510_26692_amd", "libkda.so")
    if not os.path.exists(lib):
        pytest.skip("no library: build it first (python -m paper_2510_26692_amd.build)")
    kernels = _kernel_code(lib, tmp_path, "kda_prefill_kernel")
    kernels = {k: v for k, v in kernels.items() if len(v) > 1000}        # (descriptors of the same name are data)
    assert len(kernels) == 10
    for name, code in kernels.items():
        longest = run = 0
        waited = False
        for ins in code:
            if ins.startswith("global_load_dword "):
                run = run + 1 if waited else 0
                longest, waited = max(longest, run), False
            elif ins.startswith("s_waitcnt") and "vmcnt(0)" in ins:
                waited = True
            elif ins.startswith(("global_store", "flat_store", "v_mfma", "s_barrier", "ds_")):
                run, waited = 0, False
        assert longest < 8, (name, longest)


def _scalar_registers(operands):
    found = set()
    for first, last, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", operands):
        found |= {int(one)} if one else set(range(int(first), int(last) + 1))
    return found


def _written_by_vector(ins):
    """Scalar registers that a vector instruction writes."""
    op, _, rest = ins.partition(" ")
    operands = rest.split(",")
    if op in ("v_readlane_b32", "v_readfirstlane_b32") or op.startswith("v_cmp"):
        return _scalar_registers(operands[0])
    return _scalar_registers(operands[1]) if "_co_" in op and len(operands) > 1 else set()


def early_scalar_reads(code):
    """Memory instructions that read a scalar register less than five wait states after a vector instruction wrote it: they read
    the register as it was before.  [(position, instruction that wrote, memory instruction), ..]"""
    found = []
    for i, ins in enumerate(code):
        if not ins.startswith(("buffer_", "global_", "flat_", "scratch_")):
            continue
        open_, states, j = _scalar_registers(ins), 0, i - 1
        while open_ and j >= 0 and states < 5:
            before = code[j]
            if before.startswith("v_") and _written_by_vector(before) & open_:
                found.append((i, before, ins))
                break
            if before.startswith("s_") and not before.startswith(("s_cmp", "s_bitcmp", "s_waitcnt", "s_nop", "s_barrier", "s_cbranch", "s_branch")):
                open_ -= _scalar_registers(before.partition(" ")[2].split(",")[0])       # (written again by a scalar instruction: no wait needed)
            states += int(before.split()[1]) + 1 if before.startswith("s_nop") else 1
            j -= 1
    return found


def test_early_scalar_reads_are_found():
    base = ["v_readlane_b32 s3, v255, 21"]
    load = ["global_load_dword v73, v78, s[2:3] sc1"]
    assert len(early_scalar_reads(base + load)) == 1
    assert len(early_scalar_reads(base + ["s_mov_b32 m0, s5", "s_nop 0"] + load)) == 1
    assert not early_scalar_reads(base + ["s_nop 4"] + load)
    assert not early_scalar_reads(base + ["s_mov_b64 s[2:3], s[2:3]"] + load)
    assert len(early_scalar_reads(["v_cmp_eq_u32_e64 s[4:5], v0, v1", "buffer_load_dwordx4 v177, s[4:7], 0 offen lds"])) == 1


@pytest.mark.skipif(not os.path.exists(_OBJDUMP), reason="needs llvm-objdump")
def test_no_memory_instruction_reads_a_scalar_register_too_early(tmp_path):
    """The compiler keeps the distance for the instructions it makes; those written as text have to keep it themselves."""
    lib = os.path.join(ROOT, "paper_2510_26692_amd", "libkda.so")
    if not os.path.exists(lib):
        pytest.skip("no library: build it first (python -m paper_2510_26692_amd.build)")
    for name, code in _kernel_code(lib, tmp_path, "kda_").items():
        assert early_scalar_reads(code) == [], name
