"""Compile-time properties the launch configurations rely on (no GPU needed): the projection
kernels must not spill to scratch, and the shapes that are meant to run two workgroups per CU
must leave room for them (registers per wave, both register files counted)."""
import ctypes
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_09244_amd.build import FLAGS   # (what ships is what is looked at)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_09244_amd", "csrc")
PROJECTION_KERNEL = "_ZN4mvla(?:11gemm|17small_tile)_kernelI"


def _resource_usage(src):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    cmd = [hipcc, *FLAGS, "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-c",
           os.path.join(CSRC, src), "-o", os.devnull, "-Rpass-analysis=kernel-resource-usage"]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert out.returncode == 0, out.stderr[-2000:]
    kernels, cur = {}, None
    for line in out.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = kernels.setdefault(m.group(1), {})
            continue
        m = re.search(r"remark:\s+([A-Za-z ]+?)(?: \[[^\]]*\])?: (\d+)", line)
        if m and cur is not None:
            cur[m.group(1).strip()] = int(m.group(2))
    return kernels


def test_projection_kernels_fit_their_launch_shapes():
    k = _resource_usage("gemm.hip")
    gemm = {n: v for n, v in k.items() if "gemm_kernel" in n or "small_tile_kernel" in n}
    assert len(gemm) == 48                                   # 12 tile shapes x 4 epilogues
    for name, v in gemm.items():
        assert v["ScratchSize"] == 0, (name, v)              # (a spill reload in the main loop
        four_wave_big = ("ILi256ELi256ELi64ELi2ELi2ELi2E" in name    # would also wait on the loads)
                         or "ILi288ELi192ELi64ELi2ELi2ELi2E" in name)
        assert v["Occupancy"] >= (1 if four_wave_big else 2), (name, v)
        if four_wave_big:                                    # accumulators in the second file
            assert v["AGPRs"] >= 240 and v["VGPRs"] <= 256, (name, v)
    # 128x128 on four waves with two stages is launched two workgroups per CU
    two_per_cu = [v for n, v in gemm.items() if "ILi128ELi128ELi64ELi2ELi2ELi2E" in n]
    assert len(two_per_cu) == 4
    for v in two_per_cu:
        assert v["VGPRs"] + v["AGPRs"] <= 256, v


def test_attention_kernel_keeps_two_workgroups_per_cu():
    k = _resource_usage("attention.hip")
    att = {n: v for n, v in k.items() if "attention_kernel" in n}
    assert att
    for name, v in att.items():
        assert v["ScratchSize"] == 0 and v["Occupancy"] >= 2, (name, v)


def _device_assembly(src, tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out_s = os.path.join(str(tmp_path), src + ".s")
    cmd = [hipcc, *FLAGS, "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-S",
           "--cuda-device-only", os.path.join(CSRC, src), "-o", out_s]
    out = subprocess.run(cmd, capture_output=True, text=True, timeout=900)
    assert out.returncode == 0, out.stderr[-2000:]
    return open(out_s).read().split("\n")


def _waits_among_mfmas(lines, kernel_prefix):
    """Per kernel: the compiler's own `s_waitcnt vmcnt` (not those written in inline asm) that
    stand between the first and the last MFMA instruction."""
    starts = [i for i, l in enumerate(lines) if re.match(r"^%s.*:\s*(;.*)?$" % kernel_prefix, l)]
    found = {}
    for a, b in zip(starts, starts[1:] + [len(lines)]):
        seg = lines[a:b]
        end = next((i for i, l in enumerate(seg) if "s_endpgm" in l), len(seg))
        seg = seg[:end]
        mf = [i for i, l in enumerate(seg) if "v_mfma" in l]
        if not mf:
            continue
        in_asm, waits = False, []
        for i, l in enumerate(seg):
            if "ASMSTART" in l:
                in_asm = True
            elif "ASMEND" in l:
                in_asm = False
            elif not in_asm and "s_waitcnt" in l and "vmcnt" in l and mf[0] <= i <= mf[-1]:
                waits.append(l.strip())
        found[lines[a].rstrip(":")] = waits
    return found


def _waits_in_innermost_mfma_loops(lines, kernel_prefix):
    """Per kernel: the compiler's own vmcnt waits inside the innermost loops that hold MFMA
    instructions (label ... backward branch, no loop inside), wherever in the loop they stand."""
    starts = [i for i, l in enumerate(lines) if re.match(r"^%s.*:" % kernel_prefix, l)]
    found, n_loops = {}, 0
    for a0, b0 in zip(starts, starts[1:] + [len(lines)]):
        k = lines[a0:b0]
        k = k[:next((i for i, l in enumerate(k) if "s_endpgm" in l), len(k))]
        labels = {m.group(1): i for i, l in enumerate(k)
                  for m in [re.match(r"^(\.LBB\d+_\d+):", l)] if m}
        loops = []
        for i, l in enumerate(k):
            m = re.search(r"s_c?branch\w* (\.LBB\d+_\d+)", l)
            if m and m.group(1) in labels and labels[m.group(1)] < i:
                loops.append((labels[m.group(1)], i))
        for a, b in loops:
            if any(a2 >= a and b2 <= b and (a2, b2) != (a, b) for a2, b2 in loops):
                continue
            body = k[a:b]
            if sum("v_mfma" in x for x in body) < 8:
                continue
            n_loops += 1
            in_asm, waits = False, []
            for x in body:
                if "ASMSTART" in x:
                    in_asm = True
                elif "ASMEND" in x:
                    in_asm = False
                elif not in_asm and "s_waitcnt" in x and "vmcnt" in x:
                    waits.append(x.strip())
            if waits:
                found[lines[a0].split(":")[0]] = waits
    return found, n_loops


def test_no_compiler_vmcnt_wait_inside_the_projection_main_loops(tmp_path):
    """A wait at the head of the main loop (for loads or stores of a previous tile's epilogue
    that the compiler still counts) stands before the loop's first MFMA in program order, yet
    runs every iteration and waits for the direct loads just issued.  The kernel clears the
    compiler's count once per tile; no main loop of any configuration may hold such a wait."""
    found, n_loops = _waits_in_innermost_mfma_loops(_device_assembly("gemm.hip", tmp_path),
                                                    PROJECTION_KERNEL)
    assert n_loops == 48
    assert not found, found


@pytest.mark.parametrize("src,prefix,n_kernels", [("gemm.hip", PROJECTION_KERNEL, 48),
                                                  ("attention.hip", "_ZN4mvla16attention_kernelI", 2)])
def test_no_compiler_wait_catches_the_direct_loads(src, prefix, n_kernels, tmp_path):
    """The global->LDS loads are issued from inline asm and waited for explicitly.  A wait the
    compiler adds for one of ITS loads (a spill reload, an operand fetched before the loop) counts
    every outstanding load, so inside the MFMA loops it would also wait for the direct loads of
    the next tile: there must be none between the first and the last MFMA of a kernel."""
    found = _waits_among_mfmas(_device_assembly(src, tmp_path), prefix)
    assert len(found) == n_kernels, sorted(found)
    for name, waits in found.items():
        assert not waits, (name, waits)


def _innermost_loops(lines, kernel_prefix):
    """Per kernel: the instructions of its innermost loops (label ... backward branch)."""
    starts = [i for i, l in enumerate(lines) if re.match(r"^%s.*:" % kernel_prefix, l)]
    found = {}
    for a0, b0 in zip(starts, starts[1:] + [len(lines)]):
        k = lines[a0:b0]
        k = k[:next((i for i, l in enumerate(k) if "s_endpgm" in l), len(k))]
        labels = {m.group(1): i for i, l in enumerate(k) for m in [re.match(r"^(\.LBB\d+_\d+):", l)] if m}
        loops = [(labels[m.group(1)], i) for i, l in enumerate(k)
                 for m in [re.search(r"s_c?branch\w* (\.LBB\d+_\d+)", l)] if m and labels.get(m.group(1), i) < i]
        inner = [(a, b) for a, b in loops if not any(a2 >= a and b2 <= b and (a2, b2) != (a, b) for a2, b2 in loops)]
        found[lines[a0].split(":")[0]] = [k[a:b + 1] for a, b in inner]
    return found


def test_clustering_loop_takes_one_lds_round_trip_a_patch(tmp_path):
    """The Lloyd loop of the candidate masks runs once per patch of a thread and iteration: a patch's
    score and label are read together (nothing waits in between) and nothing in the loop branches, so a
    sample of many patches is bound by one LDS round trip a patch, not by two and a branch."""
    (bodies,) = _innermost_loops(_device_assembly("mask_kernels.hip", tmp_path), "_ZN4mvla16candidate_kernel").values()
    lloyd = [b for b in bodies if any("ds_read_u8" in x for x in b) and any("ds_write_b8" in x for x in b)]
    assert len(lloyd) == 1
    body = lloyd[0]
    first_wait = next(i for i, x in enumerate(body) if "s_waitcnt" in x)
    reads = [i for i, x in enumerate(body) if "ds_read" in x]
    assert len(reads) == 2 and max(reads) < first_wait, body
    assert sum("branch" in x for x in body) == 1, body


def test_salience_loops_load_in_batches(tmp_path):
    """Rows and partial sums of the salience kernels go out eight loads at a time; what is left over is a
    shorter batch behind the loop.  A loop that takes one load a turn waits a memory round trip for each."""
    kernels = _innermost_loops(_device_assembly("prune_kernels.hip", tmp_path), "_ZN4mvla15salience_kernelILi4E")
    assert len(kernels) == 2                                  # plain and fused
    for name, loops in kernels.items():
        for what in (r"global_load_dwordx4", r"global_load_dword .* sc1"):
            counts = [n for n in (sum(bool(re.search(what, x)) for x in b) for b in loops) if n]
            assert counts and min(counts) >= 8, (name, what, counts)


def test_decomposition_workgroups_fit_their_rows(tmp_path):
    """Per-patch decomposition: four, eight and sixteen waves for up to 256, 512 and more rows (sixteen for
    a handful of rows spend their time on reductions of nothing), none of them spilling."""
    k = {n: v for n, v in _resource_usage("prune_kernels.hip").items() if "decompose_kernel" in n}
    assert {int(re.search(r"decompose_kernelILi(\d+)E", n).group(1)) for n in k} == {256, 512, 1024}
    for name, v in k.items():
        assert v["ScratchSize"] == 0, (name, v)


def test_scoring_rings_leave_room_for_a_second_workgroup():
    """Key rings of score_probs_rows16_kernel (waves x blocks ahead x 16 rows of 128 values, as its launch spells them) for
    rows of up to 1024 keys: one that takes most of a compute unit's 160 KiB of LDS halves what is resident, and a
    launch of more workgroups than compute units takes up to 1.5 times as long."""
    src = open(os.path.join(CSRC, "layer_kernels.hip")).read()
    src = src[src.index("static int launch_score_rows16("):]
    src = src[:src.index("#undef MVLA_SCR")]
    assert "lds = NW * AHEAD * 16 * DH * 2;" in src
    rings = re.findall(r"MVLA_SCR\((\d+), (\d+), \(?(?:DH == 128 \? )?(\d+)(?: : \d+\))?\);", src)
    assert len(rings) == src.count("MVLA_SCR(") - 1
    for waves, blocks, ahead in ((int(a), int(b), int(c)) for a, b, c in rings):
        if waves * blocks * 16 <= 1024:
            assert 2 * waves * ahead * 16 * 128 * 2 <= 160 * 1024 - 2 * 4096, (waves, blocks, ahead)


def test_scoring_tiles_that_one_grid_axis_cannot_hold():
    """Workgroups of 512 threads on one grid axis: fewer than 2^32 threads.  Beyond, 32 queries a workgroup take the
    launch (three axes); one tile of queries has an axis for the heads and one for the samples."""
    from paper_2604_09244_amd import binding as mv
    tile = getattr(mv.load(), "_ZN4mvla18score_tile_queriesEiiiib")
    tile.argtypes, tile.restype = [ctypes.c_int] * 4 + [ctypes.c_bool], ctypes.c_int
    assert tile(65535, 64, 17, 17, False) == 16              # 2^23 - 128 workgroups
    assert tile(65535, 65, 17, 17, False) == 32
    assert tile(1 << 16, 128, 16, 16, False) == 32           # (more samples than the second axis holds)
    assert tile(65535, 128, 16, 16, False) == tile(65535, 128, 300, 16, True) == 16


def test_no_compiler_wait_behind_the_first_key_block_of_the_scoring_rings(tmp_path):
    """score_probs_rows16_kernel: the query fragments are the compiler's own loads, asked for ahead of the ring, so its waits
    for them (at the first block of keys) count the ring too.  From the second block on a wait of its own would drain the
    ring once per block: there must be none."""
    lines = _device_assembly("layer_kernels.hip", tmp_path)
    starts = [i for i, l in enumerate(lines) if re.match(r"^_ZN4mvla25score_probs_rows16_kernelI.*:", l)]
    assert len(starts) == 20                                  # 5 row lengths x 2 head sizes x 2 outputs
    for a, b in zip(starts, starts[1:] + [len(lines)]):
        dh, blocks = (int(x) for x in re.search(r"ILi(\d+)ELi8ELi(\d+)E", lines[a]).groups())
        seg = lines[a:b]
        seg = seg[:next(i for i, l in enumerate(seg) if "s_endpgm" in l)]
        products = [i for i, l in enumerate(seg) if "v_mfma" in l]
        assert len(products) == blocks * dh // 32 and sum("global_load_lds" in l for l in seg) == blocks * dh // 32
        in_asm, waits = False, []
        for l in seg[products[dh // 32 - 1] + 1:products[-1]]:
            if "ASMSTART" in l:
                in_asm = True
            elif "ASMEND" in l:
                in_asm = False
            elif not in_asm and "s_waitcnt" in l and "vmcnt" in l:
                waits.append(l.strip())
        assert not waits, (lines[a], waits)
