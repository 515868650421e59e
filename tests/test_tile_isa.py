"""Host-side check of the generated gfx950 code of the tile kernels (no GPU needed; compiles to assembly).

The tile kernels load X straight into LDS and end every pipeline stage with an explicit wait on the load counter
followed by a plain barrier instruction.  That wait is only right if, in the instruction stream the compiler finally
emits, (1) the direct-to-LDS loads of a stage precede all of the stage's other loads, (2) the wait allows at most as
many outstanding loads as were issued between them and the wait, and (3) the wave's own LDS reads are waited for before
the barrier.  A violation would be a data race that a parity test may or may not catch.
"""
import concurrent.futures
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_15601_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
UNITS = {"tm_w4_tile_small": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
         "tm_w4_tile_kgroup": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
         "tm_w4_tile_grouped": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
         "tm_w4_tile_w8": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
         "tm_w4_tile_large": [],
         "tm_w4_tile32": []}
# barrier-terminated regions with direct-to-LDS loads that a unit has at least (a prologue and the unrolled stages of every body)
REGIONS = {"tm_w4_tile_small": 300, "tm_w4_tile_kgroup": 560, "tm_w4_tile_grouped": 420, "tm_w4_tile_w8": 360,
           "tm_w4_tile_large": 36, "tm_w4_tile32": 40}
KERNEL = r"_ZN4tmw4[^\n]*tile(?:32|_grouped)?_kernel[^\n]*"
VMCNT_MAX = 63          # six-bit counter: a wave cannot have more loads outstanding, so a larger bound is no wait at all


def _assembly(unit, extra, outdir):
    out = os.path.join(outdir, unit + ".s")
    cmd = [HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", *extra, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-S", "--cuda-device-only",
           os.path.join(CSRC, unit + ".hip"), "-o", out]
    subprocess.run(cmd, check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    return open(out).read()


def _stage_regions(text):
    """(kernel name, instructions of one barrier-terminated region) for every region that loads into LDS."""
    for m in re.finditer(rf"^({KERNEL}):\s*;[^\n]*\n(.*?)^\.Lfunc_end", text, re.S | re.M):
        region = []
        for line in m.group(2).splitlines():
            t = line.strip()
            if not t or t[0] in ";.":
                continue
            region.append(t)
            if t.startswith("s_barrier"):
                if any(x.startswith("buffer_load") and x.endswith("lds") for x in region):
                    yield m.group(1), region
                region = []


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """Unit -> its assembly."""
    if shutil.which(HIPCC) is None:
        pytest.skip("hipcc not available")
    outdir = str(tmp_path_factory.mktemp("isa"))
    with concurrent.futures.ThreadPoolExecutor(max_workers=3) as pool:
        return dict(zip(UNITS, pool.map(lambda kv: _assembly(kv[0], kv[1], outdir), UNITS.items())))


def test_stage_end_wait_covers_the_direct_to_lds_loads(assembly):
    assert set(assembly) == set(REGIONS)
    for unit, text in assembly.items():
        checked = dict.fromkeys(re.findall(rf"^({KERNEL}):\s*;", text, re.M), 0)
        for name, reg in _stage_regions(text):
            is_load = [t.startswith("buffer_load") for t in reg]
            is_lds = [ld and t.endswith("lds") for ld, t in zip(is_load, reg)]
            first, last = is_lds.index(True), len(reg) - 1 - is_lds[::-1].index(True)
            assert not any(is_load[i] and not is_lds[i] for i in range(first, last)), (name, "loads interleaved")
            # (a) the direct-to-LDS loads have landed before the barrier: some wait after the last of them leaves at
            #     most as many loads outstanding as were issued between that load and the wait (the counter retires
            #     in order); a wait without a vmcnt field only counts where 63 or more loads separate them
            covered = False
            for i in range(last + 1, len(reg)):
                if not reg[i].startswith("s_waitcnt"):
                    continue
                younger = sum(1 for k in range(last + 1, i) if is_load[k])
                m = re.search(r"vmcnt\((\d+)\)", reg[i])
                if (m and int(m.group(1)) <= younger) or (not m and "lgkmcnt" in reg[i] and younger >= VMCNT_MAX):
                    covered = True
            assert covered, (name, "no wait covers the direct-to-LDS loads before the barrier")
            # (b) this wave's own LDS reads are done before it lets others overwrite the buffer
            ds = [i for i, t in enumerate(reg) if t.startswith("ds_read")]
            if ds:
                assert any(t.startswith("s_waitcnt") and "lgkmcnt(0)" in t for t in reg[ds[-1] + 1:]), (name, "LDS reads")
            checked[name] += 1
        # every kernel has a prologue and PD*(PD+1) >= 2 unrolled stages
        assert min(checked.values()) >= 3 and sum(checked.values()) >= REGIONS[unit], (unit, checked)


def test_no_load_is_counted_that_nothing_uses(assembly):
    """The 32-row grouped FP8 kernels multiply exact codes and scale the sums of a group by quads of words: a load of the single
    words that other conversions take would have no use, and the compiler would be free to drop it from under the waits that count it."""
    body = re.compile(r"^_ZN4tmw4[^\n]*tile_grouped_kernelILi2E[^\n]*Li18EE[^\n]*:\s*;[^\n]*\n(.*?)^\.Lfunc_end", re.S | re.M)
    texts = body.findall(assembly["tm_w4_tile_grouped"])
    assert len(texts) == 3 and all(t.count("buffer_load_dwordx4") > 0 for t in texts)
    assert not any(re.search(r"^\s*buffer_load_dword v", t, re.M) for t in texts)


def test_registers_of_the_64_row_grouped_tiles(assembly):
    """Several bodies in one kernel must not cost a resident CTA: 128 registers are four waves per SIMD, 168 three (of 512, in steps
    of 8), nothing is spilled, and the fourth CTA's X buffers fit the 160 KiB of LDS."""
    found = 0
    for m in re.finditer(r"\.group_segment_fixed_size: (\d+)\n(?:(?!\.group_segment_fixed_size).)*?\.symbol:\s+(\S*tile_grouped_kernelILi4E\S*)\.kd"
                         r"(?:(?!\.group_segment_fixed_size).)*?\.vgpr_count:\s+(\d+)\n\s+\.vgpr_spill_count: (\d+)",
                         assembly["tm_w4_tile_grouped"], re.S):
        lds, name, vgprs, spilled = int(m.group(1)), m.group(2), int(m.group(3)), int(m.group(4))
        four = "Li1ELi4ELi4EE" in name               # 4-bit codes in groups of 128
        assert spilled == 0 and 512 // (-(-vgprs // 8) * 8) >= (4 if four else 3) and 4 * lds <= 160 * 1024, (name, vgprs, spilled, lds)
        found += 1
    assert found == 9
