"""Register budgets of the kernels that the pass and decode launch, checked on
the compiler's own resource report (the device assembly's .num_vgpr and
.private_seg_size symbols): none of them may spill to scratch memory, whose
reloads wait for every outstanding load, and each must fit the VGPR budget of
the occupancy it is designed for.  Runs on the CPU (hipcc cross-compiles
gfx950); skipped where hipcc is missing."""
import concurrent.futures
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2608_21541_amd import build as B

# (source, kernel symbol prefix, largest VGPR count)
KERNELS = [
    ("score.hip", "_ZN6certkv17score_mfma_kernelILi128ELi8ELi0E", 128),       # pass 1
    ("score.hip", "_ZN6certkv22score_pass2_w16_kernelILi128ELi8ELb1E", 128),  # pass 2, key sums
    ("score.hip", "_ZN6certkv22score_pass2_w16_kernelILi128ELi8ELb0E", 128),  # pass 2
    ("score.hip", "_ZN6certkv16score_f32_kernelILi64ELb0ELi256E", 128),       # fp32 passes: four
    ("score.hip", "_ZN6certkv16score_f32_kernelILi64ELb1ELi256E", 128),       # waves per SIMD,
    ("score.hip", "_ZN6certkv16score_f32_kernelILi64ELb1ELi64E", 256),        # one-wave blocks: one,
    ("score.hip", "_ZN6certkv16score_f32_kernelILi128ELb0ELi256E", 168),      # rows of 128: three
    ("score.hip", "_ZN6certkv16score_f32_kernelILi128ELb1ELi256E", 168),
    ("score.hip", "_ZN6certkv16score_f32_kernelILi128ELb1ELi64E", 168),
    ("sort.hip", "_ZN6certkv15seg_sort_kernel", 128),
    ("sort.hip", "_ZN6certkv17sort_small_kernel", 64),                        # two workgroups of
    ("sort.hip", "_ZN6certkv19sort_buckets_kernel", 64),                      # 1024 per compute unit
    ("sort.hip", "_ZN6certkv21sort_splitters_kernel", 128),
    ("sort.hip", "_ZN6certkv17sort_count_kernel", 64),
    ("sort.hip", "_ZN6certkv19sort_scatter_kernel", 64),
    ("curves.hip", "_ZN6certkv13curves_kernelILi128ELb1ELi0E", 128),         # centered
    ("curves.hip", "_ZN6certkv13curves_kernelILi128ELb1ELi1E", 128),         # uncentered
    ("curves.hip", "_ZN6certkv13curves_kernelILi128ELb1ELi2E", 128),         # tail mass
    ("curves.hip", "_ZN6certkv13curves_kernelILi64ELb0ELi0E", 128),          # fp32, d = 64
    ("curves.hip", "_ZN6certkv19curve_totals_kernelI", 64),                  # two workgroups of 1024
    ("allocate.hip", "_ZN6certkv23curve_blockstats_kernelILb1ELi8E", 128),
    ("allocate.hip", "_ZN6certkv23curve_blockstats_kernelILb1ELi2E", 64),
    ("allocate.hip", "_ZN6certkv23curve_blockstats_kernelILb0ELi8E", 64),
    ("allocate.hip", "_ZN6certkv17hull_merge_kernel", 128),
    ("allocate.hip", "_ZN6certkv20allocate_hull_kernel", 128),
    ("allocate.hip", "_ZN6certkv15allocate_kernel", 128),
    ("select.hip", "_ZN6certkv13select_kernel", 128),
    ("select.hip", "_ZN6certkv15coverage_kernel", 64),
    ("tail.hip", "_ZN6certkv18tail_gather_kernelI", 128),
    ("tail.hip", "_ZN6certkv20tail_finalize_kernelI", 64),
    ("clusters.hip", "_ZN6certkv19cluster_tail_kernelILi128EtE", 102),       # five waves per SIMD
    # the workgroups per compute unit that decode_parts counts on (not listed: sixteen
    # query tiles, whose 1024 threads have 128 VGPRs and spill)
    ("decode.hip", "_ZN6certkv13decode_kernelILi128ELi1EE", 256),
    ("decode.hip", "_ZN6certkv13decode_kernelILi128ELi2EE", 256),
    ("decode.hip", "_ZN6certkv13decode_kernelILi128ELi4EE", 256),
    ("decode.hip", "_ZN6certkv13decode_kernelILi128ELi8EE", 256),
    ("decode.hip", "_ZN6certkv13decode_kernelILi64ELi1EE", 256),
    ("decode.hip", "_ZN6certkv13decode_kernelILi64ELi2EE", 128),
    ("decode.hip", "_ZN6certkv13decode_kernelILi64ELi4EE", 168),
    ("decode.hip", "_ZN6certkv13decode_kernelILi64ELi8EE", 256),
    ("decode.hip", "_ZN6certkv21decode_combine_kernelI", 64),
    ("decode.hip", "_ZN6certkv26decode_combine_rows_kernelI", 64),
]


def _device_asm(src, out_dir):
    path = os.path.join(out_dir, src + ".s")
    cmd = [B.HIPCC, *[f for f in B.FLAGS if f != "-fPIC"], "--cuda-device-only", "-S",
           os.path.join(B.CSRC, src), "-o", path]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(path) as fh:
        return fh.read()


@pytest.fixture(scope="module")
def asm():
    if not (os.path.exists(B.HIPCC) or shutil.which(B.HIPCC)):
        pytest.skip("hipcc not available")
    srcs = sorted({s for s, _, _ in KERNELS})
    with tempfile.TemporaryDirectory() as d:
        with concurrent.futures.ThreadPoolExecutor(min(len(srcs), 8)) as ex:
            texts = dict(zip(srcs, ex.map(lambda s: _device_asm(s, d), srcs)))
    return texts


def _symbols(text, prefix, field):
    pat = re.compile(r"\.set (" + re.escape(prefix) + r"\w*)\." + field + r", (\d+)")
    return {m.group(1): int(m.group(2)) for m in pat.finditer(text)}


@pytest.mark.parametrize("src,prefix,vmax", KERNELS, ids=[k[1][-40:] for k in KERNELS])
def test_hot_kernels_do_not_spill(asm, src, prefix, vmax):
    scratch = _symbols(asm[src], prefix, "private_seg_size")
    vgprs = _symbols(asm[src], prefix, "num_vgpr")
    assert scratch, f"no kernel {prefix} in {src}"
    for name, n in scratch.items():
        assert n == 0, f"{name} spills {n} bytes per lane"
        assert vgprs[name] <= vmax, f"{name} uses {vgprs[name]} VGPRs (budget {vmax})"
