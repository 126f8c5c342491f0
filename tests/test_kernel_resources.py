"""Register and occupancy budgets of the hot kernels, read from the compiler's
resource report for gfx950 (no GPU needed).

The heavy-row numeric pass keeps three workgroups of 512 threads on a compute
unit (its LDS allows three), which takes six wavefronts per SIMD, so at most
80 VGPRs; at 88 only two workgroups fit and the pass runs about 40% longer.
The symbolic pass keeps eight wavefronts per SIMD (64 VGPRs).  The light-row
kernel, whose rows wait on random reads, keeps the wavefronts it declares: six
per SIMD for counts and Jaccard values, five for plus-times, four with 64-bit
sort keys.  The passes over (row, cell) units keep two workgroups per compute
unit, as their walks hide behind each other's output, and the record pass of
the product with one column two of 512 threads.  The mirror's copy and the
sorts keep what their loads in flight were tuned with.  No kernel here spills,
but for 12 bytes per lane of that record pass in f64, which measure faster than
reading the next tile's values later.
"""
import functools
import os
import re
import shutil
import subprocess

import pytest

from paper_2608_09713_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@functools.lru_cache(None)
def _report(src):
    flags = [f for f in build.FLAGS if f not in ("-shared",)]
    cmd = [HIPCC, *flags, "--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage",
           os.path.join(build.CSRC, src), "-o", os.devnull]
    out = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    kernels = {}
    name = None
    for line in out.splitlines():
        m = re.search(r"remark:\s+Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            kernels[name] = {}
            continue
        m = re.search(r"remark:\s+(VGPRs|ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]|LDS Size \[bytes/block\]): "
                      r"(\d+)", line)
        if m and name:
            kernels[name][m.group(1).split()[0] if not m.group(1).startswith("LDS") else "LDS"] = int(m.group(2))
    return kernels


pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC),
                                reason="hipcc not available")


def test_heavy_kernel_budgets():
    ks = {k: v for k, v in _report("heavy.hip").items() if "heavy_kernel" in k}
    assert len(ks) == 16  # four semirings x symbolic/numeric x lower/off-diagonal
    for name, r in ks.items():
        numeric = re.search(r"heavy_kernelILi\dELb1E", name) is not None
        assert r["ScratchSize"] == 0, name
        if numeric:  # three workgroups of eight wavefronts per compute unit (160 KiB of LDS)
            assert r["VGPRs"] <= 80 and r["Occupancy"] >= 6 and 3 * r["LDS"] <= 160 * 1024, (name, r)
        else:  # four
            assert r["VGPRs"] <= 64 and r["Occupancy"] >= 8 and 4 * r["LDS"] <= 160 * 1024, (name, r)


def test_light_kernel_budgets():
    report = _report("light_fused.hip")
    ks = {k: v for k, v in report.items() if "fused_kernel" in k}
    assert len(ks) == 8
    for name, r in ks.items():
        sr, lower = re.search(r"fused_kernelILi(\d)ELb(\d)E", name).groups()
        # (Jaccard off the diagonal has 64-bit keys)
        waves = 5 if sr in "01" else (4 if sr == "3" and lower == "0" else 6)
        assert r["ScratchSize"] == 0 and r["Occupancy"] >= waves, (name, r)
        assert (160 * 1024 // r["LDS"]) * 2 >= 4 * waves, (name, r)  # two wavefronts per workgroup
    wide = {k: v for k, v in report.items() if "fused_wide" in k}
    assert len(wide) == 5  # plus-times lower and off the diagonal, Jaccard lower
    for name, r in wide.items():
        assert r["ScratchSize"] == 0 and r["Occupancy"] >= 4 and (160 * 1024 // r["LDS"]) * 2 >= 16, (name, r)


def test_dense_kernel_budgets():
    ks = _report("dense.hip")
    numeric = {k: v for k, v in ks.items() if "dense_numeric_kernel" in k}
    symbolic = {k: v for k, v in ks.items() if "dense_symbolic_kernel" in k}
    assert len(numeric) == 4 and len(symbolic) == 1
    for name, r in numeric.items():
        assert r["ScratchSize"] == 0 and r["Occupancy"] >= 4 and 2 * r["LDS"] <= 160 * 1024, (name, r)
    for name, r in symbolic.items():
        assert r["ScratchSize"] == 0 and r["Occupancy"] >= 8 and 4 * r["LDS"] <= 160 * 1024, (name, r)


def test_symm_kernel_budgets():
    ks = {k: v for k, v in _report("symm.hip").items() if re.search("split_|symm_|bucket_", k)}
    records = {k: v for k, v in ks.items() if "split_records" in k}
    assert len(records) == 3
    for name, r in ks.items():
        assert r["ScratchSize"] <= (12 if "split_recordsIdd" in name else 0), (name, r)
    for name, r in records.items():
        assert r["Occupancy"] >= 4 and 2 * r["LDS"] <= 160 * 1024, (name, r)


def test_scatter_and_copy_budgets():
    scatter = {k: v for k, v in _report("radix.hip").items() if "radix_scatter" in k or "radix_hist" in k}
    copy = {k: v for k, v in _report("mirror.hip").items() if "copy_lower" in k}
    assert len(scatter) > 10 and len(copy) == 3
    for name, r in scatter.items():
        assert r["ScratchSize"] == 0 and r["Occupancy"] >= 4, (name, r)
    for name, r in copy.items():
        assert r["ScratchSize"] == 0 and r["Occupancy"] >= 5, (name, r)


def test_local_sort_budgets():
    # the packed column sort's first launch holds groups of up to 2048
    # records: at most 18 KiB of LDS and 72 VGPRs, so that seven workgroups
    # of four wavefronts share a compute unit (the second launch, for the
    # rare larger groups, keeps the 4096-record LDS arrays); no spills
    ks = _report("radix.hip")
    small = {k: v for k, v in ks.items() if "local_sort_packILi" in k}
    big = {k: v for k, v in ks.items() if "local_sort_pack_bigILi" in k}
    # f64, f32, count and Jaccard records, and f64 and f32 records that carry
    # the values in place of the entry indices
    assert len(small) == 6 and len(big) == 6
    for name, r in small.items():
        assert r["ScratchSize"] == 0 and r["VGPRs"] <= 72 and r["LDS"] <= 18 * 1024, (name, r)
        assert r["Occupancy"] >= 7 and 7 * r["LDS"] <= 160 * 1024, (name, r)
    for name, r in big.items():
        assert r["ScratchSize"] == 0 and r["LDS"] <= 36 * 1024, (name, r)
