"""Compile-time guard for the kernels whose speed hinges on occupancy: the step kernel is tuned
for four waves per SIMD (at most 128 vector registers) and must not spill; one more register
block costs a wave per SIMD and about 6 % of the step time on an MI355X.  The exact threshold's and the
selection's kernels may spill where their comments say so, and nowhere else, the quantizers' not at all.  hipcc cross-compiles
for gfx950 without a GPU, so this runs with the CPU tests."""
import os
import re
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2208_05631_amd", "csrc")


def resource_usage(source):
    import __graft_entry__ as entry
    flags = [f for f in entry.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    with tempfile.TemporaryDirectory() as tmp:
        cmd = ["hipcc", *flags, "--cuda-device-only", "-c", "-I" + os.path.join(ROOT, "include"),
               "-I" + CSRC, os.path.join(CSRC, source), "-o", os.path.join(tmp, "k.o"),
               "-Rpass-analysis=kernel-resource-usage"]
        err = subprocess.run(cmd, check=True, capture_output=True, text=True, cwd=tmp).stderr
    out = {}
    pat = (r"Function Name: (\S+).*?VGPRs: (\d+).*?ScratchSize \[bytes/lane\]: (\d+)"
           r".*?Occupancy \[waves/SIMD\]: (\d+).*?LDS Size \[bytes/block\]: (\d+)")
    for m in re.finditer(pat, err, re.S):
        out[m.group(1)] = dict(vgprs=int(m.group(2)), scratch=int(m.group(3)), waves=int(m.group(4)),
                               lds=int(m.group(5)))
    return out


@pytest.fixture(scope="module")
def step_resources():
    return resource_usage("qa_step.hip")


@pytest.fixture(scope="module")
def step_kernels(step_resources):
    return {k: v for k, v in step_resources.items() if "step_lut_kernel" in k}


def test_no_step_kernel_variant_spills(step_kernels):
    assert len(step_kernels) >= 40                       # every template combination was seen
    spilling = {k: v for k, v in step_kernels.items() if v["scratch"] != 0}
    assert not spilling, spilling


def test_step_kernel_variants_keep_four_waves_per_simd(step_kernels):
    low = {k: v for k, v in step_kernels.items() if v["vgprs"] > 128 or v["waves"] < 4}
    assert not low, low
    # four work-groups per CU must also fit the 160 KiB of LDS
    assert all(v["lds"] <= 40 * 1024 for v in step_kernels.values())


# bytes per lane: the two forms for two work-groups per compute unit, where the work-group that scans spills, and
# the sort of what the levels leave open
EXACT_SPILLS = {"exact_resident_kernelILb1E": 112, "exact_wide_level_kernelILb1E": 64, "exact_sort_open_kernel": 32}


def test_exact_threshold_kernels_spill_only_where_their_comments_say():
    kernels = resource_usage("qa_exact_wide.hip")
    for part in EXACT_SPILLS:
        assert sum(part in k for k in kernels) == 1, part
    for name, v in kernels.items():
        assert v["scratch"] <= max([n for p, n in EXACT_SPILLS.items() if p in name], default=0), (name, v)
        if "ILb1E" in name:
            assert v["waves"] == 8, (name, v)


def test_selection_kernels_do_not_spill_and_reach_the_waves_they_ask_for():
    kernels = resource_usage("qa_select.hip")
    assert len(kernels) >= 20
    assert not {k: v for k, v in kernels.items() if v["scratch"] != 0}
    for part, waves in (("gsel_quantize_multi_kernel", 5), ("quantize_selected_kernel", 4), ("indicator_kernel", 3)):
        found = [v["waves"] for k, v in kernels.items() if part in k and "indicator_or" not in k]
        assert found and all(n == waves for n in found), (part, found)


def test_quantizer_kernels_do_not_spill_and_keep_their_waves():
    """The kernels that hold a bucket use every register that their work-groups' waves leave them."""
    kernels = resource_usage("qa_quantize.hip")
    assert not {k: v for k, v in kernels.items() if v["scratch"] != 0}
    for part, waves in (("quantize_held_kernelILi2E", 8), ("quantize_held_kernelILi4E", 8), ("quantize_held_kernelILi8E", 8),
                        ("quantize_held_kernelILi16E", 4), ("stochastic_held_kernelILi16E", 4), ("quantize_tile_kernelILb0E", 8),
                        ("quantize_bucket_kernelILi8ELb0E", 8), ("quantize_bucket_kernelILi9ELb0E", 7),
                        ("quantize_bucket_kernelILi11ELb0E", 6), ("quantize_bracketed_kernel", 8), ("settle_listed_kernel", 5)):
        found = [v["waves"] for k, v in kernels.items() if part in k]
        assert found and all(n >= waves for n in found), (part, found)


def test_kernels_of_few_tiles_do_not_spill_and_fit_a_compute_unit(step_resources):
    """A work-group is 16 waves: four per SIMD."""
    kernels = {k: v for k, v in step_resources.items() if "step_few_kernel" in k}
    assert len(kernels) >= 9
    assert not {k: v for k, v in kernels.items() if v["scratch"] != 0 or v["waves"] < 4}
