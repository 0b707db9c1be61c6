"""The profile summaries' kernel names against the sources (CPU)."""
import glob
import os
import re

from paper_2604_26823_amd import rocprof_summary

CSRC = os.path.join(rocprof_summary.HERE, "csrc")


def sources():
    return "\n".join(open(p).read() for p in sorted(glob.glob(os.path.join(CSRC, "*.h"))))


def test_scopes_name_kernels_and_timer_scopes_of_the_sources():
    text = sources()
    kernels = set(re.findall(r"\b(k_\w+)\(", text))
    scopes = set(re.findall(r'scope\(\s*"(\w+)"', text)) | {"pm_step"}
    for kernel, scope in rocprof_summary.SCOPES.items():
        assert kernel in kernels, kernel
        assert scope in scopes, scope


def test_both_forms_of_a_launch_have_its_scope():
    s = rocprof_summary.SCOPES
    assert s["k_scatter_ids"] == s["k_scatter_ids_b"] == "sort_scatter_ids"
    assert s["k_x_gather_wide"] == s["k_x_gather"] == "fft_x_gather"
