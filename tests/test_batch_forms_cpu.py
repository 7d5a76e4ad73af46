"""The rules by which a batched decode picks its launches and its loads
(csrc/host_plan.h), compiled for the host: the loads follow the bytes that the
arguments allow, whatever the chunk size and the grid, and the bytes follow the
arena and the caller's bound on the codewords without wrapping."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "host_plan.h"
using namespace hm;
constexpr uint64_t MiB = uint64_t(1) << 20, none = ~uint64_t(0);
static_assert(batch_input_bytes(8 * MiB, 0) == 64 * MiB && batch_input_bytes(0, 5) == 0, "the arena");
static_assert(batch_input_bytes(8 * MiB, 1) == 16 && batch_input_bytes(8 * MiB, 4 * MiB - 1) == 64 * MiB - 16, "the bound");
static_assert(batch_input_bytes(8 * MiB, 4 * MiB) == 64 * MiB && batch_input_bytes(8 * MiB, none) == 64 * MiB, "the smaller");
static_assert(batch_input_bytes(none, 0) == none && batch_input_bytes(none, none) == none, "no wrap");
static_assert(batch_input_bytes(none, 1) == 16, "no wrap");
static_assert(batch_reads_cached(64 * MiB) && !batch_reads_cached(64 * MiB + 1) && !batch_reads_cached(none), "loads");
static_assert(batch_form(256, 4096) == BatchForm::one && batch_form(257, 1) == BatchForm::two, "packets");
static_assert(batch_form(256, 4097) == BatchForm::two && batch_form(1024, 16384) == BatchForm::two, "blocks");
static_assert(batch_form(1, 16385) == BatchForm::three && batch_form(1025, 1) == BatchForm::three, "three");
static_assert(batch_form(1, uint64_t(1) << 32) == BatchForm::three && batch_form(1, none) == BatchForm::three, "no wrap");
int main() { return 0; }
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_batch_form_and_load_rules(tmp_path):
    src = tmp_path / "rules.cpp"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_1412_6862_amd", "csrc"),
                           "-o", str(tmp_path / "rules"), str(src)])
