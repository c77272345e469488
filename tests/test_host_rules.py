"""Index and launch rules of the library's host side, compiled from its headers
without device code: what a kernel may touch, which launches are refused, and
how products are planned, checked on the CPU over whole ranges of sizes."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host_rules") / "host_rules.so")
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-fPIC", "-shared",
                    "-Wno-unused", os.path.join(HERE, "host_rules.cpp"), "-o", out], check=True)
    lib = ctypes.CDLL(out)
    lib.host_staged_reads.restype = ctypes.c_int64
    return lib


@pytest.mark.parametrize("esize", [2, 4])
def test_projection_reads_stay_in_the_staged_rows(rules, esize):
    """The decode projections multiply a 32-row tile whatever the batch; with 4,
    8 or 16 staged rows every fragment read has to come from those rows."""
    wrong = ctypes.c_int64()
    for d in range(64, 4096 // esize + 1, 64):
        for rows in (4, 8, 16, 32):
            past = rules.host_staged_reads(esize, d, rows, ctypes.byref(wrong))
            assert past <= 0 and wrong.value == 0, (d, rows, past, wrong.value)


def test_register_path_refuses_what_it_does_not_know(rules):
    """Batches, column sums and a third operand source exist on the direct
    kernel only: the other one would drop them without a word."""
    assert rules.host_register_path(96, 1, 0, -1)
    assert rules.host_register_path(96, 1, 0, 96)      # the third source starts past the last step
    assert not rules.host_register_path(96, 1, 0, 64)
    assert not rules.host_register_path(96, 2, 0, -1)
    assert not rules.host_register_path(96, 1, 1, -1)


@pytest.mark.parametrize("esize", [2, 4])
def test_append_cuts_do_not_depend_on_the_batch(rules, esize):
    """One block of each of 1 to 64 sequences: every product of the append cuts
    K and joins the slices the same way, which its own rows would not do."""
    out = (ctypes.c_int * 4)()
    own = set()
    for d in (128, 512, 1024, 2048):
        for per_block, k, count in ((8, 8, 1), (1, 8, 1), (16, 4, 1), (256, 4, 1), (1, 1, 2)):
            seen = set()
            for batch in range(1, 65):
                rules.host_row_plan(esize, batch * per_block, d, k * d, 8 * per_block, count, out)
                seen.add(tuple(out))
                rules.host_row_plan(esize, batch * per_block, d, k * d, 0, count, out)
                own.add((d, per_block, k, count) + tuple(out))
            assert len(seen) == 1, (d, per_block, k, count, seen)
    assert len(own) > 4 * 5, "the plan by a product's own rows differs from batch to batch"
