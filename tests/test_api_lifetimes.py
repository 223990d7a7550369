"""The C ABI's host side, built for the CPU against a model of the HIP calls it
makes (hip_model/), under AddressSanitizer and UBSan: what it keeps, hands out
and releases over many contexts, batches and threads.  The model faults on a
release of anything that work in flight may still use."""
import os
import subprocess

import pytest

from conftest import ROOT

HERE = os.path.join(ROOT, "tests", "hip_model")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("hip_model") / "api_lifetimes")
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", HERE, "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2111_14240_amd", "csrc"),
                    os.path.join(HERE, "api_lifetimes.cpp"), "-o", exe, "-lpthread"], check=True, timeout=300)
    return exe


@pytest.mark.parametrize("what", ["slots", "batches", "cover", "captured", "no_memory"])
def test_lifetimes(model, what):
    out = subprocess.run([model, what], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stderr[-3000:]
