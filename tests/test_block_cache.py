"""The context's cache of device blocks, against a stand-in HIP runtime."""
import os
import subprocess

import pytest

from tests.conftest import ROOT

CHECKS = ["reuse", "stream_change", "stream_change_in_capture", "release_without_host_memory",
          "other_context", "exact_size"]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("block_cache") / "check")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-isystem", f"{rocm}/include",
                    "-I", os.path.join(ROOT, "paper_1804_09494_amd", "csrc"),
                    os.path.join(ROOT, "tests", "block_cache_check.cpp"), "-o", out, "-lpthread"], check=True)
    return out


@pytest.mark.parametrize("name", CHECKS)
def test_block_cache(program, name):
    subprocess.run([program, name], check=True, timeout=60)
