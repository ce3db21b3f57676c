"""The engine's host code on the CPU: the library's sources are compiled for
the host only and linked with tests/hip_stub.h in place of the HIP runtime
(device memory is host memory, kernels are recorded, an allocation can be
made to fail); tests/host_check.cpp holds the checks."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_16144_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def host_check(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("host_check")
    flags = ["--offload-host-only", "-O1", "-g", "-std=c++17", "-Wno-unused-result", "-Wno-unused-value",
             f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}"]
    sources = [os.path.join(CSRC, "engine.hip"), os.path.join(CSRC, "abi.cpp"),
               os.path.join(ROOT, "tests", "host_check.cpp")]
    jobs = [(s, str(out / (os.path.basename(s) + ".o"))) for s in sources]
    running = [subprocess.Popen([HIPCC] + flags + ["-c", s, "-o", o], stdout=subprocess.PIPE,
                                stderr=subprocess.STDOUT, text=True) for s, o in jobs]
    for p in running:
        text, _ = p.communicate(timeout=300)
        assert p.returncode == 0, text[-4000:]
    exe = str(out / "host_check")
    # (the device code's symbol stays unresolved: nothing reads it)
    subprocess.run(["g++", *(o for _, o in jobs), "-Wl,--unresolved-symbols=ignore-all", "-no-pie", "-lpthread",
                    "-o", exe], check=True, capture_output=True, text=True)
    return exe


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name", ["failed_schedule", "failed_admission", "failed_admission_frees_slots",
                                  "failed_second_phase", "failed_reblocking", "row_limit", "long_rows",
                                  "crowded_slices", "failed_creation", "least_memory_partials",
                                  "least_memory_batch", "server_budget",
                                  "copies_of_row_sums", "launches_of_many"])
def test_host_engine(host_check, name):
    p = subprocess.run([host_check, name], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and p.stdout.strip() == f"ok {name}", p.stdout[-2000:] + p.stderr[-4000:]
