"""The quantised neighbour scan on the CPU: within its arrays, and every neighbour once."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1108_4214_amd", "csrc")


def test_quantised_scan_reads_its_arrays_and_visits_every_neighbour_once(tmp_path):
    """cell_scan.h compiled for the host with its reads checked: from a lone bead to crowded cells, three to nine cells
    per edge, beads at the end of the list and around the corner, one and four threads per bead."""
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text("#pragma once\n")   # the program brings what it needs of it
    exe = str(tmp_path / "scan")
    subprocess.run(["/opt/rocm/llvm/bin/clang++", "-std=c++17", "-O1", "-w", "-ffp-contract=off",
                    "-fsanitize=float-cast-overflow", "-fsanitize-trap=all", "-I", str(tmp_path), "-I", CSRC,
                    os.path.join(HERE, "scan_host.cpp"), "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, (run.returncode, run.stdout)
