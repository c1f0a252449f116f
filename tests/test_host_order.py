"""Host-side checks of the kernels' index maps, compiled for the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_mask_order_is_the_scans_order(tmp_path):
    exe = tmp_path / "mask_order"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", f"-I{ROOT}/paper_1806_08384_amd/csrc",
                    f"{ROOT}/tests/host/mask_order.cpp", "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.startswith("ok")


def test_batch_ticket_fits_its_place(tmp_path):
    exe = tmp_path / "batch_ticket"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", f"-I{ROOT}/paper_1806_08384_amd/csrc",
                    f"{ROOT}/tests/host/batch_ticket.cpp", "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout


def test_rowid_workspace(tmp_path):
    exe = tmp_path / "rowid_scratch"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{ROOT}/include", f"-I{ROOT}/paper_1806_08384_amd/csrc",
                    f"{ROOT}/tests/host/rowid_scratch.cpp", "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout
