"""Tiles that tag what they publish (csrc/tns_chain.h), built for the host: workgroups as fibers, their accesses to memory in
many (seeded) orders, workgroups that start late among them.  No GPU."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2311_17410_amd", "csrc")


def test_rows_of_every_tile_in_many_orders(tmp_path):
    exe = str(tmp_path / "tile_chain")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-U_FORTIFY_SOURCE", "-Wno-unknown-pragmas", "-I", os.path.join(HERE, "host_hip"), "-I", CSRC,
                           os.path.join(HERE, "tile_chain_host.cpp"), "-o", exe])
    done = subprocess.run([exe, "3000", "1500"], capture_output=True, text=True, timeout=300)
    assert done.returncode == 0, done.stdout + done.stderr
