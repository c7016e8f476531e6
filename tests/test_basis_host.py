"""The eigenvector adjoint of the reconstruction adjoint kernel on the CPU, against
central differences of the forward basis (tests/host/basis_fd.cpp, compiled with
g++ against a host stand-in of the HIP runtime header)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), 'paper_2608_10569_amd', 'csrc')
CHECKS = ['basis2_vjp_subsonic', 'basis2_vjp_at_rest', 'basis2_vjp_monatomic']


def test_basis_adjoint_matches_finite_differences(tmp_path):
    gxx = shutil.which('g++')
    if gxx is None:
        pytest.skip('g++ not available')
    exe = str(tmp_path / 'basis_fd')
    subprocess.run([gxx, '-O1', '-std=c++17', '-I', os.path.join(HERE, 'host'), '-I', CSRC,
                    os.path.join(HERE, 'host', 'basis_fd.cpp'), '-o', exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    lines = dict((ln.split()[0], ln.split()[2]) for ln in out.stdout.splitlines()
                 if len(ln.split()) == 3)
    assert lines == dict.fromkeys(CHECKS, 'OK') and out.returncode == 0, out.stdout
