"""The eigenvector adjoint of the reconstruction adjoint kernel on the CPU, against
central differences of the forward basis (tests/host/basis_fd.cpp, compiled with
g++ against a host stand-in of the HIP runtime header); and the same program with a
mistake planted in a copy of that adjoint, which it has to catch."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), 'paper_2608_10569_amd', 'csrc')
CHECKS = ['basis2_vjp_subsonic', 'basis2_vjp_at_rest', 'basis2_vjp_monatomic']
MISTAKES = [('a.a6 += y[3] * x[1];', 'a.a6 -= y[3] * x[1];'),
            ('z[2] = y[2] + e.ut * y[3];', 'z[2] = y[2] + e.un * y[3];'),
            ('g.ut -= Lb[0];', 'g.ut += Lb[0];'),
            ('g.ic += 0.5 * sg * (Lb[1] - e.un * Lb[0]);', 'g.ic += 0.5 * sg * Lb[1];'),
            ('g.c -= e.ic * e.ic * g.ic;', 'g.c -= e.ic * g.ic;'),
            ('irb += mn * g.un + mt * g.ut;', 'irb += mn * g.un;'),
            ('ub[3] += ir * a5 + K.gm1 * pb;', 'ub[3] += K.gm1 * pb;')]


def run(tmp, include):
    gxx = shutil.which('g++')
    if gxx is None:
        pytest.skip('g++ not available')
    exe = os.path.join(str(tmp), 'basis_fd')
    subprocess.run([gxx, '-O1', '-std=c++17', '-I', os.path.join(HERE, 'host')] +
                   [a for d in include for a in ('-I', d)] +
                   [os.path.join(HERE, 'host', 'basis_fd.cpp'), '-o', exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    lines = dict((ln.split()[0], ln.split()[2]) for ln in out.stdout.splitlines()
                 if len(ln.split()) == 3)
    return out, lines


def test_basis_adjoint_matches_finite_differences(tmp_path):
    out, lines = run(tmp_path, [CSRC])
    assert lines == dict.fromkeys(CHECKS, 'OK') and out.returncode == 0, out.stdout


@pytest.mark.parametrize('right,wrong', MISTAKES)
def test_planted_mistake_is_caught(tmp_path, right, wrong):
    with open(os.path.join(CSRC, 'hweno_basis2.h')) as f:
        text = f.read()
    assert text.count(right) == 1
    with open(tmp_path / 'hweno_basis2.h', 'w') as f:
        f.write(text.replace(right, wrong))
    out, _ = run(tmp_path, [str(tmp_path), CSRC])
    assert out.returncode == 1, out.stdout
