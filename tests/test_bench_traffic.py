"""bench.py's table of measured bytes covers the tiles the autotuner chooses between
for the headline grid (both reconstruction tiles, fluxes formed in the update), so
that its record always carries the measured rate of the stage pipeline."""

import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


@pytest.mark.parametrize('recon', [16, 32])
def test_both_reconstruction_tiles_have_measured_bytes(recon):
    out = bench.pipeline_hbm(dict(recon=recon, grad=32, flux=0, order=0, xcd=1), 1e9)
    assert out is not None
    # at least what the reconstruction, gradient and update kernels write
    assert 848 + 352 + 160 < out['bytes_per_cell_stage'] < 5000
    assert ('recon', recon) in bench.TRAFFIC_BYTES
