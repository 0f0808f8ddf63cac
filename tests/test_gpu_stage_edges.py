"""GPU parity at the sizes where a stage's kernels change form: labels and halo
tables equal to the oracle's, bit for bit, on the GPU's own densities."""
from __future__ import annotations

import sys

import numpy as np
import pytest

import oracle
from paper_2110_11408_amd import synth
from tests.gpu_helpers import assert_same_labels, density_violations, gpu_find

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    oracle.build(force=False)
    from paper_2110_11408_amd.api import Context
    return Context(0)


def _check(ctx, pos, **kw):
    print(f"[gpu] hf_find n={len(pos)} {kw}", file=sys.stderr, flush=True)
    g = gpu_find(ctx, pos, **kw)
    assert len(density_violations(g["density"], oracle.density(pos, **kw))) == 0
    assert_same_labels(g, oracle.find(pos, density_override=g["density"].astype(np.float64), **kw))
    return g


# The hard cases of the candidate stage are listed in one segment per workgroup
# up to 64 workgroups of 256 particles and in 64 segments beyond; sub-cells per
# cell: 27 (l = 0.25), 64 (0.2), 216 (0.13).
@pytest.mark.parametrize("l_fof", [0.25, 0.2, 0.13])
@pytest.mark.parametrize("n", [200, 256, 257, 2049, 16128, 16385, 30011])
def test_candidate_lists_and_sub_cell_counts(ctx, n, l_fof):
    pos, L, _ = synth.small_box(n, seed=n, nmax=n // 4, halo_frac=0.6, pair_frac=0.3)
    g = _check(ctx, pos, box=L, l_fof=l_fof)
    assert n < 2000 or g["stats"]["n_hard"] >= g["stats"]["n_candidates"] > 0


# FoF: boxes of exactly three cells a side (every cell is the neighbour of every
# other through one offset), mostly sparse cells, l above b, and the finest
# sub-cells (no head start inside a cell).
@pytest.mark.parametrize("n,side,kw", [
    (900, 1.21, {"mean_density": 1.0, "delta_l0_min": 30.0}),
    (700, 6.0, {"mean_density": 1.0, "delta_l0_min": 2.0}),
    (5000, 17.1, {"delta_l0_min": 5.0, "l_fof": 0.6}),
    (20011, 27.15, {"delta_l0_min": 20.0, "l_fof": 0.125}),
    (20011, 27.15, {"delta_l0_min": 0.0, "l_fof": 0.3}),
])
def test_fof_cell_links(ctx, n, side, kw):
    import torch
    from paper_2110_11408_amd import _lib
    if n < 1000:
        rng = np.random.default_rng(n)
        pos = np.concatenate([rng.random((n // 2, 3)) * side,
                              np.abs(rng.normal(0.5 * side, 0.06 * side, (n - n // 2, 3)))]) % side
        pos = np.minimum(pos.astype(np.float32), np.nextafter(np.float32(side), np.float32(0)))
    else:
        pos, _, _ = synth.small_box(n, seed=n, nmax=n // 6, halo_frac=0.6, pair_frac=0.3, side=side)
    print(f"[gpu] hf_l0_fof n={n} side={side} {kw}", file=sys.stderr, flush=True)
    p = _lib.default_params(box=side, **kw)
    t = torch.from_numpy(np.ascontiguousarray(pos)).cuda()
    dens = ctx.density(t, p)
    l0, groups = ctx.l0_fof(t, dens, p)
    ref, _ = oracle.fof(pos, dens.cpu().numpy().astype(np.float64), box=side, **kw)
    np.testing.assert_array_equal(l0.cpu().numpy(), ref)
    assert groups == len(np.unique(ref[ref > 0]))
