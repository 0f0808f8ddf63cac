"""GPU parity: the HIP path (through the C ABI) against the FP64 oracle.

Bars:
  * density: |D_gpu - D_64| <= 1e-5 * max(D_64, 1) for every particle;
  * labels: bit-exact L0 ids, halo ids and halo table when the oracle is run on
    the GPU's float32 densities (every label predicate is the same FP64
    expression on both sides);
  * against the oracle's own FP64 densities: >= 99.99% matched-label agreement.
Sizes span many 256-thread tiles with ragged tails; the 64^3 box is the small
benchmark workload, and the 256^3 box (the benchmark box) is checked on sampled
densities and on sampled L0 groups.
"""
from __future__ import annotations

import sys

import numpy as np
import pytest

import oracle
from paper_2110_11408_amd import synth
from tests.gpu_helpers import (DENS_REL, assert_same_labels, density_violations,
                               explained_mismatches, gpu_find, matched_agreement)

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def ctx():
    oracle.build(force=False)
    from paper_2110_11408_amd.api import Context
    return Context(0)


def _case(name):
    if name == "plain64":
        return synth.named_box("plain64")
    n, seed, nmax, pf = {"s3000": (3000, 101, 500, 0.3), "s9001": (9001, 102, 1500, 0.3),
                         "s40123": (40123, 103, 5000, 0.2)}[name]
    return synth.small_box(n, seed=seed, nmax=nmax, pair_frac=pf)


CASES = ["s3000", "s9001", "s40123", "plain64"]


@pytest.fixture(scope="module")
def runs(ctx):
    out = {}
    for name in CASES:
        pos, L, _ = _case(name)
        _say(f"[gpu] hf_find case={name} n={len(pos)} box={L:.3f}")
        out[name] = (pos, L, gpu_find(ctx, pos, box=L))
    return out


@pytest.mark.parametrize("name", CASES)
def test_density_within_tolerance(runs, name):
    pos, L, g = runs[name]
    ref = oracle.density(pos, box=L)
    bad = density_violations(g["density"], ref)
    assert len(bad) == 0, (name, len(bad), bad[:5], g["density"][bad[:5]], ref[bad[:5]])


@pytest.mark.parametrize("name", CASES)
def test_labels_bit_exact_given_gpu_density(runs, name):
    pos, L, g = runs[name]
    ref = oracle.find(pos, box=L, density_override=g["density"].astype(np.float64))
    assert_same_labels(g, ref)
    t = g["table"]
    if g["n_halos"]:
        np.testing.assert_array_equal(t["x"], pos[t["nucleus"], 0])
        np.testing.assert_array_equal(t["z"], pos[t["nucleus"], 2])
        K = oracle.derive(len(pos), box=L)["K"]
        np.testing.assert_allclose(t["r"], (t["n_enclosed"] / K) ** (1 / 3), rtol=1e-6)
        np.testing.assert_array_equal(t["mass"], t["n"].astype(np.float32))
    assert g["stats"]["n_halos"] == g["n_halos"]


@pytest.mark.parametrize("name", ["s40123", "plain64"])
def test_fp64_density_label_agreement(runs, name):
    """Against the oracle's FP64 densities: >= 99.99% matched-label agreement,
    and every mismatched particle is explained by a near-threshold event of the
    FP64 field (the L0 cut, the floor, the peak test or the order of nuclei,
    within the density tolerance the GPU field is held to)."""
    pos, L, g = runs[name]
    ref = oracle.find(pos, box=L)
    ev = oracle.events(pos, ref["density"], ref["l0"], tol=DENS_REL, box=L)
    for key in ("l0", "halo_id"):
        frac, bad = matched_agreement(g[key], ref[key])
        assert frac >= 0.9999, (key, frac, len(bad))
        ok = explained_mismatches(bad, g["l0"], ref["l0"], ev)
        assert ok.all(), (key, len(bad), bad[~ok][:10])


def test_split_entry_points_match_find(ctx, runs):
    import torch
    from paper_2110_11408_amd import _lib
    from paper_2110_11408_amd.api import halo_table
    pos, L, g = runs["s40123"]
    p = _lib.default_params(box=L)
    t = torch.from_numpy(pos).cuda()
    _say("[gpu] split entry points s40123")
    dens = ctx.density(t, p)
    l0, ng = ctx.l0_fof(t, dens, p)
    res = ctx.compaso(t, dens, l0, p)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(dens.cpu().numpy(), g["density"])
    np.testing.assert_array_equal(l0.cpu().numpy(), g["l0"])
    np.testing.assert_array_equal(res["halo_id"].cpu().numpy(), g["halo_id"])
    assert res["n_halos"] == g["n_halos"]
    tab = halo_table(res["halos"])
    np.testing.assert_array_equal(tab["id"], g["table"]["id"])
    ref_l0, ref_ng = oracle.fof(pos, g["density"].astype(np.float64), box=L)
    assert ng == ref_ng


def test_compaso_on_external_labels(ctx):
    """hf_compaso with labels and densities that did not come from the GPU:
    the oracle's FP64 field rounded to float32 and its L0 labels."""
    import torch
    from paper_2110_11408_amd import _lib
    pos, L, _ = _case("s9001")
    d64 = oracle.density(pos, box=L)
    d32 = d64.astype(np.float32)
    l0, _ = oracle.fof(pos, d32.astype(np.float64), box=L)
    ref = oracle.compaso(pos, d32.astype(np.float64), l0, box=L)
    p = _lib.default_params(box=L)
    _say("[gpu] hf_compaso external labels s9001")
    res = ctx.compaso(torch.from_numpy(pos).cuda(), torch.from_numpy(d32).cuda(),
                      torch.from_numpy(l0).cuda(), p)
    np.testing.assert_array_equal(res["halo_id"].cpu().numpy(), ref["halo_id"])
    assert res["n_halos"] == ref["n_halos"]


def test_run_to_run_determinism(ctx, runs):
    pos, L, g = runs["plain64"]
    _say("[gpu] determinism plain64")
    g2 = gpu_find(ctx, pos, box=L)
    for k in ("density", "l0", "halo_id"):
        np.testing.assert_array_equal(g2[k], g[k])


@pytest.mark.parametrize("want_density,want_l0", [(True, False), (False, True), (False, False)])
def test_optional_outputs(ctx, runs, want_density, want_l0):
    """The outputs a call asks for are those of the full call, whichever of
    the density and L0 arrays it leaves out (the output stage takes a
    different path when only the halo labels are wanted)."""
    import torch
    from paper_2110_11408_amd import _lib
    pos, L, g = runs["s40123"]
    _say(f"[gpu] optional outputs s40123 density={want_density} l0={want_l0}")
    out = ctx.find(torch.from_numpy(pos).cuda(), _lib.default_params(box=L), want_density=want_density,
                   want_l0=want_l0)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out["halo_id"].cpu().numpy(), g["halo_id"])
    assert out["n_halos"] == g["n_halos"]
    if want_density:
        np.testing.assert_array_equal(out["density"].cpu().numpy(), g["density"])
    else:
        assert out["density"] is None
    if want_l0:
        np.testing.assert_array_equal(out["l0_id"].cpu().numpy(), g["l0"])
    else:
        assert out["l0_id"] is None


def test_params_variants(ctx):
    """Non-default parameters (z = 0.5 thresholds of Table 1 scaled as the paper
    does, other alpha / c_Roche / kernel radius, a linking length above the
    kernel radius) stay bit-exact."""
    pos, L, _ = _case("s9001")
    for kw in (dict(delta_l0_min=77.5, delta_l1=258.2), dict(alpha_elig=0.7, c_roche=1.5),
               dict(b_kernel=0.5, l_fof=0.3, n_l1_min=20), dict(self_count=1),
               # l > b: cells wider than b (larger terms in the density's
               # matrix-core form)
               dict(b_kernel=0.3, l_fof=0.5)):
        _say(f"[gpu] params {kw}")
        g = gpu_find(ctx, pos, box=L, **kw)
        ref = oracle.find(pos, box=L, density_override=g["density"].astype(np.float64), **kw)
        assert_same_labels(g, ref)
        bad = density_violations(g["density"], oracle.density(pos, box=L, **kw))
        assert len(bad) == 0, kw


def test_edge_cases(ctx):
    import torch
    from paper_2110_11408_amd import _lib
    from paper_2110_11408_amd._lib import HfError
    # empty input
    _say("[gpu] edge: empty")
    res = ctx.find(torch.zeros((0, 3), dtype=torch.float32, device="cuda"),
                   _lib.default_params(box=10.0))
    assert res["n_halos"] == 0
    # one particle
    _say("[gpu] edge: one particle")
    one = np.array([[1.0, 2.0, 3.0]], np.float32)
    g = gpu_find(ctx, one, box=5.0, mean_density=1.0)
    assert g["density"][0] == 0.0 and g["n_halos"] == 0 and g["l0"][0] == 0
    # one particle alone sets l_mean = box, so b spans more than a third of the box
    with pytest.raises(HfError):
        gpu_find(ctx, one, box=5.0)
    # nothing above the L0 threshold
    _say("[gpu] edge: sparse")
    rng = np.random.default_rng(3)
    sparse = (rng.random((5000, 3)) * 40).astype(np.float32)
    g = gpu_find(ctx, sparse, box=40.0)
    assert g["n_halos"] == 0 and np.all(g["l0"] == 0)
    # coincident particles: equal densities, ties by index
    _say("[gpu] edge: coincident")
    same = np.tile(np.array([[5.0, 5.0, 5.0]], np.float32), (50, 1))
    g = gpu_find(ctx, same, box=10.0, mean_density=1.0)
    ref = oracle.find(same, box=10.0, mean_density=1.0,
                      density_override=g["density"].astype(np.float64))
    assert_same_labels(g, ref)
    assert g["n_halos"] == 1 and g["table"]["nucleus"][0] == 0
    # a halo straddling the periodic corner, particles at 0 and just below L
    _say("[gpu] edge: periodic corner")
    L = 12.0
    pts = rng.standard_normal((3000, 3)) * 0.25
    pos = np.mod(pts, L).astype(np.float32)
    pos[pos >= np.float32(L)] = 0.0
    pos[:5] = 0.0
    pos[5:10] = np.nextafter(np.float32(L), np.float32(0))
    g = gpu_find(ctx, pos, box=L, mean_density=1.0)
    ref = oracle.find(pos, box=L, mean_density=1.0,
                      density_override=g["density"].astype(np.float64))
    assert_same_labels(g, ref)
    assert g["n_halos"] >= 1
    assert len(density_violations(g["density"], oracle.density(pos, box=L, mean_density=1.0))) == 0
    # smallest box: exactly three cells per side (a compact clump, so that no
    # L0 group spans half the box)
    _say("[gpu] edge: three cells")
    small = np.concatenate([0.65 + 0.04 * rng.standard_normal((60, 3)), rng.random((20, 3)) * 1.3])
    small = np.mod(small, 1.3).astype(np.float32)
    small[small >= np.float32(1.3)] = 0.0
    g = gpu_find(ctx, small, box=1.3, mean_density=1.0)
    assert g["n_halos"] >= 1
    ref = oracle.find(small, box=1.3, mean_density=1.0,
                      density_override=g["density"].astype(np.float64))
    assert_same_labels(g, ref)
    # out-of-range coordinates are rejected
    _say("[gpu] edge: invalid positions")
    bad = sparse.copy()
    bad[7, 1] = 40.0
    with pytest.raises(HfError):
        ctx.find(torch.from_numpy(bad).cuda(), _lib.default_params(box=40.0))
    with pytest.raises(HfError):
        ctx.find(torch.from_numpy(sparse).cuda(), _lib.default_params(box=1.0))
    # capacity: the first attempt with cap 1 fails and is retried with the count
    _say("[gpu] edge: capacity retry")
    pos, L, _ = _case("s3000")
    res = ctx.find(torch.from_numpy(pos).cuda(), _lib.default_params(box=L), halos_cap=1)
    g = gpu_find(ctx, pos, box=L)
    assert res["n_halos"] == g["n_halos"] > 1


def _rod_box(span, L=20.0, seed=12):
    """A uniform background (mean density 1) and a dense rod along x (spacing
    0.03, thickness 0.02): one L0 group whose extent along x is `span`."""
    rng = np.random.default_rng(seed)
    bg = rng.random((int(L ** 3), 3)) * L
    x = 2.0 + np.arange(0.0, span, 0.03)
    rod = np.stack([x, np.full_like(x, 10.0), np.full_like(x, 10.0)], 1)
    rod[:, 1:] += 0.02 * rng.standard_normal((len(x), 2))
    pos = np.mod(np.concatenate([bg, rod]), L).astype(np.float32)
    pos[pos >= np.float32(L)] = 0.0
    return pos, L


def test_group_spanning_half_the_box_is_rejected(ctx):
    """Minimum images stand for the distances inside an L0 group only while it
    spans less than half the box: a group reaching L/2 along an axis (a rod of
    0.55 L, one wrapping the whole box) makes hf_find fail with HF_ERR_INVALID;
    a rod of 0.45 L is found, bit-exact against the oracle."""
    from paper_2110_11408_amd import _lib
    from paper_2110_11408_amd._lib import HfError
    for span in (11.0, 20.0):
        pos, L = _rod_box(span)
        _say(f"[gpu] rod span={span}")
        with pytest.raises(HfError) as e:
            gpu_find(ctx, pos, box=L, mean_density=1.0)
        assert e.value.status == _lib.HF_ERR_INVALID and "half the periodic box" in str(e.value)
    pos, L = _rod_box(9.0)
    _say("[gpu] rod span=9")
    g = gpu_find(ctx, pos, box=L, mean_density=1.0)
    rod = g["l0"][-300:]
    assert np.all(rod == rod[0]) and rod[0] > 0
    ref = oracle.find(pos, box=L, mean_density=1.0, density_override=g["density"].astype(np.float64))
    assert_same_labels(g, ref)


def test_compaso_rejects_negative_or_nan_density(ctx, runs):
    """hf_compaso orders densities by their bit patterns: negative values and
    NaN are rejected (HF_ERR_INVALID), -0 is taken as +0 (the same value)."""
    import torch
    from paper_2110_11408_amd import _lib
    from paper_2110_11408_amd._lib import HfError
    pos, L, g = runs["s3000"]
    p = _lib.default_params(box=L)
    t = torch.from_numpy(pos).cuda()
    l0 = torch.from_numpy(g["l0"]).cuda()
    for bad in (-1.0, float("nan")):
        d = g["density"].copy()
        d[np.argmax(d)] = bad
        with pytest.raises(HfError) as e:
            ctx.compaso(t, torch.from_numpy(d).cuda(), l0, p)
        assert e.value.status == _lib.HF_ERR_INVALID and "non-negative" in str(e.value)
    zero = np.nonzero(g["density"] == 0.0)[0]
    assert len(zero) > 0
    d = g["density"].copy()
    d[zero] = -0.0
    res = ctx.compaso(t, torch.from_numpy(d).cuda(), l0, p)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(res["halo_id"].cpu().numpy(), g["halo_id"])


def test_rejected_call_then_valid_call_on_another_stream(ctx, runs):
    """A call rejected on the device (positions outside the box) returns with
    its stream idle, so a valid call on another stream right after it gives
    its own result."""
    import torch
    from paper_2110_11408_amd import _lib
    from paper_2110_11408_amd._lib import HfError
    pos, L, g = runs["s9001"]
    bad = pos.copy()
    bad[11, 2] = L + 1.0
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(s1):
        with pytest.raises(HfError):
            ctx.find(torch.from_numpy(bad).cuda(), _lib.default_params(box=L))
    with torch.cuda.stream(s2):
        out = ctx.find(torch.from_numpy(pos).cuda(), _lib.default_params(box=L))
        s2.synchronize()
    np.testing.assert_array_equal(out["density"].cpu().numpy(), g["density"])
    np.testing.assert_array_equal(out["halo_id"].cpu().numpy(), g["halo_id"])


def test_context_budget(runs):
    """hf_create's HBM budget: a call whose arena does not fit is refused with
    HF_ERR_NOMEM; with room for it the result is unchanged."""
    import torch
    from paper_2110_11408_amd import _lib
    from paper_2110_11408_amd._lib import HfError
    from paper_2110_11408_amd.api import Context
    pos, L, g = runs["s40123"]
    t = torch.from_numpy(pos).cuda()
    small = Context(0, budget_bytes=1 << 20)
    with pytest.raises(HfError) as e:
        small.find(t, _lib.default_params(box=L))
    assert e.value.status == _lib.HF_ERR_NOMEM and "budget" in str(e.value)
    small.close()
    roomy = Context(0, budget_bytes=1 << 30)
    out = roomy.find(t, _lib.default_params(box=L))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out["halo_id"].cpu().numpy(), g["halo_id"])
    roomy.close()


@pytest.fixture(scope="module")
def run256(ctx):
    """hf_find on the 256^3 box (16.8M particles) in the benchmark's launch
    configuration."""
    pos, L, _ = synth.named_box("plain256")
    _say(f"[gpu] hf_find plain256 n={len(pos)}")
    return pos, L, gpu_find(ctx, pos, box=L)


def _pick_groups(l0, rng, big=20, rand=200):
    labels, counts = np.unique(l0[l0 > 0], return_counts=True)
    pick = np.concatenate([labels[np.argsort(counts)[-big:]],
                           rng.choice(labels, min(rand, len(labels)), replace=False)])
    return np.unique(pick)


def _compare_sampled_compaso(g, pos, L, dens, l0, pick):
    """The oracle's CompaSO on the L0 groups `pick` of labelling l0 (all other
    particles outside every group) against the GPU's halos of those groups."""
    mask = np.isin(l0, pick)
    res = oracle.compaso(pos, dens, np.where(mask, l0, 0).astype(np.int32), box=L)
    return mask, res


def test_full_size_256_density_sampled(run256):
    """Densities of ~22000 sampled particles (random plus the densest) against
    the oracle."""
    pos, L, g = run256
    rng = np.random.default_rng(0)
    which = rng.choice(len(pos), 20000, replace=False)
    dense = np.argsort(g["density"])[-2000:]
    which = np.unique(np.concatenate([which, dense]))
    ref = oracle.density_sample(pos, which, box=L)
    assert len(density_violations(g["density"][which], ref)) == 0


@pytest.mark.timeout(900)
def test_full_size_256_labels_bit_exact(run256):
    """Every one of the 16.8M L0 labels equals the oracle's FoF on the GPU
    densities, bit for bit; the oracle's CompaSO on sampled L0 groups (the 20
    largest and 200 random ones) gives the GPU's halo labels and table rows."""
    pos, L, g = run256
    dens = g["density"].astype(np.float64)
    _say("[gpu] plain256: oracle FoF over the whole box on the GPU densities")
    ref_l0, ref_ng = oracle.fof(pos, dens, box=L)
    np.testing.assert_array_equal(g["l0"], ref_l0)
    assert g["stats"]["n_groups"] == ref_ng
    pick = _pick_groups(ref_l0, np.random.default_rng(0))
    _say(f"[gpu] plain256: oracle CompaSO on {len(pick)} groups")
    mask, res = _compare_sampled_compaso(g, pos, L, dens, ref_l0, pick)
    np.testing.assert_array_equal(g["halo_id"][mask], res["halo_id"][mask])
    tab = g["table"]
    in_pick = np.isin(tab["l0_id"], pick)
    np.testing.assert_array_equal(tab["id"][in_pick], res["table"]["id"])
    np.testing.assert_array_equal(tab["n"][in_pick], res["table"]["n"])
    np.testing.assert_array_equal(tab["n_enclosed"][in_pick], res["table"]["ienc"])


@pytest.fixture(scope="module")
def d64_256(run256):
    pos, L, _ = run256
    _say("[gpu] plain256: oracle FP64 densities over the whole box")
    return oracle.density(pos, box=L)


def _cell_counts(pos, L, rmin):
    """Particles in each particle's binning cell (cells of side >= rmin)."""
    nc = int(np.floor(L / (rmin * (1 + 1e-6))))
    c = np.minimum(np.floor(pos.astype(np.float64) * (nc / L)).astype(np.int64), nc - 1)
    key = (c[:, 2] * nc + c[:, 1]) * nc + c[:, 0]
    _, inv, cnt = np.unique(key, return_inverse=True, return_counts=True)
    return cnt[inv]


@pytest.mark.timeout(900)
def test_full_size_256_density_every_particle(run256, d64_256):
    """Every one of the 16.8M densities within 1e-5 max(Delta, 1) of the
    oracle's FP64 value; the worst error relative to that bound is reported for
    particles of dense cells (matrix-core sums) and of sparse ones (FP64)."""
    pos, L, g = run256
    err = np.abs(g["density"].astype(np.float64) - d64_256) / (DENS_REL * np.maximum(np.abs(d64_256), 1.0))
    dense = _cell_counts(pos, L, 0.4) >= 8
    _say(f"[gpu] plain256 density error / bound: dense max {err[dense].max():.3f} "
         f"(p99.99 {np.percentile(err[dense], 99.99):.3f}), sparse max {err[~dense].max():.3f}")
    worst = int(np.argmax(err))
    assert err[worst] <= 1.0, (worst, g["density"][worst], d64_256[worst], bool(dense[worst]))


@pytest.mark.timeout(900)
def test_full_size_256_fp64_attribution(run256, d64_256):
    """Against the oracle's FP64 field on the whole 256^3 box: L0 labels agree
    to >= 99.99% and every mismatch is explained by a near-threshold event; on
    sampled L0 groups (the oracle's CompaSO on its own FP64 groups) every halo
    label mismatch is explained too."""
    pos, L, g = run256
    d64 = d64_256
    _say("[gpu] plain256: oracle FP64 FoF and events over the whole box")
    l0_64, _ = oracle.fof(pos, d64, box=L)
    ev = oracle.events(pos, d64, l0_64, tol=DENS_REL, box=L)
    frac, bad = matched_agreement(g["l0"], l0_64)
    assert frac >= 0.9999, frac
    ok = explained_mismatches(bad, g["l0"], l0_64, ev)
    assert ok.all(), (len(bad), bad[~ok][:10])
    pick = _pick_groups(l0_64, np.random.default_rng(1))
    _say(f"[gpu] plain256: oracle FP64 CompaSO on {len(pick)} groups")
    mask, res = _compare_sampled_compaso(g, pos, L, d64, l0_64, pick)
    idx = np.nonzero(mask)[0]
    frac, bad = matched_agreement(g["halo_id"][idx], res["halo_id"][idx])
    ok = explained_mismatches(idx[bad], g["l0"], l0_64, ev)
    assert ok.all(), (len(bad), idx[bad][~ok][:10])


def test_separate_payload_sort_gives_same_result(ctx):
    """The binning's radix sort keeps the original index in the key word when
    both fit in 64 bits, else in a payload array; both forms give one result."""
    import os
    pos, L, _ = _case("s40123")
    a = gpu_find(ctx, pos, box=L)
    os.environ["HF_RADIX_PAYLOAD"] = "1"
    try:
        b = gpu_find(ctx, pos, box=L)
    finally:
        del os.environ["HF_RADIX_PAYLOAD"]
    np.testing.assert_array_equal(a["density"], b["density"])
    assert_same_labels(a, {"l0": b["l0"], "halo_id": b["halo_id"], "n_halos": b["n_halos"],
                           "table": {"id": b["table"]["id"], "nucleus": b["table"]["nucleus"],
                                     "l0": b["table"]["l0_id"], "n": b["table"]["n"],
                                     "ienc": b["table"]["n_enclosed"]}})


def test_density_wide_record_loads_give_same_result(ctx):
    """The density of the dense cells loads its records through one buffer
    descriptor while the byte offsets fit in 32 bits (below about 2.7e8
    particles), else through a descriptor per block.  This box, whose chunks do
    not fill the chip, takes a wavefront per row block with the one descriptor
    and a wavefront per chunk with the others; the densities are the same bits.
    (A wavefront per chunk with the one descriptor: test_density_and_fof_forms.)"""
    import os
    pos, L, _ = _case("s40123")
    a = gpu_find(ctx, pos, box=L)
    os.environ["HF_DENSITY_WIDE"] = "1"
    try:
        b = gpu_find(ctx, pos, box=L)
    finally:
        del os.environ["HF_DENSITY_WIDE"]
    np.testing.assert_array_equal(a["density"], b["density"])
    np.testing.assert_array_equal(a["l0"], b["l0"])
    np.testing.assert_array_equal(a["halo_id"], b["halo_id"])


def _many_peaks_box(radius, grid, seed):
    """A uniform background with one ball at 100x the mean density (a single L0
    group) holding a grid of compact 30-particle clumps 0.85 apart: every clump
    is a density peak above the nucleation floor, so the group has as many
    candidates as clumps."""
    rng = np.random.default_rng(seed)
    L = 20.0
    bg = rng.random((int(L ** 3), 3)) * L
    c = np.array([L / 2] * 3)
    nb = int(100 * 4 / 3 * np.pi * radius ** 3)
    v = rng.standard_normal((nb, 3))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    ball = c + v * (radius * rng.random(nb) ** (1 / 3))[:, None]
    g = np.stack(np.meshgrid(*[np.arange(k) for k in grid], indexing="ij"), -1).reshape(-1, 3)
    centres = c + (g - (np.array(grid) - 1) / 2.0) * 0.85
    clumps = np.concatenate([cc + 0.05 * rng.standard_normal((30, 3)) for cc in centres])
    pos = np.mod(np.concatenate([bg, ball, clumps]), L).astype(np.float32)
    pos[pos >= np.float32(L)] = 0.0
    return pos, L


@pytest.mark.parametrize("radius,grid", [(2.6, (4, 4, 5)), (3.5, (5, 5, 5))])
def test_group_with_many_candidates(ctx, radius, grid):
    """One L0 group with more than 64 nuclei, below and above 12 288 members:
    the acceptance walk of a group with many candidates, bit-exact against the
    oracle on the GPU densities."""
    pos, L = _many_peaks_box(radius, grid, seed=11)
    _say(f"[gpu] hf_find many peaks n={len(pos)} grid={grid}")
    g = gpu_find(ctx, pos, box=L, mean_density=1.0)
    ref = oracle.find(pos, box=L, mean_density=1.0, density_override=g["density"].astype(np.float64))
    assert_same_labels(g, ref)
    labels, counts = np.unique(g["l0"][g["l0"] > 0], return_counts=True)
    big = labels[np.argmax(counts)]
    assert np.sum(g["table"]["l0_id"] == big) > 64
    assert (counts.max() > 12288) == (radius > 3.0)


def test_full_size_512_sampled(ctx):
    """The 512^3 box (134M particles, 70 % in haloes up to 200 000 particles, in
    pairs and triples): sampled densities against the oracle, the L0 membership
    rule and labels, and the oracle's CompaSO on sampled L0 groups (the largest
    below 300 000 members, whose histograms do not fit in LDS, and random ones)
    with the GPU densities."""
    pos, L, _ = synth.named_box("large512")
    _say(f"[gpu] hf_find large512 n={len(pos)}")
    g = gpu_find(ctx, pos, box=L)
    _say("[gpu] large512: sampled densities")
    rng = np.random.default_rng(512)
    which = np.unique(np.concatenate([rng.choice(len(pos), 20000, replace=False),
                                      np.argsort(g["density"])[-2000:]]))
    ref = oracle.density_sample(pos, which, box=L)
    assert len(density_violations(g["density"][which], ref)) == 0
    l0 = g["l0"]
    dens = g["density"].astype(np.float64)
    assert np.all((l0 > 0) == (dens > 60.0))
    labels, first, counts = np.unique(l0[l0 > 0], return_index=True, return_counts=True)
    assert np.all(labels == np.nonzero(l0 > 0)[0][first] + 1)      # 1 + smallest index
    _say("[gpu] large512: CompaSO on sampled groups")
    ok = counts < 300000
    big = labels[ok][np.argsort(counts[ok])[-8:]]
    pick = np.unique(np.concatenate([big, rng.choice(labels, 100, replace=False)]))
    pick = pick[np.isin(pick, labels[ok])]
    mask = np.isin(l0, pick)
    res = oracle.compaso(pos, dens, np.where(mask, l0, 0).astype(np.int32), box=L)
    np.testing.assert_array_equal(g["halo_id"][mask], res["halo_id"][mask])
    tab = g["table"]
    in_pick = np.isin(tab["l0_id"], pick)
    np.testing.assert_array_equal(tab["id"][in_pick], res["table"]["id"])
    np.testing.assert_array_equal(tab["n"][in_pick], res["table"]["n"])
    np.testing.assert_array_equal(tab["n_enclosed"][in_pick], res["table"]["ienc"])
    # the largest sampled groups have more buckets than the histogram in LDS
    assert counts[np.isin(labels, big)].max() > 36864
