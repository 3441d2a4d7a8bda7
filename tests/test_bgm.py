"""The two-sided recursion (launch variants 4 and 5 of the Berends-Giele executor) on the
host: its dual amplitudes against the one-sided recycling kernel's, flow by flow; the
mirror relation it rests on; its colour form in symmetry sectors; its operation count."""
import math

import numpy as np
import pytest

from cpu_harness import bgm_build
from cpu_harness import build as harness
from paper_2510_05392_amd import flops, rambo
from paper_2510_05392_amd.gen.colour import colour_matrix

AS = 0.118


@pytest.mark.parametrize('n,nevt', [(4, 40), (5, 6)])
def test_amplitudes_flow_by_flow(n, nevt):
    """Every row's dual amplitudes equal the one-sided recursion's (each rounds a few
    hundred operations: 1e-12 of the event's largest amplitude), and the mirrored
    helicity has their complex conjugates up to one sign for all flows."""
    assert bgm_build.table_words_off(n) == 0
    mom = rambo.generate(n + 2, nevt, 8)
    g = math.sqrt(4 * math.pi * AS)
    two, hel = bgm_build.jamps(n, mom, g, 173.0)
    assert sorted(list(hel) + [2 ** (n + 2) - 1 - h for h in hel]) == list(range(2 ** (n + 2)))
    one = harness.build_bg().jamps_recycled(n, mom, g, 173.0, list(range(2 ** (n + 2)))).transpose(1, 0, 2)
    scale = np.abs(one).max(axis=(1, 2), keepdims=True)
    assert np.max(np.abs(two - one[:, hel]) / scale) < 1e-12
    mirror = one[:, 2 ** (n + 2) - 1 - hel].conj()
    plus, minus = (np.abs(mirror - s * one[:, hel]).max(axis=2) / scale[..., 0] for s in (1, -1))
    assert np.max(np.minimum(plus, minus)) < 1e-12


def test_amplitudes_of_six_gluons():
    """A row of each quark helicity pair against the one-row recursion (1e-12 of the
    largest amplitude: each rounds some thousand operations)."""
    assert bgm_build.table_words_off(6) == 0
    mom = rambo.generate(8, 2, 8)
    g = math.sqrt(4 * math.pi * AS)
    two, hel = bgm_build.jamps(6, mom, g, 173.0)
    assert sorted(list(hel) + [255 - h for h in hel]) == list(range(256))
    rows = [0, 31, 37, 64 - 1, 64 + 5, 127]
    one = harness.build_bg().jamps(6, mom, g, 173.0, [int(h) for h in hel[rows]]).transpose(1, 0, 2)
    scale = np.abs(two).max(axis=(1, 2), keepdims=True)
    assert np.max(np.abs(two[:, rows] - one) / scale) < 1e-12


@pytest.mark.parametrize('n', [4, 5, 6])
def test_colour_sectors(n):
    """The sum over sectors is the quadratic form of the colour matrix (sums of n!^2
    products in two orders: 1e-12 of the form for amplitudes of random sign), and every
    element is exact in FP32."""
    cf = np.array(colour_matrix(n)[0])
    orb, sec = bgm_build.sectors(n, cf)
    assert sorted(set(orb.reshape(-1).tolist())) == list(range(len(cf)))
    assert np.array_equal(sec.astype(np.float32), sec)
    a = np.random.default_rng(n).normal(size=(5, len(cf)))
    g = orb.shape[1]
    sign = np.array([[(-1) ** bin(s & b).count('1') for b in range(g)] for s in range(g)])
    x = a[:, orb] @ sign.T                                    # [5][orbit][sector]
    form = np.einsum('eos,sop,eps->e', x, sec, x)
    assert np.max(np.abs(form / np.einsum('ex,xy,ey->e', a, cf, a) - 1)) < 1e-12


@pytest.mark.parametrize('n', [4, 5, 6])
def test_flops_equal_the_counted_operations(n):
    """flops.bgm_event equals the operations of the device functions for one event,
    counted with the operation-counting scalar, phase by phase (a quark with pz < 0
    takes one operation more in each of its two spinors)."""
    mom = rambo.generate(n + 2, 3, 1003)
    f = flops.bgm_event(n)
    for m in mom:
        setup, currents, spinors, qj, prefixes = bgm_build.count_event(n, m)
        assert setup == f['setup'] + 2 * int((m[2:4, 3] < 0).sum())
        assert (currents, spinors, qj, prefixes) == (f['currents'], f['spinors'], f['qj'], f['prefixes'])


def test_draw_never_takes_an_entry_of_no_weight():
    """Random weights, half of them zero: at the end of every lane's running sum, where the
    next lane's start is rounded otherwise, and at random points, the entry drawn has a
    weight and its running sum is the one that passes t but for that rounding; before the
    first entry and beyond the total as the rule says."""
    rng = np.random.default_rng(5)
    gaps = 0
    for _ in range(200):
        n = int(rng.integers(3, 129))
        w = rng.random(n) * (rng.random(n) < 0.5)
        w[rng.integers(n)] = 0.5
        _, start = bgm_build.draw(w, 0.0)
        pad = np.concatenate([w, np.zeros(128 - n)]).reshape(64, 2)
        ends = (start + pad[:, 0]) + pad[:, 1]
        gaps += int((start[1:] > ends[:-1]).sum())
        cum = np.cumsum(w)
        for t in np.concatenate([ends[ends < cum[-1]], rng.random(20) * cum[-1], [0.0]]):
            k, _ = bgm_build.draw(w, t)
            assert w[k] > 0.0
            assert cum[k] >= t * (1 - 1e-13) and (k == 0 or cum[k - 1] <= t + 1e-13 * cum[-1])
        assert bgm_build.draw(w, 2 * cum[-1])[0] == np.nonzero(w)[0][-1]
        assert bgm_build.draw(w, -1.0)[0] == 0
    assert gaps > 50
    assert bgm_build.draw(np.zeros(7), 0.0)[0] == 0


def test_flops_and_names_of_the_diagram_kernels():
    """The kernel each executor's FP64 path launches, the test that counts its operations,
    and half of the per-helicity code where one helicity of a mirror pair is evaluated."""
    name = flops.diagram_kernel_name
    for p in ('gg_ttx', 'gg_ttxg'):
        assert name(p, 0) == (f'pair_kernel<{p}>', 'tests/test_generator.py')
        assert flops.diagram_kernel(p, 0) == (flops.per_event_helicity(p) + flops.QUARK_BRANCH_MEAN) / 2
        assert flops.diagram_kernel(p, 1) == flops.per_event_helicity(p) + flops.QUARK_BRANCH_MEAN
    assert name('gg_ttxgg', 0) == ('me_kernel<gg_ttxgg>', 'tests/test_generator.py')
    assert flops.diagram_kernel('gg_ttxgg', 0) == flops.per_event_helicity('gg_ttxgg') + flops.QUARK_BRANCH_MEAN
    assert name('gg_ttxggg', 3, 3) == ('bgh_kernel<5>', 'tests/test_generator.py')
    assert name('gg_ttxggg', 3, 4) == ('bgm_fused_kernel<5>', 'tests/test_bgm.py')
    assert name('gg_ttxgggg', 3, 1) == ('bgm_fused_kernel<6>', 'tests/test_bgm.py')
    assert name('gg_ttxggg', 3, 1) == ('bg_kernel<5>', 'tests/test_generator.py')
    assert name('gg_ttxgg', 2) == ('sums_kernel<gg_ttxgg>', 'tests/test_generator.py')
    assert name('gg_ttxg', 1) == ('team_kernel<gg_ttxg_team>', 'tests/test_generator.py')


@pytest.mark.parametrize('n', [4, 5, 6])
def test_rows_of_helicities_whose_mirror_image_is_not_good(n):
    """A helicity's row is the one of its own index or of its mirror image's, and of no
    other's; pairs with one good helicity count once, whichever of the two it is."""
    _, hel = bgm_build.jamps(n, rambo.generate(n + 2, 1, 8), 1.0, 173.0)
    nhel = 2 ** (n + 2)
    for h in range(nhel):
        assert hel[bgm_build.row(n, h)] in (h, nhel - 1 - h)
    rng = np.random.default_rng(n)
    for good in ([0], [nhel - 1], [0, nhel - 1], sorted(rng.permutation(nhel)[:nhel // 3].tolist()), []):
        want = {}
        for h in good:
            want[min(h, nhel - 1 - h)] = want.get(min(h, nhel - 1 - h), 0) + 1
        assert bgm_build.mirror_pairs(good, nhel) == sorted(want.items())
