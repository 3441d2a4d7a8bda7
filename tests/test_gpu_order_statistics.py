"""Quantiles by radix selection and the ordered indices of stage 1 on the device, against
numpy on the same numbers: sizes around a block of 256, repeated values, zeros and
infinities, order statistics at both ends."""
import numpy as np
import pytest

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)


@pytest.fixture(scope='module')
def binding():
    if not torch.cuda.is_available():
        pytest.fail('GPU tests need a GPU')
    from paper_2510_05392_amd import binding as b
    b.load()
    return b


def _quantile(w, q):
    if q >= 1.0:
        return w.max()
    s = np.sort(w)
    pos = q * (len(w) - 1)
    lo = int(np.floor(pos))
    return s[lo] + (s[lo + 1] - s[lo]) * (pos - lo) if pos > lo else s[lo]


def _values(kind, n, rng):
    if kind == 'spread':       # every digit of the bit patterns takes part
        return 10.0 ** rng.uniform(-300, 300, n)
    if kind == 'close':        # differ in the last digits only
        return 1.0 + rng.integers(0, 3000, n) * 2.0 ** -52
    w = rng.integers(0, 3, n).astype(float)    # repeated, zeros
    w[rng.random(n) < 0.01] = np.inf
    return w


@pytest.mark.parametrize('n', [1, 2, 255, 256, 257, 1000, 70001])
@pytest.mark.parametrize('kind', ['spread', 'close', 'repeated'])
def test_quantiles_are_exact(binding, kind, n):
    """The order statistics are exact and the interpolation is one expression: equal bits."""
    _say(f'case quantile {kind} n={n}')
    rng = np.random.default_rng(n)
    one = torch.ones(n, dtype=torch.float64, device='cuda')
    y = torch.zeros(n, dtype=torch.float32, device='cuda')
    for q in (1e-9, 0.1, 0.5, 0.99, 1.0):
        w, x = _values(kind, n, rng), _values('close', n, rng)
        got = binding.me_unweight_quantile(torch.from_numpy(w).cuda(), one, n, q)
        with np.errstate(invalid='ignore'):
            want = _quantile(w, q)
        assert got == want or (np.isnan(got) and np.isnan(want)), (q, got, want)
        # both quantiles at once: surrogate weight exp(0) wps = wps, ratio me2 wps / wps
        wps = torch.from_numpy(2.0 ** rng.integers(-8, 8, n)).cuda()
        both = binding.me_unweight_maxima(y, wps, torch.from_numpy(x).cuda(), n, 0.0, 1.0, q)
        assert both == (_quantile(wps.cpu().numpy(), q), _quantile(x, q))


@pytest.mark.parametrize('n', [1, 63, 255, 256, 257, 300000])
def test_stage1_indices(binding, n):
    _say(f'case stage 1 n={n}')
    rng = np.random.default_rng(n)
    wps, r = rng.uniform(0.5, 2.0, n), rng.random(n)
    y = torch.zeros(n, dtype=torch.float32, device='cuda')
    for top in (1.0, 8.0, 1e9):
        what = torch.empty(n, dtype=torch.float64, device='cuda')
        idx = torch.full((n,), -1, dtype=torch.int64, device='cuda')
        m = binding.me_unweight_stage1(y, torch.from_numpy(wps).cuda(), torch.from_numpy(r).cuda(), n, 0.0, 1.0, top,
                                       what, idx)
        want = np.nonzero(r < np.minimum(1.0, wps / top))[0]
        assert np.array_equal(what.cpu().numpy(), wps)
        assert m == len(want) and np.array_equal(idx[:m].cpu().numpy(), want)
        assert torch.all(idx[m:] == -1)


@pytest.mark.parametrize('n', [257, 300000])
def test_stage1_indices_over_the_random_numbers(binding, n):
    """idx in the storage of r1, which the call no longer needs once it has decided: the
    same indices."""
    _say(f'case stage 1 in place n={n}')
    rng = np.random.default_rng(n)
    wps, r = rng.uniform(0.5, 2.0, n), rng.random(n)
    y = torch.zeros(n, dtype=torch.float32, device='cuda')
    what = torch.empty(n, dtype=torch.float64, device='cuda')
    for _ in range(5):
        rd = torch.from_numpy(r).cuda()
        idx = rd.view(torch.int64)
        m = binding.me_unweight_stage1(y, torch.from_numpy(wps).cuda(), rd, n, 0.0, 1.0, 1.5, what, idx)
        want = np.nonzero(r < np.minimum(1.0, wps / 1.5))[0]
        assert m == len(want) and np.array_equal(idx[:m].cpu().numpy(), want)
