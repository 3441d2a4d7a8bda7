"""The training step's whole-network kernels against the layer-by-layer ones, which the
same call runs when the feature rows are not 16-byte aligned: batches around a
workgroup's 32 rows, the smallest and the largest hidden widths, one and several layers."""
import numpy as np
import pytest

from paper_2510_05392_amd import rambo

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


@pytest.mark.parametrize('width,depth,nfeat', [(32, 1, 15), (64, 3, 21), (96, 2, 10), (160, 1, 28), (256, 4, 15)])
@pytest.mark.parametrize('nb', [1, 31, 32, 33, 100, 1000])
def test_whole_network_step_against_layers(binding, width, depth, nfeat, nb):
    """Both take every product's K steps in the same order, so pre-activations and
    activations are the same bits; the gradients' sums over the rows differ in order
    (FP32: nb 2^-24 of the sum of the terms' magnitudes, bounded by sqrt(nb) times the
    layer's largest entry), and the loss likewise."""
    _say(f'case training step {nfeat}-{width}x{depth} nb={nb}')
    rng = np.random.default_rng(nb)
    kpad = binding.Surrogate(nfeat, width, depth, seed=3).kpad
    x = np.zeros((nb, kpad), np.float32)
    x[:, :nfeat] = rng.normal(size=(nb, nfeat))
    rows = torch.from_numpy(x).bfloat16().view(torch.int16).reshape(-1)
    target = torch.from_numpy(rng.normal(size=nb).astype(np.float32)).cuda()
    got = []
    for shift in (0, 1):
        store = torch.zeros(nb * kpad + 8, dtype=torch.int16, device='cuda')
        feat = store[shift:shift + nb * kpad]
        feat.copy_(rows)
        sur = binding.Surrogate(nfeat, width, depth, seed=3)
        loss = torch.zeros(1, dtype=torch.float32, device='cuda')
        sur.me_sur_grads(feat, target, nb, loss)
        torch.cuda.synchronize()
        acts = [sur.me_sur_activations(k, kind, nb) for k in range(depth + 1) for kind in (0, 1)]
        g1 = sur.me_sur_get_grads()
        for _ in range(3):
            sur.me_sur_train_step(feat, target, nb, 1e-3, loss)
        torch.cuda.synchronize()
        got.append((acts, g1, float(loss.item()), sur.me_sur_get_params()))
    (fa, fg, fl, fp), (la, lg, ll, lp) = got
    assert all(np.array_equal(a, b) for a, b in zip(fa, la))
    tol = max(nb, 16) * 2.0 ** -24
    assert np.linalg.norm(fg - lg) <= tol * np.linalg.norm(lg) * 4
    assert abs(fl - ll) <= 1e-4 * abs(ll)
    # three Adam steps move a parameter by at most 3 lr each; where a gradient is no more
    # than its rounding the step's direction is not determined
    assert np.abs(fp - lp).max() <= 6.1e-3
    assert np.linalg.norm(fp - lp) <= 2e-2 * np.linalg.norm(lp)


@pytest.mark.parametrize('npar', [4, 5, 6, 7, 8])
@pytest.mark.parametrize('nb', [1, 127, 128, 129, 1000])
def test_feature_rows_against_the_event_kernel(binding, npar, nb):
    """The same expressions as the kernel that unaligned rows take: raw features equal to
    1e-6 (a rounding of the FP64 products, which is all there is of log 1 for the two
    incoming gluons), rows to one BF16 unit, padding zero."""
    _say(f'case features npar={npar} nb={nb}')
    nfeat = npar * (npar - 1) // 2
    mom = torch.from_numpy(rambo.generate(npar, nb, 6)).cuda()
    sur = binding.Surrogate(nfeat, 32, 1, seed=3)
    rng = np.random.default_rng(npar)
    sur.me_sur_set_normalisation(rng.normal(size=nfeat).astype(np.float32),
                                 rng.uniform(0.5, 2, nfeat).astype(np.float32))
    got = []
    for shift in (0, 1):
        store = torch.full((nb * sur.kpad + 8,), 0x7f7f, dtype=torch.int16, device='cuda')
        raw = torch.empty((nb, nfeat), dtype=torch.float32, device='cuda')
        sur.me_sur_features(mom, nb, npar, store[shift:], raw)
        torch.cuda.synchronize()
        row = store[shift:shift + nb * sur.kpad].clone().view(torch.bfloat16).float().reshape(nb, sur.kpad)
        assert torch.all(store[shift + nb * sur.kpad:] == 0x7f7f)
        assert torch.all(row[:, nfeat:] == 0)
        got.append((raw.cpu().numpy(), row.cpu().numpy()))
    assert np.allclose(got[0][0], got[1][0], rtol=1e-6, atol=1e-6)
    assert np.allclose(got[0][1], got[1][1], rtol=2.0 ** -7, atol=1e-6)


@pytest.mark.parametrize('nb,width', [(262144, 32), (100003, 160)])
def test_loss_of_many_rows(binding, nb, width):
    """The summed squared error of a network of zeros (outputs 0, so the errors are the
    targets) against 64 bits: FP32 sums over the 32 rows of a workgroup (five roundings) and
    one of the total are all that is rounded, 6 2^-24 of it.  Targets all alike, whose
    roundings in a running sum do not average out, and spread ones."""
    rng = np.random.default_rng(nb)
    sur = binding.Surrogate(10, width, 1, seed=3)
    sur.me_sur_set_params(np.zeros(sur.nparams, np.float32))
    feat = torch.zeros(nb * sur.kpad, dtype=torch.int16, device='cuda')
    for kind, t in (('alike', np.full(nb, 0.3)), ('spread', rng.normal(size=nb))):
        _say(f'case loss {kind} width={width} nb={nb}')
        t = t.astype(np.float32)
        loss = torch.zeros(1, dtype=torch.float32, device='cuda')
        sur.me_sur_grads(feat, torch.from_numpy(t).cuda(), nb, loss)
        want = (t * t).astype(np.float64).sum()
        assert abs(float(loss.item()) - want) <= 6 * 2.0 ** -24 * want


@pytest.mark.parametrize('width,shift', [(48, 0), (64, 1)])
def test_captured_gradients_need_no_allocation(binding, width, shift):
    """Gradients captured into a graph after an eager call of that size had been through the
    handle another way (48: prediction; 64: gradients of aligned rows, then captured ones of
    rows that are not): every replay equals the eager result of a handle of its own."""
    nfeat, depth, nb = 10, 2, 200
    _say(f'case captured gradients width={width}')
    rng = np.random.default_rng(width)
    sur, ref = (binding.Surrogate(nfeat, width, depth, seed=3) for _ in range(2))
    store = torch.zeros(nb * sur.kpad + 8, dtype=torch.int16, device='cuda')
    feat = store[shift:shift + nb * sur.kpad]
    target = torch.from_numpy(rng.normal(size=nb).astype(np.float32)).cuda()
    out = torch.empty(nb, dtype=torch.float32, device='cuda')
    if width == 48:
        sur.me_sur_predict(store, nb, out)
    else:
        sur.me_sur_grads(store, target, nb)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sur.me_sur_grads(feat, target, nb, None, torch.cuda.current_stream())
    for _ in range(3):
        rows = np.zeros((nb, sur.kpad), np.float32)
        rows[:, :nfeat] = rng.normal(size=(nb, nfeat))
        feat.copy_(torch.from_numpy(rows).bfloat16().view(torch.int16).reshape(-1))
        ref.me_sur_grads(feat, target, nb)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(sur.me_sur_get_grads(), ref.me_sur_get_grads())


@pytest.mark.parametrize('width,depth,nfeat', [(32, 1, 15), (64, 3, 21), (256, 4, 15), (48, 2, 10)])
def test_adam_steps_against_the_host(binding, width, depth, nfeat):
    """Every parameter after each of three steps against Adam (beta 0.9 and 0.999, eps 1e-8)
    on the host from the gradients read back: FP32 rounding of the step (1 - 0.999^k in FP32
    is good to 2^-25 / 0.001 = 3e-5, half of that under the root, the rest is smaller: 1e-4
    of lr together) and of the sum.  The network then acts as one that is given these
    parameters: equal predictions and gradients."""
    _say(f'case adam {nfeat}-{width}x{depth}')
    rng = np.random.default_rng(width)
    nb, lr = 300, 1e-3
    sur, ref = (binding.Surrogate(nfeat, width, depth, seed=s) for s in (3, 4))
    x = np.zeros((nb, sur.kpad), np.float32)
    x[:, :nfeat] = rng.normal(size=(nb, nfeat))
    feat = torch.from_numpy(x).bfloat16().view(torch.int16).reshape(-1).cuda()
    target = torch.from_numpy(rng.normal(size=nb).astype(np.float32)).cuda()
    b1, b2 = float(np.float32(0.9)), float(np.float32(0.999))
    m, v = np.zeros(sur.nparams), np.zeros(sur.nparams)
    for step in range(1, 4):
        before = sur.me_sur_get_params().astype(np.float64)
        sur.me_sur_train_step(feat, target, nb, lr)
        torch.cuda.synchronize()
        g, after = sur.me_sur_get_grads().astype(np.float64), sur.me_sur_get_params()
        m, v = b1 * m + (1 - b1) * g, b2 * v + (1 - b2) * g * g
        move = lr * (m / (1 - b1 ** step)) / (np.sqrt(v / (1 - b2 ** step)) + 1e-8)
        assert np.abs(move).max() > 0.9 * lr and (np.abs(move) > 0.1 * lr).mean() > 0.9
        assert np.all(np.abs(after - (before - move)) <= 1e-4 * lr + 2.0 ** -23 * np.abs(before))
    ref.me_sur_set_params(sur.me_sur_get_params())
    got = []
    for s in (sur, ref):
        y = torch.empty(nb, dtype=torch.float32, device='cuda')
        s.me_sur_predict(feat, nb, y)
        s.me_sur_grads(feat, target, nb)
        torch.cuda.synchronize()
        got.append((y.cpu().numpy(), s.me_sur_get_grads()))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
