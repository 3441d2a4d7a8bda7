"""The one-launch kernels of the processes with few flows against the one-lane kernel's
helicity sums: sizes around a workgroup's 16 events, running coupling, and the call
without allocation."""
import numpy as np
import pytest

from paper_2510_05392_amd import rambo
from test_gpu_parity import AS, NPAR, _say

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu


@pytest.fixture(scope='module')
def binding():
    if not torch.cuda.is_available():
        pytest.fail('GPU tests need a GPU')
    from paper_2510_05392_amd import binding as b
    b.load()
    return b


@pytest.mark.parametrize('name', ['gg_ttx', 'gg_ttxg'])
@pytest.mark.parametrize('nevt', [1, 15, 16, 17, 1000])
def test_one_launch_against_helicity_sums(binding, name, nevt):
    """Half of the helicities are taken from their mirror images: the same sums but for
    rounding (some thousand operations each: 1e-12 of |M|^2)."""
    _say(f'case one launch {name} nevt={nevt}')
    mom = torch.from_numpy(rambo.generate(NPAR[name], nevt, 95)).cuda()
    m = binding.MatrixElement(name)
    got = m.compute(mom, AS)
    good = m.me_good_helicities()
    sums = torch.empty((len(good), nevt), dtype=torch.float64, device='cuda')
    m.me_helicity_sums(mom, nevt, AS, good, sums)
    torch.cuda.synchronize()
    ref = sums.sum(0).cpu().numpy()
    norm = 256    # the initial-state average; the sums have the colour denominator in them
    g = got.cpu().numpy()
    assert np.max(np.abs(g * norm / ref - 1)) < 1e-12
    out = torch.empty(nevt, dtype=torch.float64, device='cuda')
    m.me_compute_noalloc(mom, nevt, AS, out)
    assert np.array_equal(out.cpu().numpy(), g)
    alphas = torch.linspace(0.08, 0.2, nevt, dtype=torch.float64, device='cuda')
    m.me_compute_alphas(mom, nevt, alphas, out)
    torch.cuda.synchronize()
    k = NPAR[name] - 2
    assert np.max(np.abs(out.cpu().numpy() / (g * (alphas.cpu().numpy() / AS) ** k) - 1)) < 1e-12


def test_more_events_than_threads_of_a_launch(binding):
    """A batch whose lanes (16 an event) are more than the 2^32 - 1 threads of a launch:
    copies of 4096 events, each with the bits of the batch of 4096."""
    name, base, nevt = 'gg_ttxg', 4096, 2 ** 28 + 4096
    _say(f'case one launch {name} nevt={nevt}')
    free = torch.cuda.mem_get_info()[0]
    if free < 60 << 30:
        pytest.skip('needs 60 GB of device memory')
    few = torch.from_numpy(rambo.generate(NPAR[name], base, 96)).cuda()
    coupling = torch.linspace(0.08, 0.2, base, dtype=torch.float64, device='cuda')
    m = binding.MatrixElement(name)
    want = torch.empty(base, dtype=torch.float64, device='cuda')
    m.me_compute_alphas(few, base, coupling, want)
    mom = few.repeat(nevt // base, 1, 1)
    alphas = coupling.repeat(nevt // base)
    out = torch.zeros(nevt, dtype=torch.float64, device='cuda')
    m.me_compute_alphas(mom, nevt, alphas, out)
    torch.cuda.synchronize()
    assert bool((out.view(-1, base) == want).all())
    del mom, alphas, out
    torch.cuda.empty_cache()
