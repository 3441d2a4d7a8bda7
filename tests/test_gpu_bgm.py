"""The two-sided recursion (launch variants 4 and 5) on the GPU against the one-sided
kernels (variant 3), at the edges of its workgroups and launches: one event, blocks of
four events with a remainder, one event more than a launch holds; running coupling;
every colour-sum mode."""
import numpy as np
import pytest

from paper_2510_05392_amd import rambo
from test_gpu_parity import AS, _say

torch = pytest.importorskip('torch')
pytestmark = pytest.mark.gpu


@pytest.fixture(scope='module')
def binding():
    if not torch.cuda.is_available():
        pytest.fail('GPU tests need a GPU')
    from paper_2510_05392_amd import binding as b
    b.load()
    return b


def _handle(binding, name, variant, mode=0):
    m = binding.MatrixElement(name, colorsum_mode=mode)
    m.me_set_executor(binding.ME_EXEC_BG)
    m.me_set_bg(variant)
    return m


# FP64: both recursions are within 1e-12 of the exact value on well-conditioned events and
# on these seeds each other's rounding is all that differs; split colour sums: each form is
# within its stated bound (1e-5 FP16, 2e-4 BF16) of FP64
BOUND = {0: 1e-12, 1: 2e-5, 2: 4e-4}


@pytest.mark.parametrize('name,npar,nevt,variants', [
    ('gg_ttxgg', 6, 1, (4, 5)), ('gg_ttxgg', 6, 3, (4, 5)), ('gg_ttxgg', 6, 4, (4,)), ('gg_ttxgg', 6, 4 * 512 + 1, (4, 5)),
    ('gg_ttxggg', 7, 1, (4, 5)), ('gg_ttxggg', 7, 2, (4,)), ('gg_ttxggg', 7, 513, (4, 5)),
    ('gg_ttxggg', 7, 34817, (4,))])
def test_two_sided_against_one_sided(binding, name, npar, nevt, variants):
    mom = torch.from_numpy(rambo.generate(npar, nevt, 91)).cuda()
    ref = _handle(binding, name, 3).compute(mom, AS).cpu().numpy()
    for v in variants:
        for mode in (0, 1, 2):
            _say(f'case two-sided {name} nevt={nevt} variant={v} mode={mode}')
            got = _handle(binding, name, v, mode).compute(mom, AS).cpu().numpy()
            assert np.max(np.abs(got / ref - 1)) < BOUND[mode]


@pytest.mark.parametrize('name,npar', [('gg_ttxgg', 6), ('gg_ttxggg', 7)])
def test_running_coupling(binding, name, npar):
    _say(f'case two-sided running coupling {name}')
    nevt = 37
    mom = torch.from_numpy(rambo.generate(npar, nevt, 92)).cuda()
    alphas = torch.linspace(0.08, 0.2, nevt, dtype=torch.float64, device='cuda')
    outs = []
    for v in (3, 4):
        out = torch.empty(nevt, dtype=torch.float64, device='cuda')
        _handle(binding, name, v).me_compute_alphas(mom, nevt, alphas, out)
        outs.append(out.cpu().numpy())
    assert np.max(np.abs(outs[1] / outs[0] - 1)) < BOUND[0]


@pytest.mark.parametrize('nevt', [1, 257, 2305])
def test_six_gluons(binding, nevt):
    """Six gluons, FP64: sampled events against the team program (whose operations are
    others: the bound of the recursions above), an event's result the same in any place
    of the batch (one event, one more than the compute units hold, more than a launch),
    and running coupling |M|^2 ~ alpha_s^6."""
    _say(f'case two-sided gg_ttxgggg nevt={nevt}')
    mom = torch.from_numpy(rambo.generate(8, nevt, 93)).cuda()
    m = binding.MatrixElement('gg_ttxgggg')
    m.me_set_executor(binding.ME_EXEC_BG)
    got = m.compute(mom, AS).cpu().numpy()
    pick = sorted({0, nevt // 2, nevt - 1})
    ref = binding.MatrixElement('gg_ttxgggg').compute(mom[pick].contiguous(), AS).cpu().numpy()
    assert np.max(np.abs(got[pick] / ref - 1)) < BOUND[0]
    back = m.compute(mom.flip(0).contiguous(), AS).cpu().numpy()
    assert np.array_equal(got, back[::-1])
    alphas = torch.linspace(0.08, 0.2, nevt, dtype=torch.float64, device='cuda')
    out = torch.empty(nevt, dtype=torch.float64, device='cuda')
    m.me_compute_alphas(mom, nevt, alphas, out)
    assert np.max(np.abs(out.cpu().numpy() / (got * (alphas.cpu().numpy() / AS) ** 6) - 1)) < BOUND[0]


@pytest.mark.parametrize('name,npar,nevt', [('gg_ttxgg', 6, 1), ('gg_ttxgg', 6, 67), ('gg_ttxggg', 7, 1),
                                            ('gg_ttxggg', 7, 41)])
def test_selection_against_the_one_lane_sums(binding, name, npar, nevt):
    """Both draws of every event against the draws from the one-lane program's helicity
    sums and dual amplitudes, except where r * total is within 1e-9 of a running sum
    (there rounding decides): any r in [0, 1), with its ends."""
    _say(f'case selection {name} nevt={nevt}')
    mom = torch.from_numpy(rambo.generate(npar, nevt, 94)).cuda()
    rng = np.random.default_rng(nevt)
    rh, rc = rng.random(nevt), rng.random(nevt)
    rh[0], rc[-1] = 0.0, 1.0 - 2.0 ** -53
    m = binding.MatrixElement(name)
    out = torch.empty(nevt, dtype=torch.float64, device='cuda')
    sh, sc = (torch.full((nevt,), -1, dtype=torch.int32, device='cuda') for _ in range(2))
    m.me_select(mom, nevt, AS, torch.from_numpy(rh).cuda(), torch.from_numpy(rc).cuda(), out, sh, sc)
    good = m.me_good_helicities()
    sums = torch.empty((len(good), nevt), dtype=torch.float64, device='cuda')
    m.me_helicity_sums(mom, nevt, AS, good, sums)
    jam = torch.empty((len(good), nevt, m.ncolor, 2), dtype=torch.float64, device='cuda')
    m.me_jamps(mom, nevt, AS, good, jam)
    me2 = m.compute(mom, AS).cpu().numpy()
    assert np.max(np.abs(out.cpu().numpy() / me2 - 1)) < BOUND[0]
    sums, flows = sums.cpu().numpy(), (jam ** 2).sum(-1).cpu().numpy()
    sh, sc = sh.cpu().numpy(), sc.cpu().numpy()

    def check(w, r, pick):
        cum = np.cumsum(w)
        t = r * cum[-1]
        first = np.nonzero(cum > t)[0]
        want = first[0] if len(first) else np.nonzero(w > 0)[0][-1]
        assert pick == want or np.abs(cum - t).min() <= 1e-9 * cum[-1], (pick, want)

    for e in range(nevt):
        k = list(good).index(sh[e])
        check(sums[:, e], rh[e], k)
        check(flows[k, e], rc[e], sc[e])


@pytest.mark.parametrize('name,npar,nevt', [('gg_ttxgg', 6, 4 * 4 * 512), ('gg_ttxgg', 6, 4 * 4 * 512 + 5),
                                            ('gg_ttxggg', 7, 4 * 512), ('gg_ttxggg', 7, 4 * 512 + 3)])
def test_selection_in_rounds_of_workgroups(binding, name, npar, nevt):
    """Four rounds of 512 resident workgroups, and the first size beyond, where a workgroup
    takes block after block: every event's sum and draws are the same bits as in batches of
    the first and the last seven events alone (an event's sums run in one order wherever it
    stands), in each of three calls."""
    _say(f'case selection in rounds {name} nevt={nevt}')
    mom = torch.from_numpy(rambo.generate(npar, nevt, 96)).cuda()
    rng = np.random.default_rng(nevt)
    rh, rc = (torch.from_numpy(rng.random(nevt)).cuda() for _ in range(2))
    m = binding.MatrixElement(name)
    m.me_filter_helicities(mom, nevt, AS)

    def select(first, n):
        out = torch.zeros(n, dtype=torch.float64, device='cuda')
        sh, sc = (torch.full((n,), -1, dtype=torch.int32, device='cuda') for _ in range(2))
        m.me_select(mom[first:first + n], n, AS, rh[first:first + n], rc[first:first + n], out, sh, sc)
        assert int(sh.min()) >= 0 and int(sc.min()) >= 0 and bool(torch.all(out > 0))
        return [x.cpu().numpy() for x in (out, sh, sc)]

    few = [select(0, 7), select(nevt - 7, 7)]
    for _ in range(3):
        all_ = select(0, nevt)
        for want, part in zip(few, (slice(0, 7), slice(nevt - 7, nevt))):
            assert all(np.array_equal(a[part], b) for a, b in zip(all_, want))


def test_selection_scratch_is_bounded(binding):
    """Scratch of a slot (123 KB with five gluons) for each event up to 2048, 252 MB, and not
    2 GB for 16384 events; a smaller batch after that needs no more."""
    _say('case selection scratch gg_ttxggg')
    nevt = 16384
    mom = torch.from_numpy(rambo.generate(7, nevt, 97)).cuda()
    r = torch.rand(nevt, dtype=torch.float64, device='cuda')
    out = torch.empty(nevt, dtype=torch.float64, device='cuda')
    sh, sc = (torch.empty(nevt, dtype=torch.int32, device='cuda') for _ in range(2))
    m = binding.MatrixElement('gg_ttxggg')
    m.me_filter_helicities(mom, nevt, AS)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    held = []
    for n in (nevt, 2048, 600):
        m.me_select(mom, n, AS, r, r, out, sh, sc)
        torch.cuda.synchronize()
        held.append(before - torch.cuda.mem_get_info()[0])
    assert held[0] < 288 << 20 and held[1:] == held[:1] * 2
