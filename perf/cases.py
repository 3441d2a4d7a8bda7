"""Timing cases: the calls that a user of this library makes, over the sizes they are made at.

Each case is one public call sequence on device data that the program already holds:
  me         me_compute / me_compute_alphas of one process (the matrix-element engine);
  select     me_select: |M|^2 with a drawn helicity and colour flow, for event output;
  unweight   SurrogatePipeline.unweight: features, network, stage 1, exact |M|^2 of the kept
             events, stage 2, summary;
  calibrate  me_unweight_maxima: the quantiles that two-stage unweighting needs;
  train      me_sur_train_step of the surrogate, with the step's gradients read back;
  predict    me_sur_features and me_sur_predict (stage 1 of unweighting, without the selection).

Momenta are flat RAMBO points (Kleiss, Stirling, Ellis 1986) at 1500 GeV, drawn on the device.
Handles are configured as the autotuner leaves them: the one-lane executor for g g -> t t~ (g),
helicity recycling with the colour form fused for four and five gluons, the recursion's rows for six.
"""
import itertools
import math

import numpy as np
import torch

from paper_2510_05392_amd import binding
from paper_2510_05392_amd.surrogate import SurrogatePipeline

SQRTS, MT, ALPHA_S = 1500.0, 173.0, 0.118
NPAR = {'gg_ttx': 4, 'gg_ttxg': 5, 'gg_ttxgg': 6, 'gg_ttxggg': 7, 'gg_ttxgggg': 8}
# the largest batch of each process that the benchmark and the tests run (six gluons: a chunk of theirs)
MOST = {'gg_ttx': 524288, 'gg_ttxg': 524288, 'gg_ttxgg': 524288, 'gg_ttxggg': 262144, 'gg_ttxgggg': 4096}
MODES = {'fp64': binding.ME_CS_FP64, 'fp16': binding.ME_CS_FP16X2, 'bf16': binding.ME_CS_BF16X2}

# log|M|^2 of flat phase-space points as a linear function of the pair invariants log(2 p_i.p_j / s), by the
# kinds of the pair (b beam, t top, g gluon): the network below starts from it, and mean, spread and the 0.99
# quantile of |M|^2 over its prediction follow from it
LOG_ME = {
    'gg_ttxgg': {'coef': {'bb': 0.0, 'bt': -0.541, 'bg': -1.026, 'tt': -1.169, 'tg': -0.058, 'gg': -0.436},
                 'mean': {'bb': 0.0, 'bt': -1.556, 'bg': -1.901, 'tt': -1.947, 'tg': -2.186, 'gg': -2.469},
                 'ymean': -15.147, 'ystd': 1.884, 'x_max': 2.58},
    'gg_ttxggg': {'coef': {'bb': 0.0, 'bt': -0.403, 'bg': -0.860, 'tt': -1.372, 'tg': -0.038, 'gg': -0.379},
                  'mean': {'bb': 0.0, 'bt': -1.696, 'bg': -2.163, 'tt': -2.333, 'tg': -2.671, 'gg': -3.077},
                  'ymean': -22.221, 'ystd': 2.173, 'x_max': 4.98},
}


def listed():
    return [
        # a program that asks event by event or in small groups: launches and latency
        {'name': 'me ttx 64', 'kind': 'me', 'process': 'gg_ttx', 'nevt': 64, 'mode': 'fp64', 'running': False},
        # a small segment with the coupling of each event from its own scale
        {'name': 'me ttxg 8192 running', 'kind': 'me', 'process': 'gg_ttxg', 'nevt': 8192, 'mode': 'fp64',
         'running': True},
        # production batches
        {'name': 'me ttxgg 524288', 'kind': 'me', 'process': 'gg_ttxgg', 'nevt': 524288, 'mode': 'fp64',
         'running': False},
        {'name': 'me ttxggg 262144', 'kind': 'me', 'process': 'gg_ttxggg', 'nevt': 262144, 'mode': 'fp64',
         'running': False},
        # the split FP16 colour sum, on a ragged batch
        {'name': 'me ttxggg 100003 fp16', 'kind': 'me', 'process': 'gg_ttxggg', 'nevt': 100003, 'mode': 'fp16',
         'running': False},
        # what is left of a batch after a first selection: fewer events than fill the chip many times
        {'name': 'me ttxggg 1000', 'kind': 'me', 'process': 'gg_ttxggg', 'nevt': 1000, 'mode': 'fp64',
         'running': False},
        # six gluons, 720 colour flows
        {'name': 'me ttxgggg 4096', 'kind': 'me', 'process': 'gg_ttxgggg', 'nevt': 4096, 'mode': 'fp64',
         'running': False},
        # event output: the helicity and colour flow of every event
        {'name': 'select ttxggg 16384', 'kind': 'select', 'process': 'gg_ttxggg', 'nevt': 16384},
        # two-stage unweighting of a batch, the whole call
        {'name': 'unweight ttxggg 262144', 'kind': 'unweight', 'process': 'gg_ttxggg', 'nevt': 262144},
        # its maxima, from a calibration sample
        {'name': 'calibrate 65536', 'kind': 'calibrate', 'nevt': 65536, 'quantile': 0.99},
        # one optimiser step on a minibatch
        {'name': 'train 4096', 'kind': 'train', 'process': 'gg_ttxggg', 'nevt': 4096, 'width': 256, 'depth': 4},
        # the surrogate on a large sample
        {'name': 'predict ttxgg 1048576', 'kind': 'predict', 'process': 'gg_ttxgg', 'nevt': 1048576, 'width': 256,
         'depth': 4},
    ]


def _size(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi], odd ones as often as even ones."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(['me', 'me', 'me', 'me', 'select', 'unweight', 'calibrate', 'train', 'predict'])
    if kind == 'me':
        p = rng.choice(sorted(NPAR))
        # the one-lane and six-gluon handles run the FP64 colour sum, as the autotuned ones do
        mode = rng.choice(['fp64', 'fp64', 'fp16', 'bf16']) if p in ('gg_ttxgg', 'gg_ttxggg') else 'fp64'
        return {'kind': kind, 'process': p, 'nevt': _size(rng, 8, MOST[p]), 'mode': mode,
                'running': rng.random() < 0.25}
    if kind == 'select':
        p = rng.choice(['gg_ttx', 'gg_ttxg', 'gg_ttxgg', 'gg_ttxggg'])
        return {'kind': kind, 'process': p, 'nevt': _size(rng, 64, 16384 if p == 'gg_ttxggg' else 65536)}
    if kind == 'unweight':
        return {'kind': kind, 'process': rng.choice(sorted(LOG_ME)), 'nevt': _size(rng, 8192, 262144)}
    if kind == 'calibrate':
        return {'kind': kind, 'nevt': _size(rng, 1024, 262144), 'quantile': rng.choice([0.9, 0.99, 0.999, 1.0])}
    p = rng.choice(sorted(LOG_ME))
    width, depth = rng.choice([64, 128, 256]), rng.choice([2, 3, 4])
    if kind == 'train':
        return {'kind': kind, 'process': p, 'nevt': _size(rng, 256, 8192), 'width': width, 'depth': depth}
    return {'kind': kind, 'process': p, 'nevt': _size(rng, 1024, 1048576), 'width': width, 'depth': depth}


# ------------------------------------------------------------------ inputs

def _device():
    return torch.device('cuda:0')


def _generator(seed):
    return torch.Generator(device=_device()).manual_seed(seed)


def _rand(shape, gen):
    return torch.rand(shape, dtype=torch.float64, device=_device(), generator=gen)


def phase_space(npar, n, gen):
    """Flat phase-space points momenta[n][npar][4] and their weights."""
    nf = npar - 2
    r = _rand((n, nf, 4), gen)
    c, f = 2.0 * r[..., 0] - 1.0, 2.0 * math.pi * r[..., 1]
    s = (1.0 - c * c).clamp_min(0.0).sqrt()
    q0 = -torch.log((1.0 - r[..., 2]) * (1.0 - r[..., 3]))
    q = q0[..., None] * torch.stack([s * f.cos(), s * f.sin(), c], -1)
    # conformal boost to the rest frame of the sum, then one common scale onto the mass shells
    tot, e = q.sum(1), q0.sum(1)
    mass = (e * e - (tot * tot).sum(-1)).sqrt()
    b, gam = -tot / mass[:, None], e / mass
    bq = (b[:, None, :] * q).sum(-1)
    q = q + b[:, None, :] * (q0 + bq / (1.0 + gam)[:, None])[..., None]
    q = (SQRTS / mass)[:, None, None] * q
    q = q - q.mean(1, keepdim=True)
    m2 = torch.zeros(nf, dtype=torch.float64, device=_device())
    m2[:2] = MT * MT
    p2 = (q * q).sum(-1)
    xi = torch.full((n, 1), math.sqrt(1.0 - (2.0 * MT / SQRTS) ** 2), dtype=torch.float64, device=_device())
    for _ in range(12):
        e = (m2 + xi * xi * p2).sqrt()
        xi = xi - (e.sum(1, keepdim=True) - SQRTS) / (xi * p2 / e).sum(1, keepdim=True)
    mom = torch.zeros((n, npar, 4), dtype=torch.float64, device=_device())
    mom[:, :2, 0] = 0.5 * SQRTS
    mom[:, 0, 3], mom[:, 1, 3] = 0.5 * SQRTS, -0.5 * SQRTS
    mom[:, 2:, 1:] = xi[..., None] * q
    mom[:, 2:, 0] = (m2 + xi * xi * p2).sqrt()
    k = xi * p2.sqrt()
    e = mom[:, 2:, 0]
    w0 = ((2.0 * math.pi) ** (4 - 3 * nf) * (math.pi / 2.0) ** (nf - 1) * SQRTS ** (2 * nf - 4)
          / (math.factorial(nf - 1) * math.factorial(nf - 2)))
    wps = (w0 * (k.sum(1) / SQRTS) ** (2 * nf - 3) * (k / e).prod(1) * SQRTS / (k * k / e).sum(1))
    return mom, wps


def _pairs(npar):
    kind = lambda q: 'b' if q < 2 else 't' if q < 4 else 'g'  # noqa: E731
    return [kind(i) + kind(j) for i in range(npar) for j in range(i + 1, npar)]


def _normalisation(process):
    """Feature mean and inverse spread, as a fit of the surrogate's inputs leaves them."""
    mean = [LOG_ME[process]['mean'][k] for k in _pairs(NPAR[process])]
    return np.array(mean, dtype=np.float32), np.ones(len(mean), dtype=np.float32)


def _weights(process, width, depth, seed, fitted=True):
    """Parameters of a network, flat, W then b, layer by layer: fitted, its first two units carry the linear fit
    of log|M|^2 (silu(z) - silu(-z) = z) and the others are small corrections; else as training starts."""
    fit, rng = LOG_ME[process], np.random.Generator(np.random.PCG64(seed))
    nin = len(_pairs(NPAR[process]))
    flat = []
    for layer in range(depth + 1):
        out = 1 if layer == depth else width
        w = rng.uniform(-1.0, 1.0, (out, nin)) * math.sqrt(3.0 / nin)
        b = rng.uniform(-0.1, 0.1, out)
        if fitted and layer == 0:
            w[0] = [fit['coef'][k] / fit['ystd'] for k in _pairs(NPAR[process])]
            w[1] = -w[0]
        elif fitted and layer < depth:
            w[:2] = 0.0
            w[0, 0], w[0, 1], w[1, 0], w[1, 1] = 1.0, -1.0, -1.0, 1.0
        elif fitted:
            w *= 0.1
            w[0, 0], w[0, 1] = 1.0, -1.0
        if fitted:
            b[:2 if layer < depth else 1] = 0.0
        flat += [w.reshape(-1), b]
        nin = out
    return np.concatenate(flat).astype(np.float32)


def _linear_fit(process, mom):
    """Normalised log|M|^2 of the linear fit (float64)."""
    fit = LOG_ME[process]
    x = _log_invariants(mom)
    mean = torch.tensor([fit['mean'][k] for k in _pairs(NPAR[process])], dtype=torch.float64, device=mom.device)
    coef = torch.tensor([fit['coef'][k] for k in _pairs(NPAR[process])], dtype=torch.float64, device=mom.device)
    return ((x - mean) * coef).sum(1) / fit['ystd']


def _handle(process, mode='fp64'):
    h = binding.MatrixElement(process, colorsum_mode=MODES[mode])
    _tune(h, process)
    return h


def _tune(h, process):
    """The executor that the autotuner picks for the process."""
    if process in ('gg_ttxgg', 'gg_ttxggg', 'gg_ttxgggg'):
        h.me_set_executor(binding.ME_EXEC_BG)
        h.me_set_bg(2 if process == 'gg_ttxgggg' else 4)


def _training_inputs(case, gen):
    """Feature rows and targets of a minibatch: normalised log invariants, and the normalised log|M|^2 of the
    linear fit with the spread around it that the exact one has."""
    p = case['process']
    mom, _ = phase_space(NPAR[p], case['nevt'], gen)
    sur = binding.Surrogate(len(_pairs(NPAR[p])), case['width'], case['depth'], seed=1)
    sur.me_sur_set_normalisation(*_normalisation(p))
    feat = torch.empty((case['nevt'], sur.kpad), dtype=torch.int16, device=_device())
    sur.me_sur_features(mom, case['nevt'], NPAR[p], feat, None, torch.cuda.current_stream())
    noise = torch.randn(case['nevt'], dtype=torch.float64, device=_device(), generator=gen)
    return sur, feat, (_linear_fit(p, mom) + 0.2 * noise).float()


def prepare(case, seed):
    gen, n, kind = _generator(seed), case['nevt'], case['kind']
    dev = _device()
    empty = lambda *s, dt=torch.float64: torch.empty(s, dtype=dt, device=dev)  # noqa: E731
    s = {'case': case, 'stream': torch.cuda.current_stream()}
    if kind == 'me':
        s['mom'], _ = phase_space(NPAR[case['process']], n, gen)
        s['alphas'] = 0.08 + 0.12 * _rand((n,), gen) if case['running'] else None
        s['me'], s['out'] = _handle(case['process'], case['mode']), empty(n)
    elif kind == 'select':
        s['mom'], _ = phase_space(NPAR[case['process']], n, gen)
        s['r'] = _rand((2, n), gen)
        s['me'], s['out'] = _handle(case['process']), empty(n)
        s['hel'], s['col'] = empty(n, dt=torch.int32), empty(n, dt=torch.int32)
    elif kind == 'unweight':
        p = case['process']
        fit = LOG_ME[p]
        s['mom'], s['wps'] = phase_space(NPAR[p], n, gen)
        s['r'] = _rand((2, n), gen)
        pipe = SurrogatePipeline(p, width=256, depth=4, seed=11, alpha_s=ALPHA_S,
                                 colorsum_mode=binding.ME_CS_FP16X2)
        _tune(pipe.me, p)
        pipe.sur.me_sur_set_normalisation(*_normalisation(p))
        pipe.sur.me_sur_set_params(_weights(p, 256, 4, seed))
        pipe.ymean, pipe.ystd = fit['ymean'], fit['ystd']
        what = torch.exp(_linear_fit(p, s['mom']) * fit['ystd'] + fit['ymean']) * s['wps']
        s['what_max'] = float(what.sort().values[int(0.99 * (n - 1))])
        s['x_max'], s['pipe'] = fit['x_max'], pipe
    elif kind == 'calibrate':
        # network outputs, phase-space weights and exact |M|^2 around the prediction
        s['y'] = torch.randn(n, dtype=torch.float64, device=dev, generator=gen).float()
        s['wps'] = torch.exp(-25.0 + 1.5 * torch.randn(n, dtype=torch.float64, device=dev, generator=gen))
        noise = torch.randn(n, dtype=torch.float64, device=dev, generator=gen)
        s['me2'] = torch.exp(s['y'].double() * 2.173 - 22.221 + 0.4 * noise)
    elif kind == 'train':
        s['sur'], s['feat'], s['target'] = _training_inputs(case, gen)
        s['sur'].me_sur_set_params(_weights(case['process'], case['width'], case['depth'], seed, fitted=False))
        s['loss'] = torch.zeros(1, dtype=torch.float32, device=dev)
    else:
        p = case['process']
        s['mom'], _ = phase_space(NPAR[p], n, gen)
        s['sur'] = binding.Surrogate(len(_pairs(NPAR[p])), case['width'], case['depth'], seed=1)
        s['sur'].me_sur_set_normalisation(*_normalisation(p))
        s['sur'].me_sur_set_params(_weights(p, case['width'], case['depth'], seed))
        s['feat'] = empty(n, s['sur'].kpad, dt=torch.int16)
        s['y'] = empty(n, dt=torch.float32)
    return s


def run(s):
    case, st = s['case'], s['stream']
    kind, n = case['kind'], case['nevt']
    if kind == 'me':
        if s['alphas'] is not None:
            s['me'].me_compute_alphas(s['mom'], n, s['alphas'], s['out'], st)
        else:
            s['me'].me_compute(s['mom'], n, ALPHA_S, s['out'], st)
        return {'me2': s['out']}
    if kind == 'select':
        s['me'].me_select(s['mom'], n, ALPHA_S, s['r'][0], s['r'][1], s['out'], s['hel'], s['col'], st)
        return {'me2': s['out'], 'hel': s['hel'], 'col': s['col']}
    if kind == 'unweight':
        res = s['pipe'].unweight(s['mom'], s['wps'], s['r'][0], s['r'][1], s['what_max'], s['x_max'])
        # the weight of every event of the batch: its residual weight, 0 where a stage rejected it
        weight = torch.zeros(n, dtype=torch.float64, device=s['mom'].device)
        weight[res['index']] = res['resid']
        return {'weight': weight, **{k: res[k] for k in ('stage1', 'accepted', 'overweight', 'sum_w', 'sum_w2')}}
    if kind == 'calibrate':
        return list(binding.me_unweight_maxima(s['y'], s['wps'], s['me2'], n, -22.221, 2.173, case['quantile'], st))
    if kind == 'train':
        s['loss'].zero_()
        s['sur'].me_sur_train_step(s['feat'], s['target'], n, 1e-4, s['loss'], st)
        return {'grads': s['sur'].me_sur_get_grads(), 'loss': s['loss']}
    s['sur'].me_sur_features(s['mom'], n, NPAR[case['process']], s['feat'], None, st)
    s['sur'].me_sur_predict(s['feat'], n, s['y'], st)
    return {'feat': s['feat'], 'y': s['y']}


# ------------------------------------------------------------------ work

def _net_sizes(case):
    nin = len(_pairs(NPAR[case['process']]))
    sizes = [nin] + [case.get('width', 256)] * case.get('depth', 4) + [1]
    return list(zip(sizes[:-1], sizes[1:]))


def _me_flops(process):
    """Operations of the colour form of one event: for each pair of mirrored helicities (equal |M|^2) half of the
    symmetric matrix on the real and imaginary parts of the flows.  The flows themselves are not counted."""
    n = NPAR[process] - 2
    ncol = math.factorial(n)
    return 2.0 ** (n + 1) * 2.0 * (ncol * (ncol + 1) // 2 * 2 + 2 * ncol)


def work(case):
    n, kind = case['nevt'], case['kind']
    if kind in ('me', 'select'):
        npar = NPAR[case['process']]
        per = 32 * npar + 8 + (8 if case.get('running') else 0) + (24 if kind == 'select' else 0)
        return {'bytes': n * per, 'flops': n * _me_flops(case['process'])}
    if kind == 'unweight':
        net = sum(2 * a * b for a, b in _net_sizes(case))
        # every event through the network; about one in fifty through the exact |M|^2
        return {'bytes': n * (32 * NPAR[case['process']] + 24), 'flops': n * (net + 0.02 * _me_flops(case['process']))}
    if kind == 'calibrate':
        return {'bytes': 20 * n, 'flops': 30 * n}
    params = sum(a * b + b for a, b in _net_sizes(case))
    net = sum(2 * a * b for a, b in _net_sizes(case))
    kpad = 16 * math.ceil(len(_pairs(NPAR[case['process']])) / 16)
    if kind == 'train':
        return {'bytes': n * (2 * kpad + 4) + 28 * params, 'flops': 3 * n * net}
    return {'bytes': n * (32 * NPAR[case['process']] + 2 * kpad + 4) + 2 * params, 'flops': n * net}


# ------------------------------------------------------------------ values in 64 bits

def _dot(a, b):
    return a[..., 0] * b[..., 0] - a[..., 1] * b[..., 1] - a[..., 2] * b[..., 2] - a[..., 3] * b[..., 3]


def _log_invariants(mom):
    npar = mom.shape[1]
    s = _dot(mom[:, 0] + mom[:, 1], mom[:, 0] + mom[:, 1])
    return torch.stack([torch.log(2.0 * _dot(mom[:, i], mom[:, j]) / s)
                        for i in range(npar) for j in range(i + 1, npar)], 1)


def _colour_matrix(n):
    """Tr(T^{s_n} .. T^{s_1} T^{t_1} .. T^{t_n}) over the orderings s, t of n gluons, SU(3): each pair of equal
    generators is 1/2 (exchange - 1/3 identity) on the colour lines, and closed lines count 3 each."""
    perms = list(itertools.permutations(range(n)))

    def trace(t):
        """s = identity: the word n-1 .. 0 t_0 .. t_{n-1}, 2 n generators on one closed line."""
        word = list(range(n))[::-1] + list(t)
        where = {g: [i for i, x in enumerate(word) if x == g] for g in range(n)}
        total = 0.0
        for cut in range(1 << n):
            # next line segment after each generator: itself (identity) or its partner's (exchange)
            sign, nxt = 1.0, list(range(2 * n))
            for g in range(n):
                i, j = where[g]
                if cut >> g & 1:
                    sign *= -1.0 / 3.0
                else:
                    nxt[i], nxt[j] = j, i
            seen, loops = [False] * (2 * n), 0
            for k in range(2 * n):
                if not seen[k]:
                    loops += 1
                    while not seen[k]:
                        seen[k] = True
                        k = nxt[(k + 1) % (2 * n)]
            total += sign * 3.0 ** loops
        return total / 2 ** n

    row = {t: trace(t) for t in perms}
    inv = {s: tuple(s.index(i) for i in range(n)) for s in perms}
    return torch.tensor([[row[tuple(inv[s][g] for g in t)] for t in perms] for s in perms], dtype=torch.float64,
                        device=_device())


def _gamma():
    s = [[[1, 0], [0, 1]], [[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]]
    g = torch.zeros((4, 4, 4), dtype=torch.complex128, device=_device())
    for mu in range(4):
        m = torch.tensor(s[mu], dtype=torch.complex128, device=_device())
        g[mu, :2, 2:] = m
        g[mu, 2:, :2] = m if mu == 0 else -m
    return g


def _slash(gam, p):
    p = p.to(torch.complex128)
    return sum(p[..., mu, None, None] * gam[mu] * (1.0 if mu == 0 else -1.0) for mu in range(4))


def _exact_me(mom, alphas, colour):
    """Helicity- and colour-summed, averaged |M|^2 by the colour-ordered recursion, in 64 bits: linear gluon
    polarisations (the sum over them is that over the helicities), all of them in one tensor dimension."""
    e, npar = mom.shape[0], mom.shape[1]
    n = npar - 2
    gam = _gamma()
    g = torch.sqrt(4.0 * math.pi * alphas)[None, :, None]
    # external gluons: momentum into the diagram, and both polarisations spread over the 2^n combinations
    ext, pin = [], []
    combos = torch.arange(1 << n, device=mom.device)
    for b in range(n):
        k = mom[:, b if b < 2 else b + 2]
        kt = (k[:, 1] ** 2 + k[:, 2] ** 2).sqrt()
        cf, sf = torch.where(kt > 0, k[:, 1] / kt, 1.0), torch.where(kt > 0, k[:, 2] / kt, 0.0)
        kabs = (kt ** 2 + k[:, 3] ** 2).sqrt()
        ct, st, zero = k[:, 3] / kabs, kt / kabs, torch.zeros_like(kt)
        e1, e2 = torch.stack([zero, ct * cf, ct * sf, -st], 1), torch.stack([zero, -sf, cf, zero], 1)
        pick = (combos >> b & 1).bool()[:, None, None]
        ext.append(torch.where(pick, e1[None], e2[None]))
        pin.append(k if b < 2 else -k)
    psum = {}
    for m in range(1, 1 << n):
        psum[m] = sum(pin[b] for b in range(n) if m >> b & 1)
    bits = lambda seq: sum(1 << b for b in seq)  # noqa: E731
    cur = {(b,): ext[b] for b in range(n)}
    for length in range(2, n + 1):
        for seq in itertools.permutations(range(n), length):
            acc = 0.0
            for j in range(1, length):
                a, b = cur[seq[:j]], cur[seq[j:]]
                pa, pb = psum[bits(seq[:j])][None], psum[bits(seq[j:])][None]
                acc = acc - g * (a * _dot(-2.0 * pa - pb, b)[..., None] + _dot(a, b)[..., None] * (pa - pb)
                                 + b * _dot(2.0 * pb + pa, a)[..., None])
            for j in range(1, length - 1):
                for k in range(j + 1, length):
                    a, b, c = cur[seq[:j]], cur[seq[j:k]], cur[seq[k:]]
                    acc = acc - g * g * (a * _dot(b, c)[..., None] - 2.0 * b * _dot(a, c)[..., None]
                                         + c * _dot(a, b)[..., None])
            p = psum[bits(seq)]
            cur[seq] = acc / _dot(p, p)[None, :, None]
    # top line: the rows of sqrt(2E)-normalised spinors are those of (pslash + m), rank two, as are those of
    # (pslash - m) of the antitop: spin sums sqrt-factored by two independent rows each
    top, anti = _slash(gam, mom[:, 2]), _slash(gam, mom[:, 3])
    eye = torch.eye(4, dtype=torch.complex128, device=mom.device)
    ubar = _factor(top + MT * eye, gam)            # [2][e][4]
    v = _factor(anti - MT * eye, gam).conj() @ gam[0]
    rows = {(): ubar[:, None].expand(2, 1 << n, e, 4)}
    amps = []
    sl = lambda r, j: _row_slash(r, j)  # noqa: E731
    gc = (1j * g)[None]
    for length in range(1, n + 1):
        new = {}
        for seq in itertools.permutations(range(n), length):
            acc = sum(sl(rows[seq[:i]], cur[seq[i:]][None]) for i in range(length)) * gc
            if length == n:
                amps.append((acc[:, None] * v[None, :, None]).sum(-1))   # [2][2][combos][e]
            else:
                q = mom[:, 2] - psum[bits(seq)]
                prop = 1j * (_slash(gam, q) + MT * eye) / (_dot(q, q) - MT * MT)[:, None, None]
                new[seq] = (acc[..., None, :] @ prop[None, None])[..., 0, :]
        rows.update(new)
    a = torch.stack(amps)
    a = torch.cat([a.real, a.imag], 1).reshape(a.shape[0], -1)
    form = ((colour @ a) * a).sum(0).reshape(-1, e).sum(0)
    return form / (256.0 * math.factorial(npar - 4))


def _row_slash(r, j):
    """r . gamma.j for rows r [..., 4] and real vectors j [..., 4], in two-component blocks."""
    j0, j1, j2, j3 = (j[..., k] for k in range(4))
    r0, r1, r2, r3 = (r[..., k] for k in range(4))
    js, jd = torch.complex(j1, j2), torch.complex(j1, -j2)
    return torch.stack([r2 * (j0 + j3) + r3 * js, r2 * jd + r3 * (j0 - j3), r0 * (j0 - j3) - r1 * js,
                        r1 * (j0 + j3) - r0 * jd], -1)


def _factor(m, gam):
    """Rows x_s, s = 0, 1, with sum_s xbar_s^dagger-weighted outer products equal to the rank-two matrix m:
    m gamma^0 is Hermitian and semidefinite, = sum_s w_s w_s^dagger; the rows are w_s^dagger gamma^0."""
    val, vec = torch.linalg.eigh(m @ gam[0])
    w = vec[..., 2:] * val[..., None, 2:].clamp_min(0.0).sqrt()
    return w.conj().permute(2, 0, 1) @ gam[0]


def _exact_net(flat, sizes, x):
    off = 0
    for k, (nin, out) in enumerate(sizes):
        w = flat[off:off + nin * out].reshape(out, nin)
        b = flat[off + nin * out:off + nin * out + out]
        off += nin * out + out
        x = x @ w.T + b
        if k + 1 < len(sizes):
            x = x * torch.sigmoid(x)
    return x[:, 0]


# events that the recursion above does in a few seconds, and per chunk
_EXACT_EVENTS = {'gg_ttx': 524288, 'gg_ttxg': 524288, 'gg_ttxgg': 524288, 'gg_ttxggg': 131072, 'gg_ttxgggg': 2048}
_EXACT_CHUNK = {'gg_ttx': 131072, 'gg_ttxg': 32768, 'gg_ttxgg': 16384, 'gg_ttxggg': 2048, 'gg_ttxgggg': 128}


def exact(case, seed):
    kind, n = case['kind'], case['nevt']
    if kind in ('me', 'select'):
        p = case['process']
        if n > _EXACT_EVENTS[p]:
            return None
        gen = _generator(seed)
        mom, _ = phase_space(NPAR[p], n, gen)
        alphas = 0.08 + 0.12 * _rand((n,), gen) if case.get('running') else torch.full_like(mom[:, 0, 0], ALPHA_S)
        colour, step = _colour_matrix(NPAR[p] - 2), _EXACT_CHUNK[p]
        me2 = torch.cat([_exact_me(mom[i:i + step], alphas[i:i + step], colour) for i in range(0, n, step)])
        return {'me2': me2} if kind == 'me' else {'me2': me2, 'hel': None, 'col': None}
    if kind == 'calibrate':
        s = prepare(case, seed)
        what = torch.exp(s['y'].double() * 2.173 - 22.221) * s['wps']
        x = s['me2'] * s['wps'] / what
        pos = min(1.0, case['quantile']) * (n - 1)
        lo = int(math.floor(pos))
        got = []
        for v in (what, x):
            v = v.sort().values
            a, b = float(v[lo]), float(v[min(lo + 1, n - 1)])
            got.append(a + (b - a) * (pos - lo))
        return got
    if kind == 'train':
        _, feat, target = _training_inputs(case, _generator(seed))
        sizes = _net_sizes(case)
        flat = _weights(case['process'], case['width'], case['depth'], seed, fitted=False)
        flat = torch.from_numpy(flat).double().to(_device()).requires_grad_(True)
        x = feat.view(torch.bfloat16).double()[:, :sizes[0][0]]
        sq = (_exact_net(flat, sizes, x) - target.double()).square()
        sq.mean().backward()
        return {'grads': flat.grad, 'loss': sq.sum().detach().reshape(1)}
    if kind == 'predict':
        p = case['process']
        mom, _ = phase_space(NPAR[p], n, _generator(seed))
        mean = torch.from_numpy(_normalisation(p)[0]).double().to(_device())
        flat = torch.from_numpy(_weights(p, case['width'], case['depth'], seed)).double().to(_device())
        step = 131072
        y = torch.cat([_exact_net(flat, _net_sizes(case), _log_invariants(mom[i:i + step]) - mean)
                       for i in range(0, n, step)])
        return {'feat': None, 'y': y}
    return None   # unweighting: its accepted events are whole numbers
