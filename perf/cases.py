"""The work this framework is used for, as cases that can be timed.

A case is one pass through the public entry points, the way a program calls
them: a whole simulator run (smc_run, smc_run_batch), or one of the calls that
a program drives by itself (an M iteration by random walk or Langevin step,
the first C and S phases, the likelihood, its gradient through autograd, the
posterior report).  Sizes are those of the workloads in the tests, the tuner
and bench.py (egarch11: 16 x 1,024 particles, T = 5,000; egarch2t and
egarch23: 64 x 1,024, T = 10,000 and 5,100; linreg: 4 x 256, T = 200) and
ragged ones around them.

listed() gives the cases, draw(rng) another of the same ranges, prepare(case,
seed) what a program holds before the call, run(state) one pass, work(case)
the bytes and operations a pass cannot do without, and exact(case, seed) the
outputs in plain 64-bit torch where they have such a value.
"""
import math

import numpy as np
import torch

import paper_1304_4334_amd as smc
from paper_1304_4334_amd import autograd, tune

GAUSS, STUDENT_T, MIXTURE = smc.SMC_SHOCK_GAUSS, smc.SMC_SHOCK_STUDENT_T, smc.SMC_SHOCK_MIXTURE

# Model families: (factors K, shock, mixture components I).
FAMILY = {"egarch11": (1, GAUSS, 0), "egarch2g": (2, GAUSS, 0), "egarch1t": (1, STUDENT_T, 0),
          "egarch2t": (2, STUDENT_T, 0), "egarch12": (1, MIXTURE, 2), "egarch23": (2, MIXTURE, 3),
          "egarch34": (3, MIXTURE, 4)}


def listed():
    return [
        # One likelihood surface evaluation of the mixture model at a few
        # hundred points: the smallest call, a chain of 777 observations.
        dict(name="loglik egarch23 f64 300", do="loglik", model="egarch23", bits=64, J=1, N=300, T=777),
        # A regression posterior from 200 observations, a run of 1,024
        # particles: launches and host decisions.
        dict(name="run linreg f64 1k", do="run", model="linreg", bits=64, J=4, N=256, T=200, every=20, graph=False),
        # The start of every run: prior draws, the first C phase up to its
        # stopping date, the first resampling.
        dict(name="cycle egarch2t f32 16k", do="cycle", model="egarch2t", bits=32, J=16, N=1000, T=2000),
        # Gradient of the log likelihood for an optimiser or a chain driven
        # from outside, ragged sizes.
        dict(name="gradient egarch2t f64 1000", do="gradient", model="egarch2t", bits=64, J=1, N=1000, T=1237),
        # Posterior report at a date: moments with their numerical errors,
        # functions of interest, relative efficiency, log marginal likelihood.
        dict(name="report egarch11 f64 65k", do="report", model="egarch11", bits=64, J=64, N=1024, T=500),
        # The same gradient for a population's worth of parameter vectors.
        dict(name="gradient egarch11 f64 4k", do="gradient", model="egarch11", bits=64, J=1, N=4096, T=5000),
        # An M iteration by the Langevin step, population of 16,384.
        dict(name="langevin egarch2t f32 16k", do="langevin", model="egarch2t", bits=32, J=16, N=1024, T=2500),
        # M iterations by the random walk driven call by call, at the two
        # heavy families' full populations.
        dict(name="step egarch23 f32 65k", do="step", model="egarch23", bits=32, J=64, N=1024, T=5100),
        dict(name="step egarch2t f64 65k", do="step", model="egarch2t", bits=64, J=64, N=1024, T=2500),
        # Whole adaptive runs at the two EGARCH workloads' full sizes.
        dict(name="run egarch11 f64 16k", do="run", model="egarch11", bits=64, J=16, N=1024, T=5000, every=0, graph=False),
        dict(name="run egarch2t f32 65k", do="run", model="egarch2t", bits=32, J=64, N=1024, T=10000, every=0, graph=False),
        # Eight series analysed together, both EGARCH families, populations
        # of 4,096 to 32,768.
        dict(name="batch 8 runs f32", do="batch", model="mixed", bits=32, J=16, N=256, T=4000, runs=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["loglik", "loglik", "run", "run", "cycle", "gradient", "gradient", "report",
                     "langevin", "step", "step", "batch"])
    bits = rng.choice([32, 64])
    model = rng.choice(sorted(FAMILY))
    if do in ("loglik", "gradient"):
        return dict(do=do, model=model, bits=bits, J=1, N=_log(rng, 50, 20000), T=_log(rng, 100, 5000))
    if do == "run":
        if rng.random() < 0.25:
            return dict(do=do, model="linreg", bits=64, J=rng.choice([4, 7, 16]), N=_log(rng, 100, 1500),
                        T=_log(rng, 100, 600), every=20, graph=rng.random() < 0.3)
        return dict(do=do, model=rng.choice(["egarch11", "egarch2t", "egarch23"]), bits=bits,
                    J=rng.choice([4, 8, 15, 16, 32]), N=_log(rng, 100, 1500), T=_log(rng, 200, 3000),
                    every=0, graph=rng.random() < 0.3)
    if do == "batch":
        return dict(do=do, model="mixed", bits=32, J=rng.choice([4, 8, 16]), N=_log(rng, 64, 256),
                    T=_log(rng, 500, 3000), runs=rng.choice([2, 3, 5, 8]))
    if do == "cycle":
        return dict(do=do, model=model, bits=bits, J=rng.choice([4, 16, 33, 64]), N=_log(rng, 100, 2500), T=2000)
    if do == "report":
        return dict(do=do, model=rng.choice(["egarch11", "egarch2g", "egarch23", "egarch34"]), bits=64,
                    J=rng.choice([4, 16, 33, 64]), N=_log(rng, 100, 2500), T=_log(rng, 100, 1000))
    if do == "langevin":
        return dict(do=do, model=rng.choice(["egarch11", "egarch2t", "egarch23"]), bits=bits,
                    J=rng.choice([4, 16, 33]), N=_log(rng, 100, 1500), T=_log(rng, 200, 2500))
    return dict(do=do, model=model, bits=bits, J=rng.choice([4, 16, 33, 64]), N=_log(rng, 100, 1500),
                T=_log(rng, 200, 5000))


# ---- inputs ----------------------------------------------------------------

def _truth(model):
    """Parameters of the simulated series, in the models' coordinates: mu_Y
    (thousandths), log sigma_Y, atanh of the persistences, log loadings,
    leverages, then the shock's own."""
    K, shock, I = FAMILY[model]
    th = [0.3, math.log(0.01)]
    th += [math.atanh(a) for a in (0.98, 0.80, 0.6)[:K]]
    th += [math.log(b) for b in (0.08, 0.15, 0.1)[:K]]
    th += [-0.04, -0.08, -0.02][:K]
    if shock == STUDENT_T:
        th += [math.log(6.0)]
    if shock == MIXTURE:
        p = {2: [0.85, 0.15], 3: [0.6, 0.3, 0.1], 4: [0.5, 0.25, 0.15, 0.1]}[I]
        m = {2: [0.06, -0.34], 3: [0.08, 0.02, -0.54], 4: [0.1, -0.02, 0.05, -0.525]}[I]
        s = list(np.linspace(0.7, 1.9, I))
        mean = sum(a * b for a, b in zip(p, m))
        m = [x - mean for x in m]
        c = 1.0 / math.sqrt(sum(a * (x * x + v * v) for a, x, v in zip(p, m, s)))
        th += [math.atanh(a - 1.0) for a in p] + [c * x for x in m] + [math.log(c * v) for v in s]
    return np.array(th)


def _series(model, T, rng):
    """A simulated return series of the family (or a regression's y and X)."""
    if model == "linreg":
        X = rng.standard_normal((T, 3))
        return X @ np.array([1.0, -0.5, 0.25]) + 0.8 * rng.standard_normal(T), X
    K, shock, I = FAMILY[model]
    th = _truth(model)
    a, b, g = np.tanh(th[2:2 + K]), np.exp(th[2 + K:2 + 2 * K]), th[2 + 2 * K:2 + 3 * K]
    if shock == STUDENT_T:
        nu = 2.0 + math.exp(th[-1])
        z = rng.standard_t(nu, T) * math.sqrt((nu - 2.0) / nu)
    elif shock == MIXTURE:
        q = 2 + 3 * K
        p = np.tanh(th[q:q + I]) + 1.0
        i = rng.choice(I, size=T, p=p / p.sum())
        z = th[q + I + i] + np.exp(th[q + 2 * I + i]) * rng.standard_normal(T)
    else:
        z = rng.standard_normal(T)
    push = b * (np.abs(z[:, None]) - math.sqrt(2.0 / math.pi)) + g * z[:, None]
    v, lh = np.zeros(K), np.empty(T)
    for t in range(T):
        lh[t] = v.sum()
        v = a * v + push[t]
    return th[0] / 1000.0 + np.exp(th[1] + 0.5 * lh) * z, None


def _model(case, rng, model=None, T=None):
    name = model or case["model"]
    prec = smc.SMC_FP32 if case["bits"] == 32 else smc.SMC_FP64
    y, X = _series(name, T or case["T"], rng)
    if name == "linreg":
        return smc.Model(smc.SMC_MODEL_LINREG, y, X=X)
    K, shock, I = FAMILY[name]
    m = smc.Model(smc.SMC_MODEL_EGARCH, y, K=K, shock=shock, precision=prec, I=I)
    tune.apply(m, name, "fp%d" % case["bits"])
    return m


def _cloud(case, seed):
    """Parameter vectors spread as a posterior after T observations is, [d, P]."""
    K, shock, I = FAMILY[case["model"]]
    r = 1.0 / math.sqrt(case["T"])
    sd = [10.0 * r, 3.0 * r] + [6.0 * r] * K + [6.0 * r] * K + [1.2 * r] * K
    sd += {GAUSS: [], STUDENT_T: [6.0 * r], MIXTURE: [6.0 * r] * I + [3.0 * r] * (2 * I)}[shock]
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = torch.randn((len(sd), case["J"] * case["N"]), generator=g, dtype=torch.float64, device="cuda")
    return _column(_truth(case["model"])) + _column(np.array(sd)) * n


def _column(x):
    return torch.from_numpy(x).cuda()[:, None]


def _log_prior(model, theta):
    """Log prior density of an EGARCH family's parameters (Table 1)."""
    K, shock, I = FAMILY[model]
    mean = [0.0, math.log(0.01)] + [math.atanh(0.95)] * K + [math.log(0.1)] * K + [0.0] * K
    sd = [1.0] * (2 + 2 * K) + [0.2] * K
    mean += {GAUSS: [], STUDENT_T: [math.log(10.0)], MIXTURE: [0.0] * (3 * I)}[shock]
    sd += [1.0] * (len(mean) - len(sd))
    z = (theta - _column(np.array(mean))) / _column(np.array(sd))
    lp = (-0.5 * z * z - 0.5 * math.log(2.0 * math.pi) - _column(np.log(sd))).sum(0)
    if shock == MIXTURE:  # log scales truncated below at -3
        lp = lp - I * math.log(0.5 * math.erfc(-3.0 / math.sqrt(2.0)))
    return lp


def _population(case, seed, m, grad=False):
    """A population at date T as a run's M phase meets it."""
    pop = smc.Population(m, case["J"], case["N"], max_chunk=16, with_grad=grad)
    pop.theta.copy_(_cloud(case, seed))
    pop.loglik.copy_(smc.smc_loglik(m, pop.theta, case["T"], state_out=pop.state))
    pop.logprior.copy_(_log_prior(case["model"], pop.theta))
    return pop


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    do = case["do"]
    if do == "batch":
        models, pops = [], []
        for r in range(case["runs"]):
            name = "egarch2t" if r % 2 else "egarch11"
            T = case["T"] * (4 + (3 * r) % 8) // 11
            m = _model(case, rng, name, T)
            m.set_launch(*tune.tuned_batch_shape())
            models.append(m)
            pops.append(smc.Population(m, case["J"], case["N"] << (r % 4), max_chunk=256))
        recs = [smc.Record(m, p.J, 256, 21) for m, p in zip(models, pops)]
        bws = torch.empty(smc.lib().smc_batch_ws_bytes(len(models)) + 256, dtype=torch.uint8, device="cuda")
        return dict(do=do, models=models, pops=pops, recs=recs, bws=bws, waves=tune.tuned_waves(),
                    seeds=[seed % 100003 + r for r in range(len(models))])
    m = _model(case, rng)
    s = dict(do=do, m=m, T=case["T"], seed=seed)
    if do in ("loglik", "gradient"):
        s["theta"] = _cloud(case, seed)
        if do == "loglik":
            s["state"] = torch.empty((m.S, case["N"]), dtype=m.state_dtype, device="cuda")
        else:
            s["theta"].requires_grad_(True)
            s["weight"] = torch.from_numpy(rng.uniform(0.5, 1.5, case["N"])).cuda()
    elif do == "report":
        s["pop"] = _population(case, seed, m)
        s["logwbar"] = torch.from_numpy(rng.normal(-40.0, 0.3, (50, case["J"]))).cuda()
    elif do == "cycle":
        s["pop"] = smc.Population(m, case["J"], case["N"], max_chunk=256)
    elif do == "run":
        s["pop"] = smc.Population(m, case["J"], case["N"], max_chunk=1024)
        s["rec"] = smc.Record(m, case["J"], 256, 21)
        s["every"], s["graph"] = case["every"], case["graph"]
    else:
        s["pop"] = _population(case, seed, m, grad=do == "langevin")
        s["hl"] = torch.zeros((m.d, m.d), dtype=torch.float64, device="cuda")
        s["mh"] = torch.full((1,), 5, dtype=torch.int32, device="cuda")
        s["it"] = 0
        if do == "langevin":
            smc.smc_posterior_grad(m, s["pop"], case["T"])
    return s


# ---- one pass --------------------------------------------------------------

def _particles(pop):
    out = dict(theta=pop.theta, logprior=pop.logprior, loglik=pop.loglik)
    if pop.state is not None:
        out["state"] = pop.state
    return out


def _record(rec):
    return dict(log_ml=rec.log_ml, group_logwbar=rec.group_logwbar, n_accept=rec.n_accept, hchol=rec.hchol,
                t_end=rec.t_end, R=rec.R, rss=rec.rss, evals=rec.c.evals, mh_steps=rec.c.mh_steps)


def run(state):
    s, do = state, state["do"]
    if do == "loglik":
        return dict(loglik=smc.smc_loglik(s["m"], s["theta"], s["T"], state_out=s["state"]), state=s["state"])
    if do == "gradient":
        ll = autograd.loglik(s["theta"], s["m"], s["T"])
        (g,) = torch.autograd.grad(ll, s["theta"], s["weight"])
        return dict(loglik=ll, grad=g)
    if do == "report":
        m, pop = s["m"], s["pop"]
        return dict(params=smc.smc_test_moments(m, pop, s["T"], smc.SMC_TEST_PARAMS),
                    functions=smc.smc_test_moments(m, pop, s["T"], smc.SMC_TEST_MODEL),
                    rne=smc.smc_rne(m, pop), log_ml=smc.smc_log_ml(s["logwbar"]))
    if do == "cycle":
        m, pop = s["m"], s["pop"]
        smc.smc_init_from_prior(m, pop, s["seed"])
        t, rss, lw = smc.smc_correct(m, pop, 0, s["T"])
        smc.smc_resample(m, pop, seed=s["seed"], cycle=1)
        return dict(_particles(pop), t=t, rss=rss, group_logwbar=lw, logw=pop.logw, ancestor=pop.ancestor)
    if do == "run":
        smc.smc_run(s["m"], s["pop"], s["seed"], force_every=s["every"], record=s["rec"], graph=s["graph"])
        return dict(_particles(s["pop"]), **_record(s["rec"]))
    if do == "batch":
        smc.smc_run_batch(s["models"], s["pops"], s["seeds"], records=s["recs"], bws=s["bws"], waves=s["waves"])
        return [dict(theta=p.theta, loglik=p.loglik, log_ml=r.log_ml, n_accept=r.n_accept, t_end=r.t_end)
                for p, r in zip(s["pops"], s["recs"])]
    # an M iteration: proposal scale, Metropolis step, step-size rule
    m, pop = s["m"], s["pop"]
    s["it"] += 1
    mala = do == "langevin"
    smc.smc_particle_moments(m, pop, s["mh"], hchol=s["hl"])
    n = smc.smc_mutate(m, pop, s["T"], s["hl"], s["seed"], cycle=1, it=s["it"],
                       kernel=smc.SMC_KERNEL_MALA if mala else smc.SMC_KERNEL_RW)
    smc.smc_adapt_scale(n, pop.P, 574 if mala else 250, s["mh"])
    out = dict(_particles(pop), n=n, hl=s["hl"], mh=s["mh"])
    if mala:
        out["grad"] = pop.grad
    return out


# ---- what a pass cannot do without ----------------------------------------

def _sizes(model):
    if model == "linreg":
        return 4, 0, 9.0
    K, shock, I = FAMILY[model]
    d = 2 + 3 * K + (1 if shock == STUDENT_T else 3 * I)
    # one observation: standardising 3, exponential and scaling 4, a factor 7,
    # the density 4, a component of a mixture 8
    return d, K + 1, 11.0 + 7.0 * K + 8.0 * I


def _run_evals(d, P, T):
    """Typical density evaluations of an adaptive run: about 0.43 d log2 T
    cycles of 7 Metropolis steps at an average date of T/4, and the C phases."""
    return P * T * (1.0 + 0.43 * d * math.log2(T) * 7.0 * 0.25)


def work(case):
    do, P, T = case["do"], case["J"] * case["N"], case["T"]
    if do == "batch":
        b = f = 0.0
        for r in range(case["runs"]):
            d, S, op = _sizes("egarch2t" if r % 2 else "egarch11")
            p, t = P << (r % 4), T * (4 + (3 * r) % 8) // 11
            f += op * _run_evals(d, p, t)
            b += 8.0 * p * (d + 3 + S) + 8.0 * t
        return dict(bytes=b, flops=f)
    d, S, op = _sizes(case["model"])
    w = case["bits"] / 8.0
    if do == "loglik":
        return dict(bytes=P * (8.0 * (d + 1) + w * S) + w * T, flops=op * P * T)
    if do == "gradient":
        return dict(bytes=P * 8.0 * (2 * d + 2) + w * T, flops=3.5 * op * P * T)
    if do == "report":
        return dict(bytes=P * (8.0 * d + w * S), flops=P * (8.0 * d + 60.0))
    if do == "cycle":
        return dict(bytes=P * (8.0 * (2 * d + 4) + w * S + 4.0), flops=P * (16.0 * op + 100.0 * d))
    if do == "run":
        return dict(bytes=P * (8.0 * (d + 3) + w * S) + w * T, flops=op * _run_evals(d, P, T))
    g = 3.5 if do == "langevin" else 1.0
    return dict(bytes=P * (8.0 * 2 * (d + 2) + w * S) + w * T, flops=P * (g * op * T + 2.0 * d * d))


# ---- the same in 64 bits, without this repository's code --------------------

def _density(model, theta, y, v, eps, first):
    """Sum of log p(y_s | y_{1:s-1}, theta) over y, the factors and the shock
    at its end, from those before it (Section 5.1)."""
    K, shock, I = FAMILY[model]
    mu, ls = theta[0] / 1000.0, theta[1]
    a, b, g = torch.tanh(theta[2:2 + K]), torch.exp(theta[2 + K:2 + 2 * K]), theta[2 + 2 * K:2 + 3 * K]
    c = math.sqrt(2.0 / math.pi)
    half = 0.5 * math.log(2.0 * math.pi)
    if shock == STUDENT_T:
        n2 = torch.exp(theta[-1])
        const = torch.lgamma(0.5 * (n2 + 3.0)) - torch.lgamma(0.5 * (n2 + 2.0)) - 0.5 * torch.log(math.pi * n2)
    if shock == MIXTURE:
        q = 2 + 3 * K
        p = torch.tanh(theta[q:q + I]) + 1.0
        p = p / p.sum(0)
        m = theta[q + I:q + 2 * I] - (p * theta[q + I:q + 2 * I]).sum(0)
        sg = torch.exp(theta[q + 2 * I:q + 3 * I])
        scale = 1.0 / torch.sqrt((p * (m * m + sg * sg)).sum(0))
        m, sg = scale * m, scale * sg
        lw = torch.log(p) - torch.log(sg)
    total = torch.zeros_like(mu)
    for k in range(len(y)):
        if not (first and k == 0):
            v = a * v + b * (torch.abs(eps) - c) + g * eps
        lh = ls + 0.5 * v.sum(0)
        eps = (y[k] - mu) * torch.exp(-lh)
        if shock == GAUSS:
            ld = -half - 0.5 * eps * eps
        elif shock == STUDENT_T:
            ld = const - 0.5 * (n2 + 3.0) * torch.log1p(eps * eps / n2)
        else:
            ld = torch.logsumexp(lw - 0.5 * ((eps - m) / sg) ** 2, 0) - half
        total = total + ld - lh
    return total, v, eps


def _value(model, theta, y, seg=100):
    """Log likelihood, and the factors and shock that open each segment."""
    v = torch.zeros((FAMILY[model][0], theta.shape[1]), dtype=torch.float64, device=theta.device)
    eps = torch.zeros_like(theta[0])
    total, opens = torch.zeros_like(theta[0]), []
    with torch.no_grad():
        for s0 in range(0, len(y), seg):
            opens.append((v, eps))
            ll, v, eps = _density(model, theta, y[s0:s0 + seg], v, eps, s0 == 0)
            total = total + ll
    return total, torch.cat([v, eps[None]]), opens


def _gradient(model, theta, y, weight, opens, seg=100):
    """Gradient of sum(weight * log likelihood), a segment at a time."""
    grad = torch.zeros_like(theta)
    vb, eb = None, None
    for j in reversed(range(len(opens))):
        th = theta.detach().requires_grad_(True)
        v, eps = (x.detach().requires_grad_(True) for x in opens[j])
        ll, v1, e1 = _density(model, th, y[j * seg:(j + 1) * seg], v, eps, j == 0)
        loss = (weight * ll).sum()
        if vb is not None:
            loss = loss + (vb * v1).sum() + (eb * e1).sum()
        gt, vb, eb = torch.autograd.grad(loss, (th, v, eps), allow_unused=True)
        vb = torch.zeros_like(v) if vb is None else vb
        eb = torch.zeros_like(eps) if eb is None else eb
        grad += gt
    return grad


def _moments(g, J, N):
    """(mean, standard deviation, NSE, RNE) of each row of g [G, J N]."""
    x = g.reshape(-1, J, N)
    group = x.mean(2)
    mean = group.mean(1)
    between = ((group - mean[:, None]) ** 2).sum(1)
    var = ((x - mean[:, None, None]) ** 2).sum((1, 2)) / (J * N - 1)
    return torch.stack([mean, var.sqrt(), (between / (J * (J - 1))).sqrt(), var / (N * between / (J - 1))], 1)


def _functions(model, theta, state):
    """Section 5.2's functions of interest at the state's date: log volatility,
    the mixture's third moment, the probability of a 3% loss."""
    K, shock, I = FAMILY[model]
    v, e = state[:K], state[K]
    a, b, g = torch.tanh(theta[2:2 + K]), torch.exp(theta[2 + K:2 + 2 * K]), theta[2 + 2 * K:2 + 3 * K]
    nxt = (a * v + b * (torch.abs(e) - math.sqrt(2.0 / math.pi)) + g * e).sum(0)
    x = (-0.03 - theta[0] / 1000.0) * torch.exp(-theta[1] - 0.5 * nxt)
    rows = [theta[1] + 0.5 * v.sum(0)]
    if shock == GAUSS:
        return torch.stack(rows + [0.5 * torch.erfc(-x / math.sqrt(2.0))])
    q = 2 + 3 * K
    p = torch.tanh(theta[q:q + I]) + 1.0
    p = p / p.sum(0)
    m = theta[q + I:q + 2 * I] - (p * theta[q + I:q + 2 * I]).sum(0)
    sg = torch.exp(theta[q + 2 * I:q + 3 * I])
    c = 1.0 / torch.sqrt((p * (m * m + sg * sg)).sum(0))
    m, sg = c * m, c * sg
    rows.append((p * (m ** 3 + 3.0 * m * sg * sg)).sum(0))
    rows.append((p * 0.5 * torch.erfc(-(x - m) / (sg * math.sqrt(2.0)))).sum(0))
    return torch.stack(rows)


def exact(case, seed):
    do, model = case["do"], case["model"]
    if do not in ("loglik", "gradient", "report"):
        return None  # random draws of the library's own generator
    rng = np.random.default_rng(seed)
    y = [float(v) for v in _series(model, case["T"], rng)[0]]
    theta = _cloud(case, seed)
    total, state, opens = _value(model, theta, y)
    if do == "loglik":
        return dict(loglik=total, state=state)
    if do == "gradient":
        weight = torch.from_numpy(rng.uniform(0.5, 1.5, case["N"])).cuda()
        return dict(loglik=total, grad=_gradient(model, theta, y, weight, opens))
    J, N = case["J"], case["N"]
    lw = torch.from_numpy(rng.normal(-40.0, 0.3, (50, J))).cuda()
    params = _moments(theta, J, N)
    sums = lw.sum(0)
    r = torch.exp(sums - sums.max())
    rbar = r.mean()
    nse = (((r - rbar) ** 2).sum() / (J * (J - 1))).sqrt() / rbar
    log_ml = torch.stack([sums.max() + rbar.log(), nse, (torch.logsumexp(lw, 1) - math.log(J)).sum()])
    return dict(params=params, functions=_moments(_functions(model, theta, state), J, N),
                rne=params[:, 3].mean().reshape(1), log_ml=log_ml)
