"""The work a user of the library has it do, as measurable cases.

A program that maps a surface phase diagram has three parts, and every case is one
call sequence out of one of them:

  sampling    chunks of a run: drop the samples already harvested, advance all
              walkers, read the new samples and the walkers' state
              (FP64 and FP32 pair terms, one slab or an uneven batch, the paper's
              own step with Monte Carlo or MD, the learned insertion proposal,
              structural observables recorded with every sample)
  reweighting samples -> free energies -> averages on a target grid, with
              bootstrap errors, or with structural observables; batch means of a
              run's samples
  training    Adam steps of the proposal network on captured configurations

Sampling starts from walkers that have been run for `burn` sweeps, as a program has
them in hand.  The samples that are reweighted come from a closed form (below) whose
law on the (T, mu) grid is exact, so they are made quickly and from the seed alone.
"""
import math

import numpy as np
import torch

from paper_1908_11118_amd import regc
from paper_1908_11118_amd import workloads as W

SAMPLE, LEARNED, PAPER = "sample", "learned", "paper"
REWEIGHT, ERRORS, OBSERVABLES, BATCH_MEANS = "reweight", "errors", "observables", "batch means"
TRAIN = "train"
TOL = 1e-12          # of every solve: the averages and their errors to about nine digits


# ---- the cases -------------------------------------------------------------------
def _sample(name, cells, layers, height, n_t, n_mu, n_max, sweeps, every, burn, fp64, classes=1, obs=False, kind=SAMPLE):
    # cells: the slab's top layer has cells x cells atoms, 1.5 sigma apart (class k of a
    # batch: cells + 2 k); height: of the gas region; every: sweeps per sample
    return {"name": name, "kind": kind, "cells": cells, "layers": layers, "height": height, "n_t": n_t, "n_mu": n_mu,
            "n_max": n_max, "sweeps": sweeps, "every": every, "burn": burn, "fp64": fp64, "classes": classes, "obs": obs}


def _grid(name, kind, n_t, n_mu, n_max, records, **more):
    return dict({"name": name, "kind": kind, "n_t": n_t, "n_mu": n_mu, "n_max": n_max, "records": records}, **more)


def listed():
    return [
        # the smallest run: the 64-replica system in the parity precision, one exchange
        # interval per call with every sweep recorded (latency and launches count)
        _sample("sample 64 replicas f64", 4, 2, 8.0, 8, 8, 40, 10, 1, 100, True),
        # the headline system: 1024 replicas at a 192-atom slab, one recorded chunk
        _sample("sample 1024 replicas f32", 8, 3, 12.0, 32, 32, 200, 100, 100, 300, False),
        # the largest: 4096 replicas in four slab classes, one recorded chunk
        _sample("sample 4096 replicas uneven f32", 6, 3, 12.0, 32, 32, 500, 100, 100, 200, False, classes=4),
        # structure recorded with every sample: axial density and lateral pair counts
        _sample("sample with observables f32", 8, 3, 12.0, 32, 32, 200, 10, 1, 200, False, obs=True),
        # the 64-replica system with the learned insertion proposal
        _sample("sample learned proposal f32", 4, 2, 8.0, 8, 8, 40, 10, 10, 300, False, kind=LEARNED),
        # the paper's own step (x0 coin, ten Monte Carlo cycles) on the same system
        dict(_sample("paper step f64", 4, 2, 8.0, 8, 8, 40, 20, 10, 40, True, kind=PAPER), md_steps=0),
        # reweighting of a small run: 64 states, 1000 records, an 8 x 8 map
        _grid("reweight 64 states", REWEIGHT, 8, 8, 40, 1000, tgt_t=8, tgt_mu=8),
        # reweighting of the headline run: 1024 states, 1.02e6 samples, a 64 x 64 map
        _grid("reweight 1024 states", REWEIGHT, 32, 32, 200, 1000, tgt_t=64, tgt_mu=64),
        # estimates with their errors: 100 bootstrap replicates
        _grid("errors 1024 states", ERRORS, 32, 32, 200, 200, tgt_t=16, tgt_mu=16, boot=100),
        # structural observables reweighted onto 16 T x 64 mu
        _grid("observables 1024 states", OBSERVABLES, 32, 32, 200, 200, tgt_t=16, tgt_mu=64, n_obs=221),
        # batch means of a run's samples, as a run that watches its errors takes them
        _grid("batch means 1024 states", BATCH_MEANS, 32, 32, 200, 1000, batches=20),
        # training of the proposal network
        {"name": "train proposal network", "kind": TRAIN, "examples": 65536, "n_max": 40, "batch": 256, "steps": 20},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice([SAMPLE, SAMPLE, SAMPLE, LEARNED, PAPER, REWEIGHT, REWEIGHT, ERRORS, OBSERVABLES, BATCH_MEANS, TRAIN])
    if kind == TRAIN:
        c = {"kind": kind, "examples": _log_int(rng, 1000, 65536), "n_max": rng.randint(12, 200),
             "batch": 64 * rng.randint(1, 8), "steps": rng.randint(2, 20)}
    elif kind in (SAMPLE, LEARNED, PAPER):
        n_t, n_mu = _log_int(rng, 2, 32), _log_int(rng, 2, 32)
        c = _sample("", rng.randint(4, 12), rng.randint(1, 3), round(rng.uniform(4.0, 12.0), 2), n_t, n_mu,
                    _log_int(rng, 12, 500), rng.randint(1, 40), rng.choice([1, 2, 5, 10]), 100, rng.random() < 0.4,
                    kind=kind)
        del c["name"]
        if kind == SAMPLE:
            c["obs"] = rng.random() < 0.2
            if not c["obs"] and rng.random() < 0.3:
                c["classes"], c["cells"] = rng.randint(2, 4), rng.randint(4, 6)
        elif kind == LEARNED:
            c.update(cells=rng.randint(4, 6), n_t=_log_int(rng, 2, 8), n_mu=_log_int(rng, 2, 8),
                     n_max=_log_int(rng, 12, 80), sweeps=rng.randint(1, 10), fp64=False)
        else:
            c.update(n_t=_log_int(rng, 2, 16), n_mu=_log_int(rng, 2, 16), n_max=_log_int(rng, 12, 80),
                     md_steps=rng.choice([0, 10]))
    else:
        n_t, n_mu = rng.randint(2, 32), rng.randint(2, 32)
        # about as many samples as a run of that grid keeps
        recs = max(20, min(1000, _log_int(rng, 20000, 1000000) // (n_t * n_mu)))
        c = {"kind": kind, "n_t": n_t, "n_mu": n_mu, "n_max": _log_int(rng, 12, 200), "records": recs}
        if kind == BATCH_MEANS:
            c["batches"] = rng.randint(5, 40)
        else:
            c.update(tgt_t=rng.randint(2, 64), tgt_mu=rng.randint(2, 64))
        if kind == ERRORS:
            c.update(tgt_t=rng.randint(2, 16), tgt_mu=rng.randint(2, 16), boot=rng.randint(10, 60),
                     records=max(20, min(recs, 200)))
        if kind == OBSERVABLES:
            c.update(tgt_t=rng.randint(2, 16), n_obs=rng.randint(20, 240), records=max(20, min(recs, 200)))
    return c


# ---- inputs ----------------------------------------------------------------------
def _temperatures(c):
    return W.linear_grid(0.5, 2.0, c["n_t"]), W.linear_grid(-8.0, -2.0, c["n_mu"])


def _workloads(c, seed):
    out = []
    t, mu = _temperatures(c)
    for k in range(c["classes"]):
        n = c["cells"] + 2 * k
        box = 1.5 * n
        out.append(W.Workload(name="case", slab=W.fcc100_slab(n, c["layers"], box, rc=2.5), lx=box, ly=box, zlo=0.0,
                              zhi=c["height"], t=t, mu=mu, n_max=c["n_max"], sample_every=c["every"], seed=seed + 1))
    return out


def _law(c):
    """A fluid whose (E, N) law is known in closed form: hard cores of a close packing of
    1.5 n_max in the volume, pair attraction, and at each N a Gaussian density of energies.
    Returns the temperatures, mu, ln of the count of states and mean and variance of E at
    each N at infinite temperature."""
    t, mu = _temperatures(c)
    n = np.arange(c["n_max"] + 1, dtype=np.float64)
    volume = 8.0 * c["n_max"]
    ln_count = n * np.log(volume) + n * np.log1p(-n / (1.5 * c["n_max"])) - np.array([math.lgamma(x + 1.0) for x in n])
    return t, mu, ln_count, -1.0 * n - 1.2 * n * n / c["n_max"], 0.35 * n + 1e-3


def _samples(c, seed):
    """records x states samples of that law, each record one sample of every walker, the
    states permuted among the walkers as replica exchange leaves them."""
    rng = np.random.default_rng(seed)
    t, mu, ln_count, mean, var = _law(c)
    states, recs, n = len(t) * len(mu), c["records"], np.arange(c["n_max"] + 1)
    e_out, n_out = np.empty((states, recs)), np.empty((states, recs), np.int32)
    for s in range(states):
        beta = 1.0 / t[s // len(mu)]
        ln_z = beta * mu[s % len(mu)] + 1.5 * math.log(t[s // len(mu)])
        ln_p = n * ln_z + ln_count - beta * mean + 0.5 * beta * beta * var
        cdf = np.cumsum(np.exp(ln_p - ln_p.max()))
        k = np.searchsorted(cdf, rng.random(recs) * cdf[-1], side="right").clip(0, c["n_max"])
        n_out[s] = k
        e_out[s] = mean[k] - beta * var[k] + np.sqrt(var[k]) * rng.standard_normal(recs)
    state = np.argsort(rng.random((recs, states)), axis=1).astype(np.int32)
    rec = np.arange(recs)[:, None]
    return e_out[state, rec].ravel(), n_out[state, rec].ravel(), state.ravel()


def _targets(c):
    return W.linear_grid(0.55, 1.95, c["tgt_t"]), W.linear_grid(-7.5, -2.5, c["tgt_mu"])


def _counts(c, seed, n):
    """Observable records of samples holding n particles: counts that scale with n."""
    rng = np.random.default_rng(seed + 7)
    scale = np.outer(n.astype(np.float32), 0.1 * rng.random(c["n_obs"], dtype=np.float32))
    return (scale * (0.5 + rng.random(scale.shape, dtype=np.float32)) + rng.random(scale.shape, dtype=np.float32)).astype(np.uint32)


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind in (SAMPLE, LEARNED, PAPER):
        wl = _workloads(c, seed)
        if kind == PAPER:
            step = W.paper_schedule if not c["md_steps"] else W.paper_schedule_md
            wl = [step(w, sample_every=c["every"]) for w in wl]
        walkers = sum(w.n_states for w in wl)
        g = regc.Regc(wl if len(wl) > 1 else wl[0], precision=regc.FP64 if c["fp64"] else regc.FP32PAIR,
                      sample_capacity=walkers * (max(c["burn"], 2 * c["sweeps"]) // c["every"] + 4))
        g.run(c["burn"])
        if kind == LEARNED:
            net = regc.Mlp(W.mlp_pack(W.mlp_init(seed=seed)))
            g.set_proposal(net, 0.9)
            net.close()
        g.clear_samples()
        if c["obs"]:
            # axial density in 0.12-sigma bins, lateral pair counts of the first layer
            g.set_observables(0.12, (0.6, 1.6), 0.05, 120)
        g.sync()
        return {"case": c, "run": g}
    if kind == TRAIN:
        rng = np.random.default_rng(seed)
        n = rng.integers(0, c["n_max"] + 1, c["examples"]).astype(np.int32)
        # particles sit low in the gas region, as adsorbed ones do
        iz = np.minimum(rng.geometric(0.35, (c["examples"], c["n_max"])) - 1, 15)
        vox = (iz * 256 + rng.integers(0, 256, iz.shape)).astype(np.uint16)
        net = regc.Mlp(W.mlp_pack(W.mlp_init(seed=seed)))
        return {"case": c, "seed": seed, "net": net, "vox": torch.from_numpy(vox.view(np.int16)).cuda(),
                "n": torch.from_numpy(n).cuda()}
    e, n, s = _samples(c, seed)
    st = {"case": c, "e": torch.from_numpy(e).cuda(), "n": torch.from_numpy(n).cuda(), "s": torch.from_numpy(s).cuda()}
    if kind != BATCH_MEANS:
        t, mu = _temperatures(c)
        st["mbar"] = regc.Mbar(t, mu, c["n_max"])
    if kind == OBSERVABLES:
        st["mbar"].set_samples_device(len(e), st["e"].data_ptr(), st["n"].data_ptr(), st["s"].data_ptr())
        st["mbar"].set_observables(_counts(c, seed, n))
        st["mbar"].solve(tol=TOL)
    return st


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind in (SAMPLE, LEARNED, PAPER):
        g = state["run"]
        g.clear_samples()
        g.run(c["sweeps"])
        # (a long run keeps its coordinates on the GPU; a small one is looked at whole)
        out = {"samples": g.samples(), "walkers": g.walkers(xyz=c["n_t"] * c["n_mu"] <= 64), "counts": g.stats()}
        if c["obs"]:
            out["observables"] = g.observables()
        return out
    if kind == TRAIN:
        net = state["net"]
        loss = net.train(c["examples"], c["n_max"], state["vox"].data_ptr(), state["n"].data_ptr(), c["steps"],
                         batch=c["batch"], seed=state["seed"])
        return {"loss": loss, "params": net.params()}
    if kind == BATCH_MEANS:
        mean, se = regc.batch_means(state["s"], state["n"], c["n_t"] * c["n_mu"], c["batches"])
        return {"mean": mean, "se": se}
    mb = state["mbar"]
    t, mu = _targets(c)
    if kind == OBSERVABLES:
        mean, cond = mb.observables(t, mu, c["n_obs"])
        return {"mean": mean, "cond": cond}
    mb.set_samples_device(c["records"] * c["n_t"] * c["n_mu"], state["e"].data_ptr(), state["n"].data_ptr(),
                          state["s"].data_ptr())
    if kind == ERRORS:
        out = mb.reweight(t, mu, tol=TOL, n_boot=c["boot"], n_sites=64.0)
        del out["converged"]
        return out
    f, _, _, _ = mb.solve(tol=TOL)
    out = mb.targets(t, mu)
    out["f_states"] = f
    return out


# ---- work and exact values ---------------------------------------------------------
FLOPS_PER_PAIR = 25


def work(case):
    """Sampling: 25 operations per pair term inside the cutoff (about ten per trial, the
    volume of the cutoff sphere at a liquid's density shared by gas and slab), the walkers'
    coordinates once in and out.  Reweighting: the samples once, and per iteration one
    exponential (about 20 operations) per sample and temperature.  Training: the dense
    layers forward and backward, the parameters and their Adam state once per step."""
    c, kind = case, case["kind"]
    if kind in (SAMPLE, LEARNED, PAPER):
        walkers = c["classes"] * c["n_t"] * c["n_mu"]
        if kind == PAPER:
            trials = c["sweeps"] * 10 * c["n_max"] // 2
        else:
            trials = c["sweeps"] * (c["n_max"] + 1)
        flops = walkers * trials * 10.0 * FLOPS_PER_PAIR
        if kind == LEARNED:
            flops += walkers * trials * 0.25 * 2.0 * (128 * 4096 + 2 * 128 * 128)
        return {"bytes": walkers * (c["n_max"] * 24.0 + 16.0 * c["sweeps"] / c["every"]), "flops": flops}
    if kind == TRAIN:
        params = 2 * 4096 * 128 + 2 * 128 * 128 + 4096 + 3 * 128
        dense = 128 * 4096 + 2 * 128 * 128
        return {"bytes": c["steps"] * params * 24.0, "flops": c["steps"] * c["batch"] * 6.0 * dense}
    samples = c["records"] * c["n_t"] * c["n_mu"]
    if kind == BATCH_MEANS:
        return {"bytes": samples * 8.0, "flops": 2.0 * samples}
    if kind == OBSERVABLES:
        return {"bytes": samples * (16.0 + 4.0 * c["n_obs"]), "flops": samples * c["tgt_t"] * (20.0 + 2.0 * c["n_obs"])}
    sweeps = 20.0 * (1 + c.get("boot", 0))
    return {"bytes": samples * 16.0, "flops": 24.0 * samples * (sweeps * c["n_t"] + c["tgt_t"])}


def _free_energies(c, e, n, state):
    """The reweighting equations solved by Newton's method in 64 bits: (f of the states,
    ln D of every sample), f = 0 at the first sampled state."""
    t, mu, ln_count, mean, var = _law(c)
    beta, cap = 1.0 / t, c["n_max"] + 1
    lnz = beta[:, None] * mu[None, :] + 1.5 * np.log(t)[:, None]
    ln_om = np.log(np.maximum(np.bincount(state, minlength=lnz.size), 1e-300)).reshape(lnz.shape)
    k = np.arange(cap, dtype=np.float64)
    # the law's own free energies are within the sampling error of the solution
    a = k * lnz[:, :, None] + (ln_count - beta[:, None] * mean + 0.5 * beta[:, None] ** 2 * var)[:, None, :]
    f = -np.logaddexp.reduce(a, axis=2)
    order = np.argsort(n, kind="stable")
    es, edges = e[order], np.searchsorted(n[order], np.arange(cap + 1))
    held = [q for q in range(cap) if edges[q + 1] > edges[q]]
    ln_d = np.empty(len(e))
    for _ in range(30):
        w = ln_om[:, :, None] + f[:, :, None] + k * lnz[:, :, None]           # [L, M, N]
        ln_a = np.logaddexp.reduce(w, axis=1)                                 # [L, N]
        share = np.exp(w - ln_a[:, None, :])
        p1, p2 = np.zeros((len(t), cap)), np.zeros((len(t), len(t), cap))
        for q in held:
            x = -beta[:, None] * es[None, edges[q]:edges[q + 1]] + ln_a[:, q, None]
            top = x.max(axis=0)
            p = np.exp(x - top)
            tot = p.sum(axis=0)
            ln_d[edges[q]:edges[q + 1]] = top + np.log(tot)
            p /= tot
            p1[:, q], p2[:, :, q] = p.sum(axis=1), p @ p.T
        weight = share * p1[:, None, :]
        got = weight.sum(axis=2).ravel()                                       # sum of each state's weights
        hess = np.einsum("lmn,lkn,kjn->lmkj", share, p2, share, optimize=True).reshape(got.size, got.size)
        hess = np.diag(got) - hess
        grad = np.exp(ln_om.ravel()) * (np.exp(ln_om.ravel()) > 0.5) - got
        live = np.flatnonzero(np.exp(ln_om.ravel()) > 0.5)
        free = live[1:]
        step = np.zeros(got.size)
        step[free] = np.linalg.solve(hess[np.ix_(free, free)], grad[free])
        f = f + step.reshape(f.shape)
        f = f - f.ravel()[live[0]]
        if np.abs(step).max() < 1e-13 * max(1.0, np.abs(f).max()):
            break
    out = np.empty(len(e))
    out[order] = ln_d
    return f, out


def _averages(c, e, n, ln_d, obs=None):
    tt, tm = _targets(c)
    cap = c["n_max"] + 1
    k = np.arange(cap, dtype=np.float64)
    size = len(tt) * len(tm)
    out = {q: np.zeros(size) for q in ("f", "mean_n", "mean_e", "mean_e2")}
    out["p_n"], out["phase"] = np.zeros((size, cap)), np.zeros(size, np.int32)
    cond = np.zeros((len(tt), cap, 0 if obs is None else obs.shape[1]))
    order = np.argsort(n, kind="stable")
    es, ds, edges = e[order], ln_d[order], np.searchsorted(n[order], np.arange(cap + 1))
    for i, temp in enumerate(tt):
        g, e1, e2 = np.full(cap, -np.inf), np.zeros(cap), np.zeros(cap)
        for q in range(cap):
            part = slice(edges[q], edges[q + 1])
            if edges[q + 1] == edges[q]:
                continue
            y = -es[part] / temp - ds[part]
            w = np.exp(y - y.max())
            g[q], e1[q], e2[q] = y.max() + np.log(w.sum()), w @ es[part] / w.sum(), w @ es[part] ** 2 / w.sum()
            if obs is not None:
                cond[i, q] = w @ obs[order[part]] / w.sum()
        for j, m in enumerate(tm):
            a = k * (m / temp + 1.5 * math.log(temp)) + g
            lse = np.logaddexp.reduce(a)
            p, at = np.exp(a - lse), i * len(tm) + j
            out["f"][at], out["p_n"][at], out["phase"][at] = -lse, p, int(np.argmax(a))
            out["mean_n"][at], out["mean_e"][at], out["mean_e2"][at] = p @ k, p @ e1, p @ e2
    return out, cond


def _batch_means(state, n, states, batches):
    mean, se = np.full(states, np.nan), np.full(states, np.nan)
    order = np.argsort(state, kind="stable")
    edges = np.searchsorted(state[order], np.arange(states + 1))
    for s in range(states):
        x = n[order[edges[s]:edges[s + 1]]].astype(np.float64)
        if len(x) < batches:
            continue
        cut = (np.arange(batches + 1) * len(x)) // batches
        means = np.array([x[cut[b]:cut[b + 1]].mean() for b in range(batches)])
        mean[s], se[s] = x.mean(), math.sqrt(means.var(ddof=1) / batches)
    return mean, se


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind not in (REWEIGHT, ERRORS, OBSERVABLES, BATCH_MEANS):
        return None                      # a Markov chain, or training steps: no value apart from its own rounding
    e, n, s = _samples(c, seed)
    states = c["n_t"] * c["n_mu"]
    if kind == BATCH_MEANS:
        mean, se = _batch_means(s, n, states, c["batches"])
        return {"mean": mean, "se": se}
    f, ln_d = _free_energies(c, e, n, s)
    if kind == OBSERVABLES:
        obs = _counts(c, seed, n).astype(np.float64)
        av, cond = _averages(c, e, n, ln_d, obs)
        tt, tm = _targets(c)
        p = av["p_n"].reshape(len(tt), len(tm), -1)
        return {"mean": np.einsum("ijq,iqk->ijk", p, cond, optimize=True), "cond": cond}
    av, _ = _averages(c, e, n, ln_d)
    if kind == REWEIGHT:
        av["f_states"] = f.ravel()
        return av
    beta = np.repeat(1.0 / _targets(c)[0], c["tgt_mu"])
    mean, se = _batch_means(s, n, states, 20)
    return {"f_states": f.ravel(), "mean_state_n": mean, "se_state_n": se, "mean_n": av["mean_n"], "se_n": None,
            "coverage": av["mean_n"] / 64.0, "se_coverage": None, "se_heat_cap": None,
            "heat_cap": beta ** 2 * (av["mean_e2"] - av["mean_e"] ** 2), "phase": av["phase"], "p_n": av["p_n"]}
