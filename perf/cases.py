"""What a program using this library has it do, as cases that can be timed and
compared: one pass of each goes through the public entry points
(paper_2407_00051_amd.Context and gan.GanLoop) on inputs made from a seed.

  listed()   the twelve cases: the discriminator step at its smallest, its
             headline and its largest sizes in fp32 and bf16, the GAN training
             step, the three-call form of the step on event buffers, the sampler
             and the per-parameter reduction on their own, the two bootstrap
             draws and the ensemble response
  draw(rng)  one more case of the same kinds and ranges
  prepare, run, work, tolerance, exact: see each function

exact() states every result in float64 with plain torch, without the library.
"""
import math

import torch

import paper_2407_00051_amd as sg
from paper_2407_00051_amd.gan import GanLoop

SLOPE = 0.2
THETA_STAR = {2: (2.0, 5.0, 1.5, 3.0), 3: (2.0, 5.0, 1.5, 3.0, 3.0, 2.0)}
FEATURES = {"identity": sg.FEAT_IDENTITY, "hd8": sg.FEAT_HD8, "proxy2": sg.FEAT_PROXY2}
GEN_WIDTHS = (6, 128, 128, 128, 128, 6)      # the paper's 51,206-parameter generator
DISC_WIDTHS = (2, 128, 128, 128, 128, 1)     # the paper's 50,049-parameter discriminator
NOISE_BATCHES = 8                            # noise batches a training program has drawn ahead


# ---------------------------------------------------------------------------
# The cases

def listed():
    return [
        # fp32 steps with the events sampled inside the call: one parameter row (a user's first
        # call, a step of a small study: latency and launches), and the batch of 32 rows that
        # the benchmark quotes
        dict(name="f32_one_row", kind="step", precision="f32", features="identity", n_theta=1, E=16384, d=2, H=64, NH=1,
             n_real=16384),
        dict(name="f32_small_batch", kind="step", precision="f32", features="identity", n_theta=32, E=8192, d=2, H=128,
             NH=2, n_real=262144),
        # the same step in its three-call form, for a program that keeps the events (its own
        # pipeline after the sampler): sample, discriminate a buffer of odd size, reduce
        dict(name="f32_three_call", kind="three_call", n_theta=37, E=1999, d=3, H=128, NH=2, n_real=70001),
        # one GAN training step at the paper's shape: generator forward and backward, bootstrap,
        # fp32 discriminator on the two observables, Adam on both networks
        dict(name="train_paper", kind="train", k=1024, E=100),
        # bf16 steps: a short ragged batch (validation, the tests' sizes), and the two wide
        # networks at full size
        dict(name="bf16_ragged", kind="step", precision="bf16", features="identity", n_theta=3, E=1000, d=2, H=256, NH=3,
             n_real=2999),
        dict(name="bf16_medium", kind="step", precision="bf16", features="identity", n_theta=256, E=16384, d=2, H=256,
             NH=3, n_real=4194304),
        dict(name="bf16_higher_dim", kind="step", precision="bf16", features="hd8", n_theta=1024, E=16384, d=3, H=512,
             NH=3, n_real=16777216),
        # the sampler and the pathwise reduction alone, at the stress size
        dict(name="param_grad_stress", kind="param_grad", n_theta=64, E=4194304, d=2),
        dict(name="sample_stress", kind="sample", n_theta=64, E=4194304, d=2),
        # one step's bootstrapped reference batch, half the size of its pool: in draw order for the
        # three-observable step, and in row order for the two-observable one
        dict(name="bootstrap_d3", kind="bootstrap", n_data=33554432, n_out=16777216, d=3, row_order=False),
        dict(name="bootstrap_rows", kind="bootstrap", n_data=8388608, n_out=4194304, d=2, row_order=True),
        # the response of an ensemble of 100 trained generators on a batch of noise
        dict(name="ensemble_100", kind="ensemble", M=100, k=1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["f32", "f32", "three_call", "train", "bf16", "bf16", "param_grad", "sample", "bootstrap",
                       "bootstrap", "ensemble"])
    if kind == "f32":
        d, H, NH = rng.choice([(2, 64, 1), (2, 64, 2), (2, 64, 3), (2, 128, 1), (2, 128, 2), (3, 64, 1), (3, 64, 2),
                               (3, 128, 2)])
        n_theta = _log_int(rng, 1, 64)
        E = _log_int(rng, 40, max(41, min(16384, 262144 // n_theta)))
        return dict(kind="step", precision="f32", features="identity", n_theta=n_theta, E=E, d=d, H=H, NH=NH,
                    n_real=_log_int(rng, max(64, n_theta * E // 2), n_theta * E + 64))
    if kind == "three_call":
        d, H, NH = rng.choice([(2, 64, 2), (2, 128, 1), (2, 128, 2), (3, 64, 2), (3, 128, 2)])
        n_theta = _log_int(rng, 4, 128)
        E = _log_int(rng, 100, 4000)
        return dict(kind="three_call", n_theta=n_theta, E=E, d=d, H=H, NH=NH, n_real=_log_int(rng, 500, 200000))
    if kind == "train":
        return dict(kind="train", k=_log_int(rng, 64, 1024), E=_log_int(rng, 50, 200))
    if kind == "bf16":
        features, d = rng.choice([("identity", 2), ("identity", 3), ("hd8", 3)])
        H = rng.choice([256, 512])
        n_theta = _log_int(rng, 1, 256)
        E = _log_int(rng, 500, max(501, min(16384, 2097152 // n_theta)))
        return dict(kind="step", precision="bf16", features=features, n_theta=n_theta, E=E, d=d, H=H,
                    NH=rng.choice([2, 3, 3]), n_real=_log_int(rng, max(500, n_theta * E // 2), n_theta * E + 500))
    if kind in ("param_grad", "sample"):
        n_theta = _log_int(rng, 1, 256)
        return dict(kind=kind, n_theta=n_theta, E=_log_int(rng, 4096, 100000000 // n_theta), d=rng.choice([2, 3]))
    if kind == "bootstrap":
        n_out = _log_int(rng, 100000, 16777216)
        return dict(kind="bootstrap", n_data=min(33554432, int(n_out * rng.uniform(1.0, 3.0))), n_out=n_out,
                    d=rng.choice([2, 3]), row_order=rng.choice([False, True]))
    return dict(kind="ensemble", M=_log_int(rng, 2, 100), k=_log_int(rng, 100, 2048))


# ---------------------------------------------------------------------------
# Inputs

def _dev():
    return torch.device("cuda:0")


def _rng(seed, salt):
    return torch.Generator(device=_dev()).manual_seed(int(seed) * 1000003 + salt)


def _theta(n, d, g):
    return 1.0 + 5.0 * torch.rand((n, 2 * d), generator=g, device=_dev())


def _kumaraswamy_events(n, d, g):
    """Reference events at theta*, [n][d] fp32."""
    ts = THETA_STAR[d]
    u = torch.rand((n, d), generator=g, device=_dev(), dtype=torch.float64).clamp_(1e-9, 1.0 - 1e-9)
    cols = [(1.0 - (1.0 - u[:, j]) ** (1.0 / ts[2 * j + 1])) ** (1.0 / ts[2 * j]) for j in range(d)]
    return torch.stack(cols, 1).float().clamp_(1e-7, 1.0 - 6e-8)


def _xavier(widths, g):
    """Discriminator weights in torch.nn.Linear layout: Xavier-uniform, biases U(+-1/sqrt(fan_in))."""
    Ws, bs = [], []
    for fi, fo in zip(widths[:-1], widths[1:]):
        Ws.append((2.0 * torch.rand((fo, fi), generator=g, device=_dev()) - 1.0) * math.sqrt(6.0 / (fi + fo)))
        bs.append((2.0 * torch.rand((fo,), generator=g, device=_dev()) - 1.0) / math.sqrt(fi))
    return Ws, bs


def _kaiming(widths, M, g):
    """M generators stacked in front: Kaiming-normal for LeakyReLU(0.2), biases U(+-1/sqrt(fan_in))."""
    Ws, bs = [], []
    for fi, fo in zip(widths[:-1], widths[1:]):
        Ws.append(torch.randn((M, fo, fi), generator=g, device=_dev()) * (math.sqrt(2.0 / (1.0 + SLOPE ** 2)) / math.sqrt(fi)))
        bs.append((2.0 * torch.rand((M, fo), generator=g, device=_dev()) - 1.0) / math.sqrt(fi))
    return Ws, bs


def _widths(case):
    f = {"identity": case["d"], "hd8": 8, "proxy2": 2}[case.get("features", "identity")]
    return (f,) + (case["H"],) * (case["NH"] + 1) + (1,)


def _inputs(case, seed):
    """The tensors of a case, from the seed alone (no library call)."""
    kind = case["kind"]
    g = _rng(seed, 7)
    t = {"seed": int(seed) * 2654435761 % (1 << 61)}
    if kind in ("step", "three_call"):
        t["theta"] = _theta(case["n_theta"], case["d"], g)
        t["W"], t["b"] = _xavier(_widths(case), g)
        t["real"] = _kumaraswamy_events(case["n_real"], case["d"], g)
    elif kind == "train":
        t["GW"], t["Gb"] = _kaiming(GEN_WIDTHS, 1, g)
        t["GW"], t["Gb"] = [w[0].contiguous() for w in t["GW"]], [v[0].contiguous() for v in t["Gb"]]
        t["DW"], t["Db"] = _xavier(DISC_WIDTHS, g)
        t["pool"] = _kumaraswamy_events(2 * case["k"] * case["E"], 3, g)
        t["noise"] = torch.randn((NOISE_BATCHES, case["k"], GEN_WIDTHS[0]), generator=g, device=_dev())
    elif kind in ("param_grad", "sample"):
        t["theta"] = _theta(case["n_theta"], case["d"], g)
    elif kind == "bootstrap":
        t["data"] = _kumaraswamy_events(case["n_data"], case["d"], g)
        t["step"] = int(seed) % 100000 + 1
    elif kind == "ensemble":
        t["W"], t["b"] = _kaiming(GEN_WIDTHS, case["M"], g)
        t["noise"] = torch.randn((case["k"], GEN_WIDTHS[0]), generator=g, device=_dev())
        t["p_true"] = torch.tensor(THETA_STAR[3], device=_dev())
    else:
        raise ValueError(kind)
    return t


def prepare(case, seed):
    """Inputs, and the buffers that such a program keeps from step to step."""
    s = dict(_inputs(case, seed), case=case, ctx=sg.default_context(0))
    kind, f32 = case["kind"], dict(dtype=torch.float32, device=_dev())
    if kind in ("step", "three_call"):
        N, d = case["n_theta"] * case["E"], case["d"]
        o = {"logits_fake": torch.empty(N, **f32), "logits_real": torch.empty(case["n_real"], **f32),
             "loss_d": torch.empty(1, **f32), "loss_g": torch.empty(1, **f32),
             "dW": [torch.empty_like(w) for w in s["W"]], "db": [torch.empty_like(v) for v in s["b"]]}
        if kind == "step":
            o["dLg_dtheta"] = torch.empty((case["n_theta"], 2 * d), **f32)
            if case["precision"] == "bf16":
                o["dLg_dx"] = torch.empty((N, d), **f32)
        else:
            o["dLg_dx"] = torch.empty((N, d), **f32)
            s["x"] = torch.empty((N, d), **f32)
            s["dtheta"] = torch.empty((case["n_theta"], 2 * d), **f32)
        s["outs"] = o
    elif kind == "train":
        s["loop"] = GanLoop(s["ctx"], s["GW"], s["Gb"], s["DW"], s["Db"], s["pool"], case["k"], case["E"],
                            fake_seed=s["seed"], boot_seed=s["seed"] + 5)
    elif kind == "param_grad":
        s["out"] = torch.empty((case["n_theta"], 2 * case["d"]), **f32)
        s["loss"] = torch.empty(1, **f32)
    elif kind == "sample":
        s["out"] = torch.empty((case["n_theta"] * case["E"], case["d"]), **f32)
    elif kind == "bootstrap":
        s["out"] = torch.empty((case["n_out"], case["d"]), **f32)
    return s


# ---------------------------------------------------------------------------
# One pass

def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "step":
        return ctx.disc_fwd_bwd(s["W"], s["b"], s["real"],
                                fake_source=dict(theta=s["theta"], events_per_theta=case["E"], seed=s["seed"]),
                                precision=sg.F32 if case["precision"] == "f32" else sg.BF16,
                                features=FEATURES[case["features"]], slope=SLOPE, outputs=s["outs"],
                                want_dx="dLg_dx" in s["outs"])
    if kind == "three_call":
        ctx.sample_events(s["theta"], case["E"], s["seed"], out=s["x"])
        o = dict(ctx.disc_fwd_bwd(s["W"], s["b"], s["real"], fake_x=s["x"], slope=SLOPE, outputs=s["outs"]))
        o["x"] = s["x"]
        o["dLg_dtheta"] = ctx.param_grad(s["theta"], case["E"], s["seed"], dL_dx=o["dLg_dx"], out=s["dtheta"])
        return o
    if kind == "train":
        loop = s["loop"]
        loop.step(s["noise"][loop.t % NOISE_BATCHES])
        return {"theta": loop.theta, "loss_d": loop.outs["loss_d"], "loss_g": loop.outs["loss_g"],
                "dW": loop.outs["dW"], "db": loop.outs["db"], "dLg_dtheta": loop.outs["dLg_dtheta"],
                "gW": loop.gW, "gb": loop.gb, "G_W": loop.G_W, "G_b": loop.G_b, "D_W": loop.D_W, "D_b": loop.D_b}
    if kind == "param_grad":
        g, loss = ctx.param_grad(s["theta"], case["E"], s["seed"], out=s["out"], loss_out=s["loss"])
        return {"dL_dtheta": g, "loss": loss}
    if kind == "sample":
        return ctx.sample_events(s["theta"], case["E"], s["seed"], out=s["out"])
    if kind == "bootstrap":
        return ctx.bootstrap(s["data"], case["n_out"], s["seed"], s["step"], out=s["out"], row_order=case["row_order"])
    r = ctx.ensemble_response(s["W"], s["b"], s["noise"], p_true=s["p_true"], slope=SLOPE)
    return {"p_hat": r["p_hat"], "sigma": r["sigma"], "r_hat": r["r_hat"]}


# ---------------------------------------------------------------------------
# What one pass cannot do without

def _macs(widths):
    return sum(a * b for a, b in zip(widths[:-1], widths[1:]))


def _params(widths):
    return sum(a * b + b for a, b in zip(widths[:-1], widths[1:]))


def _disc_flops(widths, n_fake, n_real):
    """Forward and weight gradients on every event; the backward signal down to the input on
    the fake ones and down to the first hidden layer on the real ones."""
    S = _macs(widths)
    return 6.0 * S * n_fake + (6.0 * S - 2.0 * widths[0] * widths[1]) * n_real


# A sampled event: ten Philox rounds of two 32x32->64 products and two three-way xors (8
# operations a round), and per coordinate about 25 fp32 operations of the quantile.
def _sample_ops(n, d):
    return n * (80.0 + 25.0 * d)


def work(case):
    kind = case["kind"]
    if kind in ("step", "three_call"):
        w, d = _widths(case), case["d"]
        nf, nr = case["n_theta"] * case["E"], case["n_real"]
        by = 4.0 * (2 * _params(w) + nf + nr + nr * d + 4 * case["n_theta"] * d)   # weights and dW, logits, real, theta
        if case.get("precision") == "bf16":
            by += 4.0 * nf * d                                                      # dL_G/dx
        if kind == "three_call":
            by += 4.0 * nf * d * 4                                                  # x and dL_G/dx out and in
        return {"bytes": by, "flops": _disc_flops(w, nf, nr) + _sample_ops(nf, d)}
    if kind == "train":
        k, N = case["k"], case["k"] * case["E"]
        S = _macs(GEN_WIDTHS)
        flops = _disc_flops(DISC_WIDTHS, N, N) + k * (2.0 * S + 6.0 * S - 2.0 * GEN_WIDTHS[0] * GEN_WIDTHS[1])
        by = 4.0 * (3 * N * 2 + 8 * (_params(DISC_WIDTHS) + _params(GEN_WIDTHS)) + k * 24)
        return {"bytes": by, "flops": flops + _sample_ops(N, 3)}
    if kind == "param_grad":
        n = case["n_theta"] * case["E"]
        return {"bytes": 16.0 * case["n_theta"] * case["d"] + 4, "flops": _sample_ops(n, case["d"]) + 14.0 * n * case["d"]}
    if kind == "sample":
        n = case["n_theta"] * case["E"]
        return {"bytes": 4.0 * n * case["d"], "flops": _sample_ops(n, case["d"])}
    if kind == "bootstrap":
        return {"bytes": 8.0 * case["n_out"] * case["d"], "flops": 80.0 * case["n_out"]}
    S = _macs(GEN_WIDTHS)
    return {"bytes": 4.0 * (case["M"] * _params(GEN_WIDTHS) + case["k"] * 6 + 24), "flops": 2.0 * S * case["M"] * case["k"]}


def tolerance(case):
    kind = case["kind"]
    if kind == "bootstrap":
        return "exact"                       # copies of rows, chosen by whole numbers
    if kind == "sample":
        return {"rel": 2e-6, "max": 2e-5}    # hardware exp2 / log2 within an ulp, a few of them in a row
    if kind == "param_grad":
        return {"rel": 2e-5}                 # 32-bit sums of up to 2^22 terms of both signs
    if kind == "ensemble":
        return {"rel": 1e-5}
    if case.get("precision") == "bf16":
        # an activation that rounds the other way moves the layers that follow; per event dL_G/dx
        # changes where a hidden unit crosses the LeakyReLU kink
        return {"rel": 2e-2, "max": 0.99}
    # fp32: an event with a hidden unit within rounding of the LeakyReLU kink takes either slope; the
    # per-event dL_G/dx of that event, and the parameter row it falls in, move by that unit's share
    return {"rel": 3e-3, "max": 0.9}


# ---------------------------------------------------------------------------
# The results in float64

_M32 = 0xFFFFFFFF


def _mul32(a, m):
    """(high, low) 32-bit words of a * m for int64 tensors a < 2^32 and m < 2^32 (the int64
    product wraps, its bit pattern is the 64-bit product)."""
    p = a * m
    return (p >> 32) & _M32, p & _M32


def _philox(ids, c2, c3, seed):
    """Philox4x32-10 words of counters (id lo, id hi, c2, c3) under key = seed."""
    c0, c1 = ids & _M32, (ids >> 32) & _M32
    c2, c3 = torch.full_like(ids, c2), torch.full_like(ids, c3)
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    m0, m1 = 0xD2511F53, 0xCD9E8D57
    for _ in range(10):
        h0, l0 = _mul32(c0, m0)
        h1, l1 = _mul32(c2, m1)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c0, c1, c2, c3


def _events64(theta, E, i0, i1, seed, base=0):
    """x, dx/da, dx/db of events [i0, i1), each [n][d] float64, theta [rows][2d] float64."""
    ids = torch.arange(i0, i1, device=theta.device, dtype=torch.int64)
    row = torch.div(ids, E, rounding_mode="floor")
    words = _philox(ids + base, 0, 0, seed)
    xs, das, dbs = [], [], []
    for j in range(theta.shape[1] // 2):
        a, b = theta[row, 2 * j], theta[row, 2 * j + 1]
        l = torch.log1p(-((words[j] >> 9).double() + 0.5) * 2.0 ** -23)
        s = torch.exp(l / b)
        g = -torch.expm1(l / b)
        x = g ** (1.0 / a)
        xs.append(x)
        das.append(-x * torch.log(g) / (a * a))
        dbs.append(x * s * l / (a * b * b * g))
    return torch.stack(xs, 1), torch.stack(das, 1), torch.stack(dbs, 1)


def _features64(x, features):
    if features == "identity":
        return x
    x1, x2, x3 = x[:, 0], x[:, 1], x[:, 2]
    if features == "proxy2":
        return torch.stack([x1 + x3, x2 + x3], 1)
    return torch.stack([x1, x2, x3, x1 * x2, x2 * x3, x1 * x3, torch.log(x1), torch.log1p(-x3)], 1)


def _features_back64(gf, x, features):
    if features == "identity":
        return gf
    x1, x2, x3 = x[:, 0], x[:, 1], x[:, 2]
    if features == "proxy2":
        return torch.stack([gf[:, 0], gf[:, 1], gf[:, 0] + gf[:, 1]], 1)
    return torch.stack([gf[:, 0] + gf[:, 3] * x2 + gf[:, 5] * x3 + gf[:, 6] / x1,
                        gf[:, 1] + gf[:, 3] * x1 + gf[:, 4] * x3,
                        gf[:, 2] + gf[:, 4] * x2 + gf[:, 5] * x1 - gf[:, 7] / (1.0 - x3)], 1)


def _softplus64(t):
    return torch.clamp(t, min=0.0) + torch.log1p(torch.exp(-t.abs()))


def _disc64(W, b, n_fake, fake_chunk, real, features, fake_done=None, chunk=1 << 18):
    """The discriminator step.  fake_chunk(i0, i1) gives the raw fake events of a range (float64)
    and anything fake_done(i0, i1, that, dL_G/dx) wants with them."""
    W, b = [w.double() for w in W], [v.double() for v in b]
    n, n_real, dev = len(W), real.shape[0], real.device
    f64 = dict(dtype=torch.float64, device=dev)
    o = {"logits_fake": torch.empty(n_fake, **f64), "logits_real": torch.empty(n_real, **f64),
         "dW": [torch.zeros_like(w) for w in W], "db": [torch.zeros_like(v) for v in b]}
    for fake, N in ((True, n_fake), (False, n_real)):
        for i0 in range(0, N, chunk):
            i1 = min(N, i0 + chunk)
            got = fake_chunk(i0, i1) if fake else (real[i0:i1].double(),)
            hs = [_features64(got[0], features)]
            for l in range(n - 1):
                p = torch.addmm(b[l], hs[-1], W[l].T)
                hs.append(torch.where(p > 0, p, SLOPE * p))
            z = hs[-1] @ W[-1][0] + b[-1]
            sig = torch.sigmoid(z)
            e = sig / n_fake if fake else (sig - 1.0) / n_real
            o["logits_fake" if fake else "logits_real"][i0:i1] = z
            o["dW"][-1] += (e @ hs[-1])[None, :]
            o["db"][-1] += e.sum()
            d = W[-1] * torch.where(hs[-1] > 0, 1.0, SLOPE)
            for l in range(n - 2, -1, -1):
                ed = e[:, None] * d
                o["dW"][l] += ed.T @ hs[l]
                o["db"][l] += ed.sum(0)
                if l > 0 or fake:
                    d = d @ W[l]
                if l > 0:
                    d = d * torch.where(hs[l] > 0, 1.0, SLOPE)
            if fake and fake_done is not None:
                gx = _features_back64(d * ((sig - 1.0) / n_fake)[:, None], got[0], features)
                fake_done(i0, i1, got, gx)
    zf, zr = o["logits_fake"], o["logits_real"]
    o["loss_d"] = (_softplus64(-zr).mean() + _softplus64(zf).mean()).reshape(1)
    o["loss_g"] = _softplus64(-zf).mean().reshape(1)
    return o


def _sampled_disc64(W, b, theta, E, seed, real, features, want_dx):
    theta = theta.double()
    N, d = theta.shape[0] * E, theta.shape[1] // 2
    dtheta = torch.zeros_like(theta)
    dx = torch.empty((N, d), dtype=torch.float64, device=theta.device) if want_dx else None

    def done(i0, i1, got, gx):
        row = torch.div(torch.arange(i0, i1, device=gx.device), E, rounding_mode="floor")
        terms = torch.stack([gx * got[1], gx * got[2]], 2).reshape(i1 - i0, 2 * d)
        dtheta.index_add_(0, row, terms)
        if dx is not None:
            dx[i0:i1] = gx

    o = _disc64(W, b, N, lambda i0, i1: _events64(theta, E, i0, i1, seed), real, features, done)
    o["dLg_dtheta"] = dtheta
    if dx is not None:
        o["dLg_dx"] = dx
    return o


def _generator64(W, b, noise):
    """theta and the hidden activations; W[l] [out][in] float64."""
    hs = [noise.double()]
    for l in range(len(W) - 1):
        p = torch.addmm(b[l], hs[-1], W[l].T)
        hs.append(torch.where(p > 0, p, SLOPE * p))
    o = torch.addmm(b[-1], hs[-1], W[-1].T)
    return 1.0 + _softplus64(o), o, hs


def _adam64(p, g, lr):
    """The first Adam step from zero moments: beta-corrected m = g, v = g^2."""
    return p - lr * g / (g.abs() + 1e-8)


def exact(case, seed):
    t, kind = _inputs(case, seed), case["kind"]
    if kind == "step":
        bf16 = case["precision"] == "bf16"
        o = _sampled_disc64(t["W"], t["b"], t["theta"], case["E"], t["seed"], t["real"], case["features"], False)
        if bf16:
            o["dLg_dx"] = None      # bf16 activations move hidden units across the kink: a tenth off by definition
        return o
    if kind == "three_call":
        o = _sampled_disc64(t["W"], t["b"], t["theta"], case["E"], t["seed"], t["real"], "identity", True)
        o["x"] = _events64(t["theta"].double(), case["E"], 0, case["n_theta"] * case["E"], t["seed"])[0]
        return o
    if kind == "train":
        k, E, seed = case["k"], case["E"], t["seed"]
        N = k * E
        GW, Gb = [w.double() for w in t["GW"]], [v.double() for v in t["Gb"]]
        DW, Db = [w.double() for w in t["DW"]], [v.double() for v in t["Db"]]
        theta, pre, hs = _generator64(GW, Gb, t["noise"][0])
        w0 = _philox(torch.arange(N, device=_dev(), dtype=torch.int64), 4, 1, seed + 5)[0]
        real = t["pool"][(w0 * t["pool"].shape[0]) >> 32]
        o = _sampled_disc64(DW, Db, theta, E, seed, real, "proxy2", False)
        d = o["dLg_dtheta"] * torch.sigmoid(pre)
        gW, gb = [None] * len(GW), [None] * len(GW)
        for l in range(len(GW) - 1, -1, -1):
            gW[l], gb[l] = d.T @ hs[l], d.sum(0)
            if l > 0:
                d = (d @ GW[l]) * torch.where(hs[l] > 0, 1.0, SLOPE)
        return {"theta": theta[None], "loss_d": o["loss_d"], "loss_g": o["loss_g"], "dW": o["dW"], "db": o["db"],
                "dLg_dtheta": o["dLg_dtheta"], "gW": gW, "gb": gb,
                "G_W": [_adam64(p, g, 1e-5) for p, g in zip(GW, gW)], "G_b": [_adam64(p, g, 1e-5) for p, g in zip(Gb, gb)],
                "D_W": [_adam64(p, g, 1e-4) for p, g in zip(DW, o["dW"])],
                "D_b": [_adam64(p, g, 1e-4) for p, g in zip(Db, o["db"])]}
    if kind in ("param_grad", "sample"):
        theta, E = t["theta"].double(), case["E"]
        N, chunk = case["n_theta"] * E, 1 << 24
        if kind == "sample":
            x = torch.empty((N, case["d"]), dtype=torch.float64, device=_dev())
            for i0 in range(0, N, chunk):
                x[i0:min(N, i0 + chunk)] = _events64(theta, E, i0, min(N, i0 + chunk), t["seed"])[0]
            return x
        g, loss = torch.zeros_like(theta), torch.zeros(1, dtype=torch.float64, device=_dev())
        for r in range(case["n_theta"]):
            for i0 in range(r * E, (r + 1) * E, chunk):
                x, da, db = _events64(theta, E, i0, min((r + 1) * E, i0 + chunk), t["seed"])
                loss += (x - 0.5).square().sum()
                g[r, 0::2] += (2.0 * (x - 0.5) * da).sum(0)
                g[r, 1::2] += (2.0 * (x - 0.5) * db).sum(0)
        return {"dL_dtheta": g, "loss": loss}
    if kind == "bootstrap":
        w0 = _philox(torch.arange(case["n_out"], device=_dev(), dtype=torch.int64), 4, t["step"], t["seed"])[0]
        idx = (w0 * case["n_data"]) >> 32
        if case["row_order"]:
            idx = idx.sort().values
        return t["data"][idx]
    th = torch.stack([_generator64([w[m].double() for w in t["W"]], [v[m].double() for v in t["b"]], t["noise"])[0]
                      for m in range(case["M"])])
    mean = th.mean(0)
    p_hat, sigma = mean.mean(0), (th - mean).square().mean(0).sqrt().mean(0)
    p = t["p_true"].double()
    return {"p_hat": p_hat, "sigma": sigma, "r_hat": (p - p_hat) / p}
