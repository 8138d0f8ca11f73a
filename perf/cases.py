"""The work that programs have this framework do, as cases that can be timed.

A case is a dict of plain values.  ``listed()`` gives the standing ones,
``draw(rng)`` one more of the same ranges, ``prepare(case, seed)`` what a
program holds before the call (resident filter-output planes, thresholds, the
plan, output buffers), ``run(state)`` one pass through the public entry
points, ``work(case)`` the bytes and operations a pass cannot do without, and
``exact(case, seed)`` the floating-point results in 64 bits.

Kinds of case:

* ``detect``: planes and detection fused on one filter-output plane (FOP),
  then what a search keeps of it: the whole list in canonical order
  (``keep = "list"``) or the capped N_hp x N_cand list under one of the
  policies (``"top"``, ``"last_alg2"``, ``"last_alg1"``).  Both need the
  number of candidates on the host, as a program does.
* ``batch``: FOPs of uneven lengths (the DM trials of one observation) in one
  persistent launch, then each trial's capped list.
* ``planes``: the harmonic planes written out.
* ``train_sum``: planes and the gradient of a loss on them (autograd).
* ``train_lse``: the log-sum-exp statistic's loss and its gradient (autograd).

Inputs are Exp(1) noise powers with harmonic signals added (power P0/n at the
n-th harmonic); thresholds are k + 6 sqrt(k).  Reduced-precision planes hold
an eighth of the power.
"""
import math

import numpy as np
import torch

import paper_1805_12258_amd as hs

TAU = 0.5                 # of the log-sum-exp statistic
N_CAND = 200              # of the capped lists
SCALE = 0.125             # stored / power of 16-bit planes
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}

_BASE = {"kind": "detect", "T": 85, "N": 1 << 21, "H": 8, "dtype": "f32", "mapping": "paper", "keep": "list", "lens": ""}

# Ranges of draw(): what the listed cases stand for.
POINTS_MAX = 85 << 21     # points of a single FOP
SUM_POINTS_MAX = 85 << 19  # of one whose planes are written out
TERMS_MAX = (85 << 19) * 36   # points x source points of a fractional plane


def _case(name, **kw):
    return dict(_BASE, name=name, **kw)


def listed():
    return [
        # a small plane, whole list: launches and the host's part
        _case("detect_21x64k", T=21, N=1 << 16),
        # an odd shape between the small and the full plane, few planes
        _case("detect_64x100003_h5", T=64, N=100003, H=5),
        # the survey's plane (85 templates x 2^21 bins, 8 planes), whole list
        _case("detect_85x2m", T=85, N=1 << 21),
        # the same plane stored in 16 bits, largest 200 of each harmonic plane
        _case("detect_85x2m_f16_top", T=85, N=1 << 21, dtype="f16", keep="top"),
        # a ragged bin count in bfloat16, whole list
        _case("detect_85x1m_bf16", T=85, N=(1 << 20) + 77, dtype="bf16"),
        # twice the harmonic planes, the last 200 met in Algorithm 2 order
        _case("detect_85x1m_h16_last", T=85, N=1 << 20, H=16, keep="last_alg2"),
        # an observation's DM trials of uneven lengths, capped lists
        _case("batch_6_h16_top", kind="batch", T=85, N=0, H=16, keep="top",
              lens="524288,2097152,1048576,524288,1048576,2097152"),
        # fractional mapping, capped lists
        _case("frac_85x512k_top", T=85, N=1 << 19, mapping="fractional", keep="top"),
        # the planes themselves, for a program that looks at them
        _case("planes_85x512k", kind="planes", T=85, N=1 << 19),
        # one training step through the planes
        _case("train_sum_85x256k", kind="train_sum", T=85, N=1 << 18),
        # one training step on the statistic, small plane
        _case("train_lse_21x64k", kind="train_lse", T=21, N=1 << 16),
        # and the plane of the differentiation workload
        _case("train_lse_85x1m", kind="train_lse", T=85, N=1 << 20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _bits(x):
    return max(0, (int(x) - 1).bit_length())


def draw(rng):
    kind = rng.choice(["detect"] * 6 + ["frac"] + ["batch"] * 2 + ["planes"] + ["train_sum"] * 2 + ["train_lse"] * 2)
    T = rng.choice([21, 33, 43, 64, 85, 85, 85, 101, 127, 128, rng.randrange(5, 129)])
    H = rng.choice([8, 8, 8, 16, 16, 4, 5, 12, rng.randrange(1, 17)])
    c = dict(_BASE, T=T, H=H)
    if kind == "batch":
        c["dtype"] = rng.choice(["f32", "f32", "f16", "bf16"])
        lens = []
        for _ in range(rng.randrange(2, 9)):
            n = rng.choice([1 << 17, 1 << 18, 1 << 19, 1 << 20, 1 << 21, _log_int(rng, 5000, 1 << 20)])
            if (sum(lens) + n) * T * H <= 85 * 16 * 7340032 and _bits(T) + _bits(H) + _bits(n) <= 32:
                lens.append(n)
        return dict(c, kind="batch", N=0, lens=",".join(map(str, lens or [70000, 131072])), keep=rng.choice(["top", "last_alg2"]))
    most = POINTS_MAX if kind == "detect" else SUM_POINTS_MAX if kind in ("planes", "train_sum") else 85 << 20
    if kind == "train_sum":
        most //= 2
    if kind == "train_lse":
        most = most * 8 // max(8, H)
    if kind in ("planes", "train_sum"):
        most = most * 8 // max(8, H)
    if kind == "frac":
        most = min(most, TERMS_MAX * 2 // (H * (H + 1)))
    top = min(most // T, 1 << (32 - _bits(T) - _bits(H)), 1 << 21)
    if H > 8 and kind == "detect":
        top = min(top, (POINTS_MAX * 8) // (T * H))
    N = _log_int(rng, 4000, top)
    if rng.random() < 0.4:                      # powers of two are what transforms give
        N = 1 << (N.bit_length() - 1)
    c["N"] = N
    if kind == "detect":
        c["dtype"] = rng.choice(["f32", "f32", "f16", "bf16"])
        c["keep"] = rng.choice(["list", "list", "top", "last_alg2", "last_alg1"])
        return c
    if kind == "frac":
        return dict(c, mapping="fractional", dtype=rng.choice(["f32", "f16", "bf16"]), keep=rng.choice(["list", "top"]))
    if kind == "planes":
        return dict(c, kind=kind, dtype=rng.choice(["f32", "f32", "f16", "bf16"]))
    return dict(c, kind=kind)


# --- inputs ---------------------------------------------------------------------

def _plane(T, N, H, seed, dtype):
    """[T][ld] stored powers (ld: N rounded up to the pitch the calls take)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    # |complex N(0, 1)|^2 / 2 is Exp(1)
    x = torch.empty((T, N), dtype=torch.float32, device="cuda").exponential_(1.0, generator=g)
    rng = np.random.default_rng(seed)
    c = T // 2
    rows, bins, powers = [], [], []
    for _ in range(max(3, min(50, N >> 15))):
        nh = int(rng.integers(1, H + 1))
        z0 = int(rng.integers(-((T - 1 - c) // nh), (T - 1 - c) // nh + 1))
        f0 = int(rng.integers(min(H + 1, (N - 1) // nh), (N - 1) // nh + 1))
        p0 = float(rng.uniform(8.0, 40.0))
        for n in range(1, nh + 1):
            rows.append(n * z0 + c)
            bins.append(n * f0)
            powers.append(p0 / n)
    x.index_put_((torch.tensor(rows, device="cuda"), torch.tensor(bins, device="cuda")),
                 torch.tensor(powers, dtype=torch.float32, device="cuda"), accumulate=True)
    if dtype != "f32":
        x = (x * SCALE).to(DTYPES[dtype])
    pitch = 4 if dtype == "f32" else 8
    ld = (N + pitch - 1) // pitch * pitch
    if ld == N:
        return x
    out = torch.zeros((T, ld), dtype=x.dtype, device="cuda")
    out[:, :N] = x
    return out


def _thresholds(H, T):
    t = torch.tensor([k + 6.0 * math.sqrt(k) for k in range(1, H + 1)], dtype=torch.float64)
    return t.float()[:, None].repeat(1, T).cuda()


def _capacity(points, H):
    return 16384 + points * H // 500


def _plan(c, lens=None):
    plan = hs.Plan(c["T"], c["N"], c["H"], dtype=c["dtype"], input_scale=1.0 if c["dtype"] == "f32" else SCALE,
                   n_chans=lens, mapping=c["mapping"])
    hs.hs_plan_upload(plan.handle)
    return plan


def prepare(case, seed):
    c = dict(case)
    T, N, H = c["T"], c["N"], c["H"]
    if c["kind"] == "batch":
        lens = [int(n) for n in c["lens"].split(",")]
        planes = [_plane(T, n, H, seed * 1009 + f, c["dtype"]) for f, n in enumerate(lens)]
        caps = [_capacity(T * n, H) for n in lens]
        offs = [sum(caps[:f]) for f in range(len(caps))]

        def i64(v):
            return torch.tensor(v, dtype=torch.int64, device="cuda")
        return {"c": c, "plan": _plan(c, lens), "planes": planes, "ta": _thresholds(H, T),
                "fops": i64([p.data_ptr() for p in planes]), "lds": i64([p.stride(0) for p in planes]),
                "caps": caps, "offs": offs, "caps_d": i64(caps), "offs_d": i64(offs),
                "out": torch.empty((sum(caps), 2), dtype=torch.int32, device="cuda"),
                "counts": torch.empty((len(lens), H + 1), dtype=torch.int64, device="cuda")}
    fop = _plane(T, N, H, seed, c["dtype"])
    s = {"c": c, "plan": _plan(c), "fop": fop}
    if c["kind"] == "detect":
        s["ta"] = _thresholds(H, T)
        s["out"] = torch.zeros((_capacity(T * N, H), 2), dtype=torch.int32, device="cuda")
        s["counts"] = torch.empty(H + 1, dtype=torch.int64, device="cuda")
    elif c["kind"] == "train_sum":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed + 77)
        s["x"] = fop[:, :N].detach().requires_grad_(True)
        s["cotangent"] = torch.randn((H, T, N), generator=g, device="cuda")
    elif c["kind"] == "train_lse":
        s["x"] = fop[:, :N].detach().requires_grad_(True)
    return s


# --- one pass ---------------------------------------------------------------------

def run(state):
    c, plan = state["c"], state["plan"]
    if c["kind"] == "detect":
        out, counts = plan.detect(state["fop"], state["ta"], out=state["out"], counts=state["counts"])
        n = min(int(counts[-1]), out.shape[0])
        if c["keep"] == "list":
            return {"list": hs.sort_candidates(out, n), "counts": counts}   # past the n entries: zeros
        kept, kept_counts = plan.select(out, n, N_CAND, c["keep"])
        return {"kept": kept, "kept_counts": kept_counts, "counts": counts}
    if c["kind"] == "batch":
        hs.hs_detect_batched(plan.handle, state["fops"], state["lds"], state["ta"], state["out"], state["offs_d"],
                             state["caps_d"], state["counts"])
        totals = state["counts"][:, -1].tolist()
        kept = []
        for f, total in enumerate(totals):
            n = min(total, state["caps"][f])
            kept.append(plan.select(state["out"][state["offs"][f]:state["offs"][f] + n], n, N_CAND, c["keep"]))
        return {"kept": kept, "counts": state["counts"]}
    if c["kind"] == "planes":
        return {"planes": plan.sum(state["fop"])}
    if c["kind"] == "train_sum":
        planes = hs.HarmonicSum.apply(state["x"], plan)
        (grad,) = torch.autograd.grad(planes, state["x"], state["cotangent"])
        return {"planes": planes.detach(), "grad": grad}
    loss = hs.HarmonicLSE.apply(state["x"], plan, TAU)
    (grad,) = torch.autograd.grad(loss, state["x"])
    return {"loss": loss.detach(), "grad": grad}


# --- what a pass cannot do without ---------------------------------------------------

def work(case):
    c = case
    T, H = c["T"], c["H"]
    eb = 4 if c["dtype"] == "f32" else 2
    if c["kind"] == "batch":
        points = T * sum(int(n) for n in c["lens"].split(","))
        return {"bytes": points * eb + 4 * H * T, "flops": points * (2 * H - 1)}
    points = T * c["N"]
    if c["kind"] == "detect":
        adds = H * (H - 1) // 2 if c["mapping"] == "fractional" else H - 1
        return {"bytes": points * eb + 4 * H * T, "flops": points * (adds + H)}
    if c["kind"] == "planes":
        return {"bytes": points * (eb + 4 * H), "flops": points * (H - 1)}
    boxes = points * (2 * H - 2)                  # suffix sums, then each value into its box
    if c["kind"] == "train_sum":
        return {"bytes": points * (4 + 4 * H + 4 * H + 4), "flops": points * (H - 1) + boxes}
    # the planes are formed for the statistic and again for its gradient
    return {"bytes": points * 8, "flops": points * (2 * (H - 1) + 2 * 4 * H) + boxes}


# --- the results in 64 bits -------------------------------------------------------------

def _sources(T, N, m):
    rows = torch.div(torch.arange(T, device="cuda") - T // 2, m, rounding_mode="floor") + T // 2
    return rows, torch.div(torch.arange(N, device="cuda"), m, rounding_mode="floor")


def _planes64(x, H):
    T, N = x.shape
    x = x.double()
    hp = torch.empty((H, T, N), dtype=torch.float64, device=x.device)
    hp[0] = x
    for m in range(2, H + 1):
        rows, bins = _sources(T, N, m)
        torch.add(hp[m - 2], x[rows][:, bins], out=hp[m - 1])
    return hp


def _transpose64(g):
    """dL/dFOP from dL/dHP [H][T][N] (overwritten by its suffix sums)."""
    H, T, N = g.shape
    for k in range(H - 2, -1, -1):
        g[k] += g[k + 1]
    out = g[0].clone()
    for m in range(2, H + 1):
        rows, _ = _sources(T, N, m)
        wide = (N + m - 1) // m
        part = torch.zeros((T, wide * m), dtype=torch.float64, device=g.device)
        part[:, :N] = g[m - 1]
        out[:, :wide].index_add_(0, rows, part.view(T, wide, m).sum(2))
    return out


def exact(case, seed):
    c = case
    if c["kind"] in ("detect", "batch"):
        return None                               # candidate words and counts: whole numbers
    T, N, H = c["T"], c["N"], c["H"]
    s = prepare(c, seed)
    x = s["fop"][:, :N]
    hp = _planes64(x, H)
    if c["dtype"] != "f32":
        hp /= SCALE
    if c["kind"] == "planes":
        return {"planes": hp}
    if c["kind"] == "train_sum":
        return {"planes": hp, "grad": _transpose64(s["cotangent"].double())}
    loss = 0.0
    for k in range(H):
        h = hp[k].div_(TAU)
        top = h.max()
        lse = top + torch.log(torch.exp(h - top).sum())
        loss = loss + TAU * lse
        h.sub_(lse).exp_()
    return {"loss": loss, "grad": _transpose64(hp)}
