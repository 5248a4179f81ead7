"""Performance cases of the Muon step: what a training program has it do.

One pass is one optimizer step over a set of weight matrices, through
``MuonPlan.step`` (a fixed list of matrices, buffers handed over at each call)
or through the torch-style ``Muon`` optimizer.  The sets are the ones this
repository is used on (``paper_2606_27153_amd/workloads.py``: a tiny
transformer, Llama-style 1B and 8B layers, a vision-language-action model,
an MoE expert bank) and generic odd shapes, from 8 small matrices, where
launches and latency count, up to four layers of the 8B model (one owner's
share of 8).

Matrices of one shape are kept as slices of one buffer (an expert bank, a
stack of layers), which is also how the outputs come: one tensor of W and one
of the fp32 momentum per shape, and one of the orthogonalised update where
the program asks for it.
"""
import math

import torch

from paper_2606_27153_amd.optim import Muon, MuonPlan

LR, MOMENTUM, DECAY = 0.02, 0.95, 0.01
QUINTIC = (3.4445, -4.7750, 2.0315)
CUBIC = (1.5, -0.5, 0.0)
# a per-step coefficient set: aggressive first steps, the textbook quintic last
SCHEDULE = (QUINTIC, QUINTIC, QUINTIC, QUINTIC, (1.875, -1.25, 0.375))
_DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def _case(name, shapes, **kw):
    """``shapes``: "RxC*count" items separated by blanks.  param / grad:
    stored dtypes.  precision, aspect, coefs, steps, nesterov: the plan's and
    the step's options.  idle: share of the matrices of the ``idle_from``-th
    and later shapes that got no token this step, with an all-zero gradient
    (idle_kind "zero") or none (idle_kind "none").  out: the caller also asks for the update O.
    api: "plan" (MuonPlan.step) or "optimizer" (Muon.step)."""
    c = {"shapes": shapes, "param": "bf16", "grad": "bf16", "precision": "bf16", "aspect": -1.0, "coefs": "fixed",
         "steps": 5, "nesterov": True, "idle": 0.0, "idle_from": 0, "idle_kind": "zero", "out": False, "api": "plan"}
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def _llama(d, kv, ffn, layers):
    return f"{d}x{d}*{2 * layers} {d}x{kv}*{2 * layers} {d}x{ffn}*{2 * layers} {ffn}x{d}*{layers}"


def listed():
    return [
        # the tiny 2-layer transformer, fp32 weights: launches and latency
        _case("tiny_set", "256x768*2 256x256*2 256x1024*2 1024x256*2", param="f32", grad="f32"),
        # ragged odd shapes (probe heads, adapters, routers), fp32 master weights and bf16 gradients, update logged
        _case("ragged_set", "65x200*1 200x65*1 130x700*1 700x130*1 257x513*1 513x257*1 1000x1000*1 96x4304*1 "
              "7x13*1 1152x1200*1 300x300*1", param="f32", out=True),
        # the 200 small projections of the vision-language-action model
        _case("small_projections", "32x512*25 32x1024*25 64x512*25 64x1024*25 128x512*25 128x1024*25 256x512*25 "
              "256x1024*25"),
        # one large square weight on its own, update logged
        _case("one_square", "4096x4096*1", out=True),
        # one Llama-style 1B layer through the torch optimizer
        _case("layer_1b_optimizer", _llama(2048, 512, 5632, 1), api="optimizer"),
        # two such layers with fp16 Newton-Schulz and a per-step coefficient set, update logged
        _case("layers_1b_fp16", _llama(2048, 512, 5632, 2), precision="fp16", coefs="schedule", out=True),
        # fp32 Newton-Schulz (validation runs) over a small decoder layer
        _case("layer_fp32", _llama(1024, 256, 2816, 1), param="f32", grad="f32", precision="fp32", out=True),
        # Eq. 2 for every matrix (gram_min_aspect 0), no Nesterov momentum: an action-expert stack
        _case("action_expert_eq2", "1024x1024*12 1024x256*12 1024x4096*12 4096x1024*6", aspect=0.0, nesterov=False),
        # the vision tower and action expert of the vision-language-action model
        _case("vla_towers", "1152x3456*27 1152x1152*27 1152x4304*27 4304x1152*27 1024x1024*36 1024x256*36 "
              "1024x4096*36 4096x1024*18"),
        # two MoE layers: 64 experts each, a quarter of them unrouted (zero gradients)
        _case("moe_layers", "2048x2048*4 2048x512*4 2048x1408*256 1408x2048*128", idle=0.25, idle_from=2),
        # the whole 16-layer 1B model
        _case("set_1b", _llama(2048, 512, 5632, 16)),
        # one owner's share (of 8) of the 8B model: four layers
        _case("share_8b", _llama(4096, 1024, 14336, 4)),
    ]


def _log(rng, lo, hi, step=1):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step
    return max(step, min(hi // step * step, max(lo, v)))


_LARGEST = 4.6e13  # flops of the largest listed case, a little under


def draw(rng):
    """A case of the same ranges: family, sizes, counts, dtypes and options."""
    while True:
        fam = rng.choice(["small", "ragged", "projections", "layers", "layers", "towers", "moe", "square"])
        kw = {}
        kw["param"], kw["grad"] = rng.choice([("bf16", "bf16")] * 4 + [("f32", "f32"), ("f32", "bf16")])
        kw["nesterov"] = rng.random() < 0.85
        kw["steps"] = rng.choice([5, 5, 5, 5, 4, 6])
        kw["precision"] = rng.choice(["bf16"] * 6 + ["fp16"] * 2 + ["fp32"])
        if rng.random() < 0.15:
            kw["coefs"] = rng.choice(["schedule", "cubic"])
            kw["steps"] = 5
        if rng.random() < 0.12:
            kw["aspect"] = 0.0
        if fam == "small":
            d = _log(rng, 64, 512, 8)
            n = rng.randint(1, 4)
            s = f"{d}x{3 * d}*{n} {d}x{d}*{n} {d}x{4 * d}*{n} {4 * d}x{d}*{n}"
            kw["api"] = rng.choice(["plan", "optimizer"])
        elif fam == "ragged":
            s = " ".join(f"{_log(rng, 5, 1500)}x{_log(rng, 5, 4400)}*1" for _ in range(rng.randint(3, 12)))
            kw["out"] = rng.random() < 0.5
        elif fam == "projections":
            s = " ".join(f"{_log(rng, 16, 384, 4)}x{_log(rng, 256, 1600, 4)}*{rng.randint(4, 30)}"
                         for _ in range(rng.randint(3, 9)))
        elif fam == "layers":
            d = _log(rng, 512, 4096, 64)
            s = _llama(d, max(64, d // rng.choice([4, 4, 8, 1])), int(d * rng.choice([2.6875, 2.75, 3.5, 4])) // 32 * 32,
                       rng.randint(1, 6))
            kw["api"] = rng.choice(["plan", "plan", "optimizer"])
        elif fam == "towers":
            d, e = _log(rng, 640, 1536, 32), _log(rng, 512, 1280, 32)
            f, n = _log(rng, 3 * d, 4 * d, 16), rng.randint(2, 20)
            s = f"{d}x{3 * d}*{n} {d}x{d}*{n} {d}x{f}*{n} {f}x{d}*{n} {e}x{e}*{n} {e}x{4 * e}*{n} {4 * e}x{e}*{n}"
        elif fam == "moe":
            d, f, n = _log(rng, 768, 2560, 64), _log(rng, 384, 1792, 64), rng.choice([16, 32, 64])
            s = f"{d}x{d}*2 {d}x{f}*{2 * n} {f}x{d}*{n}"
            kw.update(idle=rng.choice([0.0, 0.25, 0.5]), idle_from=1, idle_kind=rng.choice(["zero", "none"]))
        else:
            d = _log(rng, 512, 4608, 16)
            s = f"{d}x{d}*{rng.randint(1, 3)}"
            kw["out"] = rng.random() < 0.5
        if kw.get("api") == "optimizer":  # torch keeps a gradient in its parameter's dtype
            kw["grad"] = kw["param"]
        case = _case(None, s, **kw)
        # fp32 matrix cores run at a sixteenth of the 16-bit rate
        cost = work(case)["flops"] * (16 if case["precision"] == "fp32" else 1)
        if cost <= _LARGEST and _elements(case) <= 1.1e9:
            return case


# ---------------------------------------------------------------- the set

def _shapes(case):
    out = []
    for item in case["shapes"].split():
        rc, n = item.split("*")
        r, c = rc.split("x")
        out.append((int(r), int(c), int(n)))
    return out


def _elements(case):
    return sum(r * c * n for r, c, n in _shapes(case))


def _idle(case, group, n):
    """Which of the n matrices of a shape got no gradient: evenly spread."""
    k = int(n * case["idle"]) if group >= case["idle_from"] else 0
    return {int((i + 0.5) * n / k) for i in range(k)} if k else set()


def _inputs(case, seed):
    """Per shape, banks of W, G and M: [count, rows * cols] with rows padded to
    16 bytes.  Gradients carry a low-rank part over noise, on a scale of their
    own per matrix; momentum is a few steps' worth of such gradients."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)
    banks = []
    for group, (r, c, n) in enumerate(_shapes(case)):
        stride = (r * c + 7) // 8 * 8
        bank = {k: torch.zeros(n, stride, device="cuda", dtype=t) for k, t in
                (("w", _DT[case["param"]]), ("g", _DT[case["grad"]]), ("m", torch.float32))}
        idle = _idle(case, group, n)
        for i in range(n):
            view = {k: b[i, :r * c].view(r, c) for k, b in bank.items()}
            scale = 1e-3 * 10.0 ** (2.0 * torch.rand((), device="cuda", generator=g) - 1.0)
            view["w"].copy_(torch.randn(r, c, device="cuda", generator=g) * 0.02)
            low = torch.randn(r, 4, device="cuda", generator=g) @ torch.randn(4, c, device="cuda", generator=g)
            if i not in idle:
                view["g"].copy_((torch.randn(r, c, device="cuda", generator=g) + 0.5 * low) * scale)
                view["m"].copy_((torch.randn(r, c, device="cuda", generator=g) + 0.5 * low) * (3.0 * scale))
            elif case["idle_kind"] == "none":  # momentum from steps in which it was routed
                view["m"].copy_(torch.randn(r, c, device="cuda", generator=g) * (3.0 * scale))
        banks.append(bank)
    return banks


def _coefs(case):
    if case["coefs"] == "schedule":
        return SCHEDULE
    if case["coefs"] == "cubic":
        return (QUINTIC,) * 4 + (CUBIC,)
    return None


def _views(case, banks, key):
    return [b[key][i, :r * c].view(r, c) for b, (r, c, n) in zip(banks, _shapes(case)) for i in range(n)]


def prepare(case, seed):
    banks = _inputs(case, seed)
    ws, gs, ms = (_views(case, banks, k) for k in "wgm")
    if case["idle_kind"] == "none":
        j = 0
        for group, (_, _, n) in enumerate(_shapes(case)):
            for i in _idle(case, group, n):
                gs[j + i] = None
            j += n
    state = {"case": case, "banks": banks, "steps": case["steps"], "nesterov": case["nesterov"]}
    aspect = None if case["aspect"] < 0 else case["aspect"]
    if case["api"] == "optimizer":
        params = [torch.nn.Parameter(w) for w in ws]
        opt = Muon(params, lr=LR, momentum=MOMENTUM, weight_decay=DECAY, ns_steps=case["steps"],
                   nesterov=case["nesterov"], precision=case["precision"], gram_min_aspect=aspect,
                   ns_coefficients=_coefs(case))
        for p, g, m in zip(params, gs, ms):
            p.grad = g
            opt.state[p]["momentum_buffer"] = m
        state["opt"] = opt
        return state
    descs = [(r, c, case["param"], case["grad"]) for r, c, n in _shapes(case) for _ in range(n)]
    plan = MuonPlan(descs, precision=case["precision"], gram_min_aspect=aspect, abc=_coefs(case))
    if case["out"]:
        for b in banks:
            b["o"] = torch.zeros_like(b["m"])
    state.update(plan=plan, w=ws, g=gs, m=ms, o=_views(case, banks, "o") if case["out"] else None,
                 workspace=plan.workspace("cuda"))
    return state


def run(state):
    if "opt" in state:
        state["opt"].step()
    else:
        state["plan"].step(state["w"], state["g"], state["m"], lr=LR, momentum=MOMENTUM, weight_decay=DECAY,
                           ns_steps=state["steps"], nesterov=state["nesterov"], workspace=state["workspace"],
                           update_out=state["o"])
    return [{k: b[k] for k in ("w", "m", "o") if k in b} for b in state["banks"]]


# ---------------------------------------------------------------- what a pass needs

def work(case):
    """Bytes: G read once, W and M read and written once (O written once).
    Flops: the Newton-Schulz products with symmetry used, in the cheaper of
    the two forms the method has: Eq. 2 (3 m^2 n + m^3 a step) or the
    Gram-space recurrence (Eq. 4) restarted every 2 steps, which it needs in
    16 bits (3 m^2 n and (4L - 3) m^3 per segment of L steps).  A matrix
    without a gradient, or with an all-zero one, needs none."""
    size = {"f32": 4, "bf16": 2}
    k = case["steps"]
    nbytes = flops = 0.0
    for group, (r, c, n) in enumerate(_shapes(case)):
        m, q = float(min(r, c)), float(max(r, c))
        idle = len(_idle(case, group, n))
        moved = n - idle if case["idle_kind"] == "none" else n
        nbytes += moved * r * c * (size[case["grad"]] + 2 * size[case["param"]] + 8 + (4 if case["out"] else 0))
        segs = [2] * (k // 2) + [1] * (k % 2)
        eq2 = k * (3 * m * m * q + m ** 3)
        eq4 = sum(3 * m * m * q + (4 * s - 3) * m ** 3 for s in segs)
        flops += (n - idle) * min(eq2, eq4)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Largest relative error of any output.  With the update O among them it
    is O's, the error of the 16-bit (fp32) Newton-Schulz products; otherwise
    W's, in which O counts by lr * |O| / |W|, about 1.5 %, next to the
    rounding of W to its own type.  About four times the distance to ``exact``
    (O: 1.3e-2 in bf16, 7e-4 in fp16 and 2e-3 there for small m, 1e-6 in
    fp32; fp32 W: 7e-4, 1e-4, 6e-8); bf16 W is at most 2.0e-3 away, almost all
    of it its final rounding, which every implementation shares."""
    if case["out"]:
        return {"rel": {"bf16": 5e-2, "fp16": 7e-3, "fp32": 5e-6}[case["precision"]]}
    if case["param"] == "bf16":
        return {"rel": 3e-3}
    return {"rel": {"bf16": 2.5e-3, "fp16": 4e-4, "fp32": 3e-7}[case["precision"]]}


def exact(case, seed):
    """The step in 64 bits: momentum, Newton-Schulz (Eq. 2) on the normalised,
    wide-oriented input, and the update with decoupled weight decay."""
    banks = _inputs(case, seed)
    lr, mu, wd = (float(torch.tensor(v, dtype=torch.float32)) for v in (LR, MOMENTUM, DECAY))
    coefs = _coefs(case) or (QUINTIC,) * case["steps"]
    coefs = [tuple(float(torch.tensor(v, dtype=torch.float32)) for v in t) for t in coefs]
    out = []
    for group, (b, (r, c, n)) in enumerate(zip(banks, _shapes(case))):
        idle = _idle(case, group, n)
        res = {k: torch.zeros(b["m"].shape, device="cuda", dtype=torch.float64)
               for k in (("w", "m", "o") if case["out"] else ("w", "m"))}
        for i in range(n):
            w, g, m = (b[k][i, :r * c].view(r, c).double() for k in "wgm")
            if i in idle and case["idle_kind"] == "none":
                res["w"][i, :r * c], res["m"][i, :r * c] = w.reshape(-1), m.reshape(-1)
                continue
            m = mu * m + g
            u = g + mu * m if case["nesterov"] else m
            x = u.T if r > c else u
            norm = float(x.norm())
            x = x / (norm + 1e-7) if norm else x
            for a, bb, cc in coefs[:case["steps"]] if norm else ():
                gram = x @ x.T
                x = a * x + (bb * gram + cc * (gram @ gram)) @ x
            o = x.T if r > c else x
            w = w * (1.0 - lr * wd) - lr * math.sqrt(max(1.0, r / c)) * o
            res["w"][i, :r * c], res["m"][i, :r * c] = w.reshape(-1), m.reshape(-1)
            if case["out"]:
                res["o"][i, :r * c] = o.reshape(-1)
        out.append(res)
    return out
