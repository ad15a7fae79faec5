"""What a program that profiles gradients with this package has it do, as cases to measure.

A window of the profiler is: describe the blocks, feed one gradient per sampled step, take the per-block statistics
and the risk table, solve the allocation.  `step` cases are one steady-state step, `finalize` cases the statistics and
the risk table of a window that is under way, `window` cases the whole of it up to the risk table, `sampled` cases one
step on a sparse sample (gather, then the step on the compact buffer), `allocate` the solver on a risk table.
"""
import math
import random

import numpy as np
import torch

import paper_2605_04711_amd as B
from paper_2605_04711_amd import binding

DEVICE = "cuda:0"
F32, BF16 = binding.GRAD_F32, binding.GRAD_BF16
DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
GROUP = 256                    # coordinates per 8-bit group; the states of a block are padded to whole groups
RING = 4                       # distinct gradients a window cycles through
WARM = 3                       # steps already taken in the state of a step or finalize case


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def listed():
    resnet = dict(layout="convnet", depth="3,4,6,3", width=64, classes=1000)
    gpt2 = dict(layout="gpt", layers=12, d=768, vocab=50257, positions=1024)
    gpt_1p3b = dict(layout="gpt", layers=24, d=2048, vocab=50257, positions=2048)
    llama = dict(layout="llama", layers=16, d=4096, ffn=11008, vocab=32000)      # half of the 7B layout's layers: 3.5 G coordinates
    ragged = dict(layout="mixed", blocks=240, total=60_000_000, shapes=11)
    return [
        # a step inside the training loop of a toy model: launches and host work only
        dict(name="step_tiny_f32", op="step", layout="equal", blocks=8, rows=64, cols=64, grad="f32", pad=64),
        # image model, 161 blocks, most of them small vectors next to 3 x 3 convolutions; 25.6 M coordinates
        dict(name="step_resnet50_f32", op="step", grad="f32", pad=64, **resnet),
        # the largest fp32-gradient step: decoder with biased linears, 1.3 G coordinates
        dict(name="step_gpt_1p3b_f32", op="step", grad="f32", pad=64, **gpt_1p3b),
        # the largest step: bf16 gradients of a decoder without biases
        dict(name="step_llama_bf16", op="step", grad="bf16", pad=64, **llama),
        # statistics, structure residual and distortion, risk over 6 candidates: image model, fp32 parameters
        dict(name="finalize_resnet50_f32", op="finalize", grad="f32", theta="f32", k=6, pad=64, **resnet),
        # the same for a small language model in bf16, one embedding a third of all coordinates
        dict(name="finalize_gpt2_bf16", op="finalize", grad="bf16", theta="bf16", k=6, pad=64, **gpt2),
        # the same for the largest layout
        dict(name="finalize_llama_bf16", op="finalize", grad="bf16", theta="bf16", k=6, pad=64, **llama),
        # a whole window on a toy model
        dict(name="window_tiny_f32", op="window", layout="equal", blocks=8, rows=64, cols=64, grad="f32", theta="f32", k=4, steps=16, pad=64),
        # a whole window on blocks of odd sizes packed without gaps (arbitrary alignment), fp32 master parameters
        dict(name="window_ragged_bf16", op="window", grad="bf16", theta="f32", k=6, steps=32, pad=1, **ragged),
        # a whole window of a small language model with all 21 candidates
        dict(name="window_gpt2_f32", op="window", grad="f32", theta="f32", k=21, steps=16, pad=64, **gpt2),
        # the paper's sparse profiling: one sampled step at 1 % of the largest layout
        dict(name="sampled_llama_bf16", op="sampled", grad="bf16", ratio=0.01, pad=64, **llama),
        # the solver on a risk table of a diffusion model's size, all 21 candidates, memory and time row
        dict(name="allocate_686x21", op="allocate", blocks=686, k=21, memory=0.5, time=1.0),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_layout(rng, lo, hi):
    """A layout of between lo and hi coordinates."""
    total = int(_log_uniform(rng, lo, hi))
    if rng.random() < 0.6 or total < 1_000_000:
        n = max(1, min(int(_log_uniform(rng, 2, 700)), total // 64))
        return dict(layout="mixed", blocks=n, total=total, shapes=rng.randrange(1 << 30), pad=rng.choice([1, 1, 64]))
    layers = rng.randint(1, 32)
    llama = rng.random() < 0.5
    d = max(64, int(math.sqrt(total / (layers * (12.06 if llama else 12.0) + 16))))     # the vocabulary is 8 d
    d = rng.choice([d // 64 * 64, d // 4 * 4, d]) if d >= 128 else 64
    if llama:
        return dict(layout="llama", layers=layers, d=d, ffn=int(2.6875 * d), vocab=8 * d, pad=rng.choice([1, 64]))
    return dict(layout="gpt", layers=layers, d=d, vocab=8 * d + rng.choice([0, 17]), positions=d, pad=rng.choice([1, 64]))


def draw(rng):
    op = rng.choice(["step", "step", "finalize", "finalize", "window", "sampled", "allocate"])
    grad, theta = rng.choice(["f32", "bf16"]), rng.choice(["f32", "bf16", "bf16", "none"])
    if op == "step":
        return dict(op=op, grad=grad, **_draw_layout(rng, 3e4, 1.3e9 if grad == "f32" else 3e9))
    if op == "finalize":
        return dict(op=op, grad=grad, theta=theta, k=rng.choice([4, 6, 21]), **_draw_layout(rng, 3e4, 2.5e9))
    if op == "window":
        return dict(op=op, grad=grad, theta=theta, k=rng.choice([4, 6, 21]), steps=rng.randint(4, 32), **_draw_layout(rng, 3e4, 6e7))
    if op == "sampled":
        return dict(op=op, grad=grad, ratio=round(_log_uniform(rng, 1e-3, 0.1), 5), **_draw_layout(rng, 1e6, 1e9))
    return dict(op=op, blocks=rng.randint(8, 686), k=rng.choice([4, 6, 21]), memory=round(rng.uniform(0.25, 0.9), 2),
                time=round(rng.uniform(0.7, 1.3), 2))


# ---------------------------------------------------------------------------
# layouts: (offset, numel, rows, cols) per block; rows = cols = 0 for vectors
# ---------------------------------------------------------------------------

def _shapes(case):
    kind, out = case["layout"], []
    if kind == "equal":
        return [(case["rows"], case["cols"])] * case["blocks"]
    if kind == "convnet":            # bottleneck residual network: convolution, then two norm vectors
        def conv(cin, cout, k):
            out.extend([(cout, cin * k * k), (cout, 0), (cout, 0)])
        w0 = case["width"]
        conv(3, w0, 7)
        cin = w0
        for stage, n in enumerate(int(x) for x in case["depth"].split(",")):
            w = w0 << stage
            for unit in range(n):
                conv(cin, w, 1); conv(w, w, 3); conv(w, 4 * w, 1)
                if unit == 0:
                    conv(cin, 4 * w, 1)
                cin = 4 * w
        return out + [(case["classes"], cin), (case["classes"], 0)]
    if kind == "gpt":                # learned positions, biased linears, two norms per layer
        d = case["d"]
        out = [(case["vocab"], d), (case["positions"], d)]
        for _ in range(case["layers"]):
            out += [(d, 0), (d, 0), (d, 3 * d), (3 * d, 0), (d, d), (d, 0), (d, 0), (d, 0), (d, 4 * d), (4 * d, 0), (4 * d, d), (d, 0)]
        return out + [(d, 0), (d, 0)]
    if kind == "llama":              # no biases, gated MLP, separate head
        d, f = case["d"], case["ffn"]
        out = [(case["vocab"], d)]
        for _ in range(case["layers"]):
            out += [(d, 0), (d, d), (d, d), (d, d), (d, d), (d, 0), (f, d), (f, d), (d, f)]
        return out + [(d, 0), (case["vocab"], d)]
    if kind == "mixed":              # sizes over four decades, a third vectors, the rest matrices of any shape
        rng = random.Random(case["shapes"])
        weight = [math.exp(rng.uniform(0.0, math.log(1e4))) for _ in range(case["blocks"])]
        for w in weight:
            n = max(1, int(case["total"] * w / sum(weight)))
            if n < 16 or rng.random() < 0.33:
                out.append((n, 0))
            else:
                rows = min(n // 2, max(2, int(math.sqrt(n) * math.exp(rng.uniform(-1.5, 1.5)))))
                out.append((rows, max(2, n // rows)))
        return out
    raise KeyError(kind)


def _blocks(case):
    at, out = 0, []
    for r, c in _shapes(case):
        at = -(-at // case["pad"]) * case["pad"]
        out.append((at, r * c if c else r, r if c else 0, c))
        at += out[-1][1]
    return out, -(-at // 64) * 64


def _padded(n):
    return -(-n // GROUP) * GROUP


CONFIGS4 = [(1, 1, 0, 0, 32), (1, 1, 0, 0, 8), (1, 1, 0, 0, 16), (0, 0, 0, 0, 32)]
CONFIGS6 = [(1, 1, 0, 0, 32), (1, 1, 0, 0, 16), (1, 1, 0, 0, 8), (0, 1, 0, 0, 32), (0, 0, 0, 0, 32), (1, 0, 0, 1, 32)]
MECHANISMS = [(1, 1, 1, 0), (1, 1, 0, 0), (0, 0, 0, 0), (0, 1, 0, 0), (0, 0, 1, 0), (0, 1, 1, 0), (1, 0, 0, 1)]
CONFIGS = {4: CONFIGS4, 6: CONFIGS6, 21: [(*y, b) for y in MECHANISMS for b in (32, 16, 8)]}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gradients(case, seed, count, blocks, numel):
    """`count` flat gradients: a persistent direction plus fresh noise, times a log-normal scale per coordinate
    (spread 0, 0.5 and 2 in turn, so light and heavy tails); noise levels over three decades from block to block."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(1_000_003 * seed + 17)
    rng = random.Random(seed)
    bufs = [torch.zeros(numel, dtype=DTYPE[case["grad"]], device=DEVICE) for _ in range(count)]
    for i, (o, n, _, _) in enumerate(blocks):
        delta, sigma, spread = rng.random(), 10.0 ** rng.uniform(-4.0, -1.0), (0.0, 0.5, 2.0)[i % 3]
        scale = torch.randn(n, device=DEVICE, generator=gen).mul_(spread).exp_()
        fixed = torch.randn(n, device=DEVICE, generator=gen).mul_(delta / math.sqrt(n)).mul_(scale)
        scale.mul_(sigma)
        for buf in bufs:
            buf[o:o + n].copy_(torch.randn(n, device=DEVICE, generator=gen).mul_(scale).add_(fixed))
    return bufs


def _theta(case, seed, numel):
    if case.get("theta", "none") == "none":
        return None
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(7_919 * seed + 5)
    return torch.randn(numel, device=DEVICE, generator=gen).mul_(0.02).to(DTYPE[case["theta"]])


def _span(prof, blocks):
    """m, v and g_prev of all blocks: the states of consecutive blocks lie next to each other, padded to whole groups."""
    total = sum(_padded(n) for _, n, _, _ in blocks)
    base, out = prof.workspace.data_ptr(), []
    for view in prof.state(0):
        at = view.data_ptr() - base
        out.append(prof.workspace[at:at + total * view.element_size()].view(view.dtype))
    return out


def _allocation(case, seed):
    """Risk table from block signals as a profile gives them, state bytes and time costs of the candidates."""
    rng = np.random.default_rng([seed, 0xA110C])
    n, cfgs = case["blocks"], CONFIGS[case["k"]]
    numel = np.exp(rng.uniform(math.log(320.0), math.log(3e7), n)).astype(np.int64)
    s_a, s_m, c, f = np.clip(rng.normal(0.7, 0.5, n), 0, 1), rng.random(n) ** 2, rng.random(n), rng.random(n)
    loss = {32: np.zeros(n), 16: rng.uniform(1e-7, 1e-4, n), 8: rng.uniform(1e-3, 3.0, n)}
    risk, mem, time = (np.zeros((n, len(cfgs)), t) for t in (np.float64, np.int64, np.float64))
    for k, (ya, ym, yd, yf, bits) in enumerate(cfgs):
        agg = (1 - ya) + (1 - ym) + (1 - yd) + yf + 32.0 / bits - 1.0
        risk[:, k] = s_a * (1 - ya) + s_m * (1 - ym) + c * (1 - yd) + f * yf + loss[bits] + 0.1 * agg
        state = numel * (bits // 8) + (4 * (-(-numel // GROUP)) if bits == 8 else 0)
        factored = 2 * np.sqrt(numel.astype(np.float64)).astype(np.int64) * (bits // 8)
        mem[:, k] = ym * state + ya * (factored if yf else state)
        time[:, k] = (0.4 + 0.2 * ym + 0.4 * ya + 0.5 * yf + 0.05 * yd) * (1.3 if bits == 8 else 1.0)
    return dict(risk=risk, mem=mem, time=time, budget=int(case["memory"] * 8 * int(numel.sum())), cap=float(case["time"] * n))


def prepare(case, seed):
    op = case["op"]
    if op == "allocate":
        return dict(op=op, **_allocation(case, seed))
    blocks, numel = _blocks(case)
    dtype = F32 if case["grad"] == "f32" else BF16
    params = binding.default_profile_params(grad_dtype=dtype)
    if op == "window":
        return dict(op=op, blocks=blocks, params=params, grads=_gradients(case, seed, RING, blocks, numel), steps=case["steps"],
                    theta=_theta(case, seed, numel), configs=CONFIGS[case["k"]],
                    workspace=torch.empty(binding.workspace_bytes(blocks, params), dtype=torch.uint8, device=DEVICE))
    if op == "sampled":
        grads = _gradients(case, seed, WARM + 1, blocks, numel)
        sampler = B.Sampler(blocks, case["ratio"], seed=seed, device=DEVICE)
        compact = torch.zeros(sampler.compact_numel, dtype=DTYPE[case["grad"]], device=DEVICE)
        prof = B.Profiler(sampler.compact_blocks, params, device=DEVICE)
        for g in grads[:WARM]:
            prof.step(sampler.gather(g, out=compact))
        return dict(op=op, sampler=sampler, prof=prof, compact=compact, grad=grads[WARM], span=_span(prof, sampler.compact_blocks))
    grads = _gradients(case, seed, WARM + (op == "step"), blocks, numel)
    prof = B.Profiler(blocks, params, device=DEVICE)
    for g in grads[:WARM]:
        prof.step(g)
    if op == "step":
        return dict(op=op, prof=prof, grad=grads[WARM], span=_span(prof, blocks))
    return dict(op=op, prof=prof, theta=_theta(case, seed, numel), configs=CONFIGS[case["k"]])


# every statistic of a block that is not a constant; the fp32 direction against itself (lQ32) is one
FIELDS = ["rho_bar", "cos_last", "snr", "A", "q10", "q90", "Q16", "Q8", "lQ16", "lQ8", "err_m16", "err_v16", "err_m8", "err_v8",
          "s_A", "s_rho", "s_snr", "s_M", "C_tilde", "s_F", "m_sq", "v_l1", "g_sq_last", "C", "F"]
_COLUMN = {f: getattr(binding.BlockStats, f).offset // 8 for f in FIELDS}


def _finalized(stats, risk):
    a = np.frombuffer(stats, np.float64).reshape(len(stats), -1)
    out = {f: a[:, k] for f, k in _COLUMN.items()}
    out["risk"] = risk
    return out


def run(state):
    op = state["op"]
    if op == "step":
        state["prof"].step(state["grad"])
        return state["span"]
    if op == "finalize":
        return _finalized(*state["prof"].finalize(state["configs"], theta=state["theta"]))
    if op == "sampled":
        state["prof"].step(state["sampler"].gather(state["grad"], out=state["compact"]))
        return [state["compact"], *state["span"]]
    if op == "allocate":
        choice, objective, mem, time = B.allocate(state["risk"], state["mem"], state["time"], state["budget"], state["cap"])
        return [choice.astype(np.int64), objective, mem, time]
    prof = B.Profiler(state["blocks"], state["params"], device=DEVICE, workspace=state["workspace"])
    grads = state["grads"]
    for t in range(state["steps"]):
        prof.step(grads[t % RING])
    out = _finalized(*prof.finalize(state["configs"], theta=state["theta"]))
    prof.close()
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    if case["op"] == "allocate":
        entries = case["blocks"] * case["k"]
        return dict(bytes=24 * entries + 4 * case["blocks"], flops=3 * entries)
    blocks, _ = _blocks(case)
    size = {"f32": 4, "bf16": 2, "none": 0}
    g, th = size[case["grad"]], size[case.get("theta", "none")]
    d = sum(n for _, n, _, _ in blocks)
    # a step reads the gradient, the previous one and two fp32 states, and writes the latter three; about 70 operations
    # per coordinate (Eq. 3, the sums of Eq. 5, three directions and two round trips of Eq. 8)
    if case["op"] == "step":
        return dict(bytes=(16 + 3 * g) * d, flops=70 * d)
    # the statistics read the second moment and the parameters; about 20 operations per coordinate
    last = dict(bytes=(4 + th) * d, flops=20 * d)
    if case["op"] == "finalize":
        return last
    if case["op"] == "window":                     # the first step reads no state
        return dict(bytes=(16 + 3 * g) * d * (case["steps"] - 1) + (8 + 2 * g) * d + last["bytes"], flops=70 * d * case["steps"] + last["flops"])
    taken = sum(_sample_shape(n, r, c, case["ratio"])[0] for _, n, r, c in blocks)
    return dict(bytes=(2 * g + 16 + 3 * g) * taken, flops=70 * taken)


# Measured over the listed cases and 24 drawn ones.  States against 64 bits: 6.0e-8, largest single difference 1.9e-5 of
# the root mean square.  Statistics with the sums in another order: 2.1e-6 (lQ16, a difference of nearly equal directions;
# everything else 1.1e-7), largest single difference 1.0e-5.  Four times that.
def tolerance(case):
    if case["op"] == "allocate":
        return "exact"                             # whole numbers throughout: the canonical optimum of an integer instance
    if case["op"] in ("step", "sampled"):
        return dict(rel=2.5e-7, max=8e-5)
    return dict(rel=1e-5, max=4e-5)


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

BETA_M, BETA_V = float(np.float32(0.9)), float(np.float32(0.999))
EPS, EPS_U = 1e-12, float(np.float32(1e-8))


def _ema(slices):
    m = v = 0.0
    for g in slices:
        g = g.double()
        m = BETA_M * m + (1.0 - BETA_M) * g
        v = BETA_V * v + (1.0 - BETA_V) * g * g
    return m, v


def _exact_states(slices_of, blocks, grad, last):
    """m, v, g_prev over all blocks, padded: slices_of(i) gives block i's gradients, step by step."""
    total = sum(_padded(n) for _, n, _, _ in blocks)
    m_all, v_all = (torch.zeros(total, dtype=torch.float64, device=DEVICE) for _ in range(2))
    g_all = torch.zeros(total, dtype=DTYPE[grad], device=DEVICE)
    at = 0
    for i, (_, n, _, _) in enumerate(blocks):
        s = slices_of(i)
        m_all[at:at + n], v_all[at:at + n] = _ema(s)
        g_all[at:at + n] = s[last]
        at += _padded(n)
    return [m_all, v_all, g_all]


def _mix(x):
    x = np.asarray(x, np.uint64)
    x = (x ^ (x >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    x = (x ^ (x >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return x ^ (x >> np.uint64(31))


def _sample_shape(n, rows, cols, ratio):
    """(count, rows, cols) of a block's sample: a sub-matrix where it has at least 2 x 2, a vector otherwise."""
    count = min(n, max(1, math.ceil(ratio * n)))
    if rows >= 2 and cols >= 2:
        r = min(rows, max(1, math.floor(rows * math.sqrt(ratio) + 0.5)))
        c = min(cols, -(-count // r))
        if r >= 2 and c >= 2:
            return r * c, r, c
    return count, 0, 0


def _strata(key, count, size):
    j = np.arange(count, dtype=np.uint64)
    lo, hi = j * np.uint64(size) // np.uint64(count), (j + np.uint64(1)) * np.uint64(size) // np.uint64(count)
    return lo + _mix(key + (j + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)) % (hi - lo)


def _sample(case, seed, blocks):
    """The sampled positions of each block and the compact layout (blocks start on multiples of 64)."""
    index, compact, at = [], [], 0
    with np.errstate(over="ignore"):
        for i, (o, n, rows, cols) in enumerate(blocks):
            count, r, c = _sample_shape(n, rows, cols, case["ratio"])
            key = _mix(_mix(np.uint64(seed)) + np.uint64(i))
            if r:
                a, b = _strata(_mix(key + np.uint64(0x52)), r, rows), _strata(_mix(key + np.uint64(0x43)), c, cols)
                pos = (a.astype(np.int64)[:, None] * cols + b.astype(np.int64)[None, :]).reshape(-1)
            else:
                pos = _strata(key, count, n).astype(np.int64)
            at = -(-at // 64) * 64
            index.append(torch.from_numpy(pos + o).to(DEVICE))
            compact.append((at, count, r, c))
            at += count
    return index, compact, -(-at // 64) * 64


def _quantile(v, q):
    pos = q * (v.numel() - 1)
    lo = math.floor(pos)
    hi = min(lo + 1, v.numel() - 1)
    a, b = v[lo].item(), v[hi].item()
    return a + (pos - lo) * (b - a)


def _eight_bits(x, levels):
    pad = torch.zeros(_padded(x.numel()), dtype=x.dtype, device=x.device)
    pad[:x.numel()] = x
    a = pad.view(-1, GROUP).abs().amax(1, keepdim=True)
    scale = levels / a
    scale[~torch.isfinite(scale)] = 0.0
    return ((pad.view(-1, GROUP) * scale).round() * (a / levels)).view(-1)[:x.numel()]


def _dot(a, b):
    return (a * b).sum().item()


def _clip(x, lo, hi):
    return lo if x < lo else hi if x > hi else x


def _block_stats(slices, last_two, rho, rows, cols, theta):
    m, v = _ema(slices)
    z = dict(m_sq=_dot(m, m), v_l1=v.sum().item(), g_sq_last=_dot(last_two[1], last_two[1]), rho_bar=rho[0], cos_last=rho[1])
    z["snr"] = z["m_sq"] / (z["v_l1"] + EPS)
    order = v.sort().values
    z["q10"], z["q90"] = _quantile(order, 0.1), _quantile(order, 0.9)
    del order
    z["A"] = math.log((z["q90"] + EPS) / (z["q10"] + EPS))
    u = m / (v.sqrt() + EPS_U)
    for bits in (16, 8):
        mb, vb = (m.to(torch.bfloat16).double(), v.to(torch.bfloat16).double()) if bits == 16 else (_eight_bits(m, 127.0), _eight_bits(v, 255.0))
        ub = mb / (vb.sqrt() + EPS_U)
        q = _dot(u, ub) / (math.sqrt(_dot(u, u)) * math.sqrt(_dot(ub, ub)) + EPS)
        z["Q%d" % bits] = _clip(0.0 if q != q else q, EPS, 1.0)
        if bits == 16:                             # 1 - Q from the difference of the directions, which is small
            du = ub - u
            miss = 0.5 * (_dot(du, du) - (math.sqrt(_dot(u, u)) - math.sqrt(_dot(ub, ub))) ** 2) / (math.sqrt(_dot(u, u)) * math.sqrt(_dot(ub, ub)) + 1e-300)
            z["lQ16"] = -math.log1p(EPS - miss)
        else:
            z["lQ8"] = -math.log(z["Q8"] + EPS)
        z["err_m%d" % bits] = math.sqrt(_dot(mb - m, mb - m)) / (math.sqrt(z["m_sq"]) + EPS)
        z["err_v%d" % bits] = math.sqrt(_dot(vb - v, vb - v)) / (math.sqrt(_dot(v, v)) + EPS)
    z["C"] = z["F"] = 0.0
    if theta is not None:
        p, th = 1.0 / (v.sqrt() + EPS), theta.double()
        y = (p / p.mean() - 1.0) * th
        z["C"] = math.sqrt(_dot(y, y)) / (math.sqrt(_dot(th, th)) + EPS)
    if rows >= 2 and cols >= 2:
        s = v.view(rows, cols)
        r, c = s.mean(1), s.mean(0)
        mu = r.mean().item()
        off = s - r[:, None] * (c / mu if mu else c * 0.0)[None, :]
        z["F"] = math.sqrt((off * off).sum().item()) / (math.sqrt(_dot(v, v)) + EPS)
    z["s_A"] = _clip((z["A"] - math.log(2.0)) / math.log(5.0), 0.0, 1.0)
    z["s_rho"] = _clip((z["rho_bar"] - 0.2) / 0.4, 0.0, 1.0)
    z["s_snr"] = _clip(math.log1p(z["snr"]) / 2.0, 0.0, 1.0)
    z["s_M"], z["C_tilde"], z["s_F"] = z["s_rho"] * z["s_snr"], math.log1p(z["C"]), _clip(z["F"], 0.0, 1.0)
    return z


def _stability(cosines):
    rho = 0.0
    for i, c in enumerate(cosines):
        rho = c if i == 0 else 0.9 * rho + 0.1 * c
    return rho, cosines[-1] if cosines else 0.0


def _exact_window(case, seed, blocks, numel):
    steps = case["steps"] if case["op"] == "window" else WARM
    ring = _gradients(case, seed, RING if case["op"] == "window" else WARM, blocks, numel)
    theta, configs, rows = _theta(case, seed, numel), CONFIGS[case["k"]], []
    for o, n, r, c in blocks:
        g = [b[o:o + n] for b in ring]
        d = [x.double() for x in g]
        norm = [math.sqrt(_dot(x, x)) for x in d]
        pair = {}
        for t in range(1, steps):
            a, b = (t - 1) % len(g), t % len(g)
            if (a, b) not in pair:
                pair[a, b] = _dot(d[a], d[b]) / (norm[a] * norm[b] + EPS)
        rho = _stability([pair[(t - 1) % len(g), t % len(g)] for t in range(1, steps)])
        last = (d[(steps - 2) % len(g)], d[(steps - 1) % len(g)])
        rows.append(_block_stats([g[t % len(g)] for t in range(steps)], last, rho, r, c, None if theta is None else theta[o:o + n]))
    out = {f: np.array([z[f] for z in rows]) for f in FIELDS}
    loss = {32: 0.0 * out["lQ8"], 16: out["lQ16"], 8: out["lQ8"]}
    out["risk"] = np.stack([out["s_A"] * (1 - ya) + out["s_M"] * (1 - ym) + out["C_tilde"] * (1 - yd) + out["s_F"] * yf + loss[bits]
                            + 0.1 * ((1 - ya) + (1 - ym) + (1 - yd) + yf + 32.0 / bits - 1.0) for ya, ym, yd, yf, bits in configs], 1)
    return out


def exact(case, seed):
    if case["op"] == "allocate":
        return None                                # an integer programme: nothing that 64-bit arithmetic alone would give
    blocks, numel = _blocks(case)
    if case["op"] in ("finalize", "window"):
        return _exact_window(case, seed, blocks, numel)
    grads = _gradients(case, seed, WARM + 1, blocks, numel)
    if case["op"] == "step":
        return _exact_states(lambda i: [g[blocks[i][0]:blocks[i][0] + blocks[i][1]] for g in grads], blocks, case["grad"], WARM)
    index, compact, size = _sample(case, seed, blocks)
    packed = torch.zeros(size, dtype=DTYPE[case["grad"]], device=DEVICE)
    for (o, n, _, _), pos in zip(compact, index):
        packed[o:o + n] = grads[WARM][pos]
    return [packed, *_exact_states(lambda i: [g[index[i]] for g in grads], compact, case["grad"], WARM)]
