"""The work that a program has this library do, as cases that can be timed and compared.

Weights, biases and tokens follow the recipes of ``paper_2501_10054_amd.synth`` (N(0, 0.02^2) weights with 1 % of the
input columns of W1 and of the neurons' W2 columns scaled by 8, N(0, 1) tokens), drawn on the GPU from the seed.
Ranges and lines of the online cases are central quantiles and least-squares lines of a calibration sample, computed
here with torch, so that ``exact`` starts from the same numbers as the library.
"""
import math

import torch

from paper_2501_10054_amd import tardis as T

DEV = "cuda"
N_CAL = 512            # calibration tokens behind the online cases' ranges
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}


def _case(name, kind, d, h, n, **more):
    c = {"name": name, "kind": kind, "d": d, "h": h, "n": n, "dtype": "bf16", "coverage": 0.95, "act": "gelu_erf",
         "bias": False, "sketch_bits": 8, "folded_fp8": False, "layers": 1}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: one token through a small 32-bit layer, where launches are all there is
        _case("tiny_token", "forward", 64, 256, 1, dtype="f32", coverage=0.9),
        # a decode step of one sequence: one layer of a 7B-class GELU model
        _case("token", "forward", 4096, 16384, 1),
        # a decode step of one sequence through every FFN of such a model: the layers name their successors, and what
        # stands between them (attention, norms) hands each its token
        _case("step_token", "step", 4096, 16384, 1, layers=32),
        # decode steps of a few sequences; the tight, the usual and the loose range
        _case("batch_4", "forward", 4096, 16384, 4, coverage=0.99),
        _case("batch_16", "forward", 4096, 16384, 16),
        _case("batch_64", "forward", 4096, 16384, 64, coverage=0.85),
        # a ragged batch on a narrower layer with biases, the tanh activation and the 4-bit sketch
        _case("batch_23_narrow", "forward", 2048, 8192, 23, bias=True, act="gelu_tanh", sketch_bits=4),
        # a short prompt of odd length, and the prompt shape the library is measured on
        _case("prompt_333", "forward", 4096, 16384, 333),
        _case("prompt_2048", "forward", 4096, 16384, 2048),
        # the unmodified FFN on that prompt, which the method is compared with and which a program falls back to
        _case("dense_2048", "dense", 4096, 16384, 2048),
        # preparing a layer: ranges and lines from calibration tokens, then folding and the predictor
        _case("calibrate_4096", "calibrate", 4096, 16384, 4096),
        _case("fold", "fold", 4096, 16384, 1),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["tiny", "tokens", "tokens", "pass", "prompt", "prompt", "step", "dense", "calibrate", "fold"])
    coverage = rng.choice([0.99, 0.95, 0.9, 0.85])
    common = dict(coverage=coverage, act=rng.choice(["gelu_erf", "gelu_tanh", "relu"]), bias=rng.random() < 0.4)
    if kind == "tiny":       # small 32-bit layers, sizes that are not round
        return _draw("forward", log_int(32, 256), log_int(64, 1024), log_int(1, 32), dtype="f32", **common)
    d = rng.choice([512, 1024, 1536, 2048, 3072, 4096])
    h = rng.choice([4 * d, 4 * d, 2 * d, log_int(1000, 4 * d) // 8 * 8])
    sketch = rng.choice([8, 8, 4])
    fp8 = rng.random() < 0.15
    if kind == "tokens":
        return _draw("forward", d, h, log_int(1, 16), sketch_bits=sketch, folded_fp8=fp8, **common)
    if kind == "pass":
        return _draw("forward", d, h, rng.randint(17, 64), sketch_bits=sketch, **common)
    if kind == "prompt":
        return _draw("forward", d, h, log_int(65, 3000), sketch_bits=sketch, **common)
    if kind == "step":
        d = rng.choice([1024, 2048, 4096])
        return _draw("step", d, 4 * d, log_int(1, 16), layers=rng.randint(2, 12), sketch_bits=sketch, **common)
    if kind == "dense":
        return _draw("dense", d, h, log_int(1, 2500), **common)
    if kind == "calibrate":
        return _draw("calibrate", d, h, log_int(500, 4096), **common)
    return _draw("fold", d, h, 1, sketch_bits=sketch, **common)


def _draw(kind, d, h, n, **more):
    c = _case("", kind, d, h, n, **more)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _weights(case, gen):
    """W1, W2, b1, b2 of one layer."""
    d, h, dt = case["d"], case["h"], _TORCH[case["dtype"]]
    W1 = torch.randn(h, d, device=DEV, generator=gen).mul_(0.02)
    W2 = torch.randn(d, h, device=DEV, generator=gen).mul_(0.02)
    if case["dtype"] == "bf16":
        W1[:, torch.randperm(d, device=DEV, generator=gen)[:max(1, d // 100)]] *= 8.0
        W2[:, torch.randperm(h, device=DEV, generator=gen)[:max(1, h // 100)]] *= 8.0
    b1 = b2 = None
    if case["bias"]:
        b1 = torch.randn(h, device=DEV, generator=gen).mul_(0.05).to(dt)
        b2 = torch.randn(d, device=DEV, generator=gen).mul_(0.05).to(dt)
    return W1.to(dt), W2.to(dt), b1, b2


def _act(z, act):
    if act == "gelu_erf":
        return 0.5 * z * (1.0 + torch.erf(z * math.sqrt(0.5)))
    if act == "gelu_tanh":
        return 0.5 * z * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (z + 0.044715 * z ** 3)))
    return z.clamp_min(0.0) if act == "relu" else z


def _fit(z, coverage, act):
    """Central ranges and least-squares lines per row of z (neurons x samples): lo, hi, a, c in 64 bits."""
    n = z.shape[1]
    z = z.sort(dim=1).values

    def quantile(q):
        pos = q * (n - 1)
        i = min(max(int(math.floor(pos)), 0), n - 1)
        lo_v, hi_v = z[:, i], z[:, min(i + 1, n - 1)]
        return lo_v + (pos - i) * (hi_v - lo_v)

    # (the library is given the portion as a 32-bit number)
    t = float(torch.tensor(coverage, dtype=torch.float32))
    lo, hi = (quantile(0.5 * (1.0 - t)).float().double(), quantile(0.5 * (1.0 + t)).float().double())
    inside = ((z >= lo[:, None]) & (z < hi[:, None])).double()
    s = _act(z, act)
    cnt = inside.sum(1).clamp_min(1.0)
    mz, ms = (z * inside).sum(1) / cnt, (s * inside).sum(1) / cnt
    dz = (z - mz[:, None]) * inside
    var = (dz * dz).sum(1)
    a = torch.where(var > 0, (dz * (s - ms[:, None])).sum(1) / var.clamp_min(1e-300), torch.zeros_like(var))
    return lo, hi, a, ms - a * mz


def _pre(X, W1, b1):
    z = W1.double() @ X.double().T
    return z if b1 is None else z + b1.double()[:, None]


def _ranges(case, W1, b1, gen):
    X = torch.randn(N_CAL, case["d"], device=DEV, generator=gen).to(W1.dtype)
    z = W1.float() @ X.float().T                                     # neurons x samples
    if b1 is not None:
        z += b1.float()[:, None]
    parts = [_fit(p.double(), case["coverage"], case["act"]) for p in z.split(4096)]
    return tuple(torch.cat([p[i] for p in parts]).float().contiguous() for i in range(4))


def _inputs(case, seed):
    """Weights, ranges and lines (where the case is given them) of every layer, and the tokens (a set for each)."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    layers = []
    for _ in range(case["layers"]):
        W = _weights(case, gen)
        layers.append((W, None if case["kind"] == "calibrate" else _ranges(case, W[0], W[2], gen)))
    x = torch.randn(case["layers"], case["n"], case["d"], device=DEV, generator=gen).to(_TORCH[case["dtype"]])
    return layers, x


def _fold(case, ffn, ranges, max_batch):
    return T.tardis_fold(ffn, *ranges, max_batch=max_batch, sketch_bits=case["sketch_bits"],
                         folded_fp8=case["folded_fp8"])


def prepare(case, seed):
    layers, x = _inputs(case, seed)
    ffns = [T.FFN(W1, W2, b1, b2, case["act"]) for (W1, W2, b1, b2), _ in layers]
    state = {"case": case, "x": list(x) if case["kind"] == "step" else x[0], "ffns": ffns, "ranges": [r for _, r in layers]}
    if case["kind"] in ("forward", "step", "dense"):
        state["layers"] = [_fold(case, f, r, case["n"]) for f, r in zip(ffns, state["ranges"])]
    if case["kind"] == "step":
        for k, layer in enumerate(state["layers"]):                  # the first layer follows the last one
            T.tardis_set_next_layer(layer, state["layers"][(k + 1) % case["layers"]])
    return state


# ------------------------------------------------------------------ one pass
def run(state):
    case, x = state["case"], state["x"]
    if case["kind"] == "forward":
        if case["n"] == 1:
            return T.tardis_ffn_forward(state["layers"][0], x)
        return T.tardis_ffn_forward_batched(state["layers"][0], x)
    if case["kind"] == "step":
        return [T.tardis_ffn_forward_batched(layer, t) for layer, t in zip(state["layers"], x)]
    if case["kind"] == "dense":
        return T.tardis_dense_forward(state["layers"][0], x)
    if case["kind"] == "calibrate":
        return T.tardis_calibrate(state["ffns"][0], x, case["coverage"])
    layer = _fold(case, state["ffns"][0], state["ranges"][0], 1)
    Wp, bp = T.tardis_get_folded(layer)
    Q, tlo, thi = T.tardis_get_predictor_state(layer)
    layer.close()
    return Wp, bp, Q, tlo, thi


def work(case):
    d, h, n, L = case["d"], case["h"], case["n"], case["layers"]
    es = 4 if case["dtype"] == "f32" else 2
    sketch = d * h if case["sketch_bits"] == 8 else d * h // 2 + h * ((d + 31) // 32)
    folded = d * d * (1 if case["folded_fp8"] else es)
    p = 1.0 - case["coverage"]
    if case["kind"] in ("forward", "step"):
        union = h * (1.0 - (1.0 - p) ** n)                           # neurons that some token has repaired
        nbytes = L * (folded + sketch + union * 2 * d * es + 2 * n * d * es)
        flops = L * 2.0 * n * (d * d + d * h + 2 * p * h * d)
    elif case["kind"] == "dense":
        nbytes, flops = 2 * d * h * es + 2 * n * d * es, 4.0 * n * d * h
    elif case["kind"] == "calibrate":
        nbytes, flops = d * h * es + n * d * es + 16 * h, 2.0 * n * d * h
    else:
        nbytes, flops = 2 * d * h * es + folded + d * h + 24 * h, 2.0 * d * d * h
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # measured against exact(): calibration 1.5e-5 (a sample within rounding of a range's end counts on one side or the
    # other), the folded matrix 1.7e-3 (one bf16 rounding), 32-bit layers 4e-7 .. 1e-6, bf16 outputs 2.0e-3 .. 2.4e-3
    if case["kind"] == "calibrate":
        return {"rel": 1e-4}
    if case["kind"] == "fold":
        return {"rel": 4e-3, "max": 0.05}
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 1e-2}


# ------------------------------------------------------------------ the same in 64 bits, with torch alone
def _div(x, v):
    """x / v, rounded once (torch multiplies by the reciprocal of a number on the GPU)."""
    return x / torch.full_like(x, v)


def _codes(W1, bits):
    """Integer codes of the predictor and the unit of each row."""
    W = W1.double()
    if bits == 8:
        s = _div(W.abs().amax(1), 127.0)
        return torch.round(W / s[:, None]).clamp_(-127, 127), s
    h, d = W.shape
    ng = (d + 31) // 32
    g = torch.nn.functional.pad(W.abs(), (0, ng * 32 - d)).view(h, ng, 32).amax(2)
    s = _div(g.amax(1), 7.0 * 15.0)
    m = torch.ceil(g / (7.0 * s[:, None])).clamp_(1, 15).repeat_interleave(32, dim=1)[:, :d]
    return torch.round(W / (m * s[:, None])).clamp_(-7, 7) * m, s


def _bounds(ranges, b1, s):
    b = 0.0 if b1 is None else b1.double()
    return tuple(((r.double() - b) / s).float() for r in ranges[:2])


def _flags(case, W1, b1, ranges, x):
    """tokens x neurons: what the predictor flags."""
    Q, s = _codes(W1, case["sketch_bits"])
    tlo, thi = _bounds(ranges, b1, s)
    m = x.double().abs().amax(1)
    e = torch.floor(torch.log2(m)) - 6
    xq = torch.round(x.double() * torch.exp2(-e)[:, None]).clamp_(-127, 127)
    v = (xq @ Q.T).float() * torch.exp2(e).float()[:, None]          # the sums are whole numbers below 2^53
    return ~((v >= tlo) & (v < thi))


def _forward64(case, W, ranges, x):
    W1, W2, b1, b2 = W
    z = _pre(x, W1, b1).T
    flags = _flags(case, W1, b1, ranges, x)
    a, c = ranges[2].double(), ranges[3].double()
    y = torch.where(flags, _act(z, case["act"]), a * z + c) @ W2.double().T
    if case["folded_fp8"]:                                           # the folded matrix as it is stored
        Wp = W2.double() @ (a[:, None] * W1.double())
        top = torch.ceil(torch.log2(Wp.abs().amax(1) / 448.0))
        scale = torch.exp2(top)[:, None]
        y += x.double() @ ((Wp / scale).float().to(torch.float8_e4m3fn).double() * scale - Wp).T
    return y if b2 is None else y + b2.double()


def exact(case, seed):
    layers, x = _inputs(case, seed)
    (W1, W2, b1, b2), ranges = layers[0]
    if case["kind"] == "step":
        return [_forward64(case, W, r, t) for (W, r), t in zip(layers, x)]
    x = x[0]
    if case["kind"] == "forward":
        return _forward64(case, layers[0][0], ranges, x)
    if case["kind"] == "dense":
        y = _act(_pre(x, W1, b1), case["act"]).T @ W2.double().T
        return y if b2 is None else y + b2.double()
    if case["kind"] == "calibrate":
        parts = [_fit(_pre(x, W1[i:i + 2048], None if b1 is None else b1[i:i + 2048]), case["coverage"], case["act"])
                 for i in range(0, case["h"], 2048)]
        return tuple(torch.cat([p[i] for p in parts]) for i in range(4))
    a, c = ranges[2].double(), ranges[3].double()
    Wp = W2.double() @ (a[:, None] * W1.double())
    bp = W2.double() @ (c if b1 is None else c + a * b1.double())
    Q, s = _codes(W1, case["sketch_bits"])
    return (Wp, bp if b2 is None else bp + b2.double(), None, *_bounds(ranges, b1, s))
