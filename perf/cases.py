"""What the speed of this framework is measured on: one data-parallel step's hot path over the range of gradients that
a training run hands it, through the public entry points of ``paper_2511_10333_amd``.

A case is one pass of a user's step in the steady state of a run (unless it says otherwise): the entropy estimate of the
gradients' sample, then compress and decompress of every tensor with the error feedback of the step before, all on the
current stream; or the entropy estimate alone.  The forms are the ones the library offers: the single-tensor calls, the
batched calls with the residual stored or deferred, and the two phases between which a data-parallel job exchanges P.

Fields of a case: ``shapes`` ("MxN" a matrix, "N" a vector; a tensor whose factors would not be smaller is sent as it
stands), ``dtype``, ``rank``, ``calls`` ("single", "batch", "exchange", "estimate"), ``residual`` ("stored", "deferred",
"zero": the first step), ``power_iters``, and the estimate's ``stride``, ``bins``.
"""
import math

import torch

import paper_2511_10333_amd as edgc
from paper_2511_10333_amd.binding import ENTROPY_RESULT_BYTES

CHUNK = 64          # elements per sampled chunk
EST_SEED = 7        # of the sampler


# ---------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------
def _text(shapes):
    return ",".join("x".join(str(d) for d in s) for s in shapes)


def _block(hidden, shards=1):
    """The four 2-D gradients of a GPT block (of one of `shards` tensor-parallel ranks)."""
    h, k = hidden, shards
    return [(h, 3 * h // k), (h // k, h), (h, 4 * h // k), (4 * h // k, h)]


def _vectors(hidden):
    """Its norm weights and biases: these are sent as they stand."""
    h = hidden
    return [(h,), (h,), (3 * h,), (h,), (h,), (h,), (4 * h,), (h,)]


def _step(name, shapes, dtype, rank, calls, residual, power_iters=1, stride=100, bins=1024):
    c = {"shapes": _text(shapes), "dtype": dtype, "rank": rank, "calls": calls, "residual": residual,
         "power_iters": power_iters, "stride": stride, "bins": bins}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one square layer through the single-tensor calls; launches and latency
        _step("matrix_1024_f32_r4", [(1024, 1024)], "f32", 4, "single", "stored", bins=256),
        # a stage of two small blocks with everything a model has: 8 matrices and 16 norm and bias vectors
        _step("stage_h768_bf16_r16", 2 * (_block(768) + _vectors(768)), "bf16", 16, "batch", "deferred"),
        # one GPT block at hidden 2048, fp32, low rank: the ordinary single-GPU layer
        _step("block_h2048_f32_r16", _block(2048), "f32", 16, "batch", "deferred"),
        # one GPT block at hidden 4096, fp32, with the residual itself stored (what checkpoints hold)
        _step("block_h4096_f32_r64_stored", _block(4096), "f32", 64, "batch", "stored"),
        # the largest layers, bf16 gradients, highest rank
        _step("block_h5120_bf16_r128", _block(5120), "bf16", 128, "batch", "deferred"),
        # one of four tensor-parallel ranks of a hidden-3584 block, the two phases of a data-parallel exchange
        _step("shard_h3584_bf16_r64_exchange", _block(3584, 4), "bf16", 64, "exchange", "deferred"),
        # an embedding table: rows that no tile divides
        _step("embedding_50257x1024_bf16_r32", [(50257, 1024)], "bf16", 32, "single", "stored"),
        # odd sizes on both sides and an odd rank: nothing is aligned
        _step("odd_f32_r13", [(2047, 3001), (1001, 4099), (5003, 777)], "f32", 13, "batch", "deferred"),
        # the first step after a rank decision: no residual yet, two power iterations from a random start
        _step("first_4096x4096_f32_r32_pi2", [(4096, 4096)], "f32", 32, "single", "zero", power_iters=2),
        # the entropy of a stage's four gradient buffers, 1 % sample (every step of a run does this)
        _step("entropy_4x_f32_1pct", _block(4096), "f32", 1, "estimate", "none", bins=4096),
        # the entropy of a whole flat bf16 buffer
        _step("entropy_bf16_all", [(1 << 27,)], "bf16", 1, "estimate", "none", stride=1, bins=4096),
        # a 10 % sample of a flat fp32 buffer of odd length on many bins
        _step("entropy_f32_10pct_65536", [(100000007,)], "f32", 1, "estimate", "none", stride=10, bins=65536),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _rank_for(rng, shapes):
    """Any rank at which the factors of the smallest of the matrices are at most a quarter of its size."""
    m, n = min((s for s in shapes if len(s) == 2), key=lambda s: s[0] * s[1])
    return _log_int(rng, 1, max(1, min(128, m * n // (4 * (m + n)))))


def draw(rng):
    kind = rng.choice(["single", "single", "batch", "batch", "batch", "odd", "exchange", "estimate"])
    dtype = rng.choice(["f32", "bf16"])
    stride = rng.choice([10, 100, 1000])
    bins = rng.choice([256, 1024, 4096])
    if kind == "estimate":
        parts = rng.choice([1, 1, 4, 12])
        shapes = [(_log_int(rng, 1e6, 1.5e8) // parts,) for _ in range(parts)]
        return _step(None, shapes, dtype, 1, "estimate", "none", stride=rng.choice([1, 10, 100, 1000]),
                     bins=rng.choice([256, 1024, 4096, 65536]))
    if kind == "single":
        shapes = [(_log_int(rng, 256, 16384), _log_int(rng, 256, 16384))]
        if rng.random() < 0.5:
            shapes = [tuple((d + 63) // 64 * 64 for d in shapes[0])]
        residual = rng.choice(["stored", "stored", "zero"])
        return _step(None, shapes, dtype, _rank_for(rng, shapes), "single", residual,
                     power_iters=2 if residual == "zero" and rng.random() < 0.5 else 1, stride=stride, bins=bins)
    if kind == "odd":
        shapes = [(_log_int(rng, 100, 6000), _log_int(rng, 100, 6000)) for _ in range(rng.randint(1, 5))]
        return _step(None, shapes, dtype, _rank_for(rng, shapes), "batch", rng.choice(["stored", "deferred"]),
                     stride=min(stride, 100), bins=bins)      # (the smallest still has a chunk in every residue class)
    hidden = _log_int(rng, 512, 4600)
    step = rng.choice([8, 64, 128])
    hidden = (hidden + step - 1) // step * step
    if kind == "exchange":
        shapes = _block(hidden, rng.choice([1, 2, 4]))
        return _step(None, shapes, dtype, _rank_for(rng, shapes), "exchange", rng.choice(["stored", "deferred"]),
                     stride=stride, bins=bins)
    shapes = _block(hidden) + (_vectors(hidden) if rng.random() < 0.5 else [])
    if hidden < 1500 and rng.random() < 0.5:
        shapes = 2 * shapes
    return _step(None, shapes, dtype, _rank_for(rng, shapes), "batch", rng.choice(["stored", "deferred", "deferred"]),
                 stride=stride, bins=bins)


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------
def _shapes(case):
    return [tuple(int(d) for d in s.split("x")) for s in case["shapes"].split(",")]


def _sent_as_it_stands(s, r):
    return len(s) == 1 or min(s) == 1 or (s[0] + s[1]) * r >= s[0] * s[1]


def _tdtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _laplace(n, g):
    """Laplace(0, 1e-3) with one value in a thousand at 100 times the scale: the entries of a gradient."""
    x = torch.rand(n, generator=g, device="cuda").sub_(0.5)
    x = -torch.sign(x) * torch.log1p(-2.0 * x.abs().clamp_(max=0.4999999)) * 1e-3
    return torch.where(torch.rand(n, generator=g, device="cuda") < 1e-3, 100.0 * x, x)


def _inputs(case, seed):
    """Per tensor: the gradient and, where it is compressed, what the step before left: the residual buffer (E, or D
    where the residual is deferred), Q (columns up to the rank) and, deferred, P.  A gradient is a decaying spectrum
    plus noise; the step before found the leading part of the same spectrum, so its factors are U and V * s."""
    g = torch.Generator(device="cuda").manual_seed(seed * 1000003 + 17)
    r, out = case["rank"], []
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda")
    for s in _shapes(case):
        if case["calls"] == "estimate" or _sent_as_it_stands(s, r):
            x = _laplace(s[0] * (s[1] if len(s) == 2 else 1), g)
            out.append({"G": x.view(*s).to(_tdtype(case))})
            continue
        m, n = s
        k = min(m, n, 4 * r + 32)
        decay = 0.97 if r >= 64 else 0.95
        sv = decay ** torch.arange(k, device="cuda", dtype=torch.float32)
        U, V = randn(m, k).div_(math.sqrt(m)), randn(n, k).div_(math.sqrt(n))
        low = (U * sv) @ V.t()
        t = {"G": (low + 1e-4 * randn(m, n)).to(_tdtype(case))}
        if case["residual"] == "zero":
            t["Q"] = randn(n, r)
        else:
            # error feedback carries what the rank did not: the rest of the spectrum and the noise
            t["Q"] = (V[:, :r] * sv[:r]).contiguous()
            t["P"] = U[:, :r].contiguous()
            if case["residual"] == "deferred":
                t["R"] = low + 1.5e-4 * randn(m, n)
            else:
                t["R"] = (U[:, r:] * sv[r:]) @ V[:, r:].t() + 1.5e-4 * randn(m, n)
        out.append(t)
    return out


def prepare(case, seed):
    r = case["rank"]
    ldf = (r + 3) // 4 * 4
    tensors = []
    for t in _inputs(case, seed):
        if "Q" not in t:
            tensors.append(edgc.Tensor(t["G"], torch.empty_like(t["G"])))
            continue
        m, n = t["G"].shape
        Q, P = torch.zeros((n, ldf), device="cuda"), torch.zeros((m, ldf), device="cuda")
        Q[:, :r] = t["Q"]
        if "P" in t:
            P[:, :r] = t["P"]
        E = t["R"] if "R" in t else torch.zeros((m, n), device="cuda")
        tensors.append(edgc.Tensor(t["G"], torch.empty_like(t["G"]), E, Q, P, case["residual"] == "zero"))
    single = case["calls"] == "single"
    rows, cols = (tensors[0].grad.shape if single else (64, 64))
    # a program sizes its context for the largest rank that the rule may decide on, not for the rank of the moment
    ctx = edgc.Context(0, max_bins=case["bins"], max_rank=128, max_rows=rows, max_cols=cols)
    state = {"case": case, "ctx": ctx, "tensors": tensors, "flats": [t.grad.view(-1) for t in tensors],
             "result": torch.empty(ENTROPY_RESULT_BYTES, dtype=torch.uint8, pin_memory=True),
             "counts": torch.zeros(case["bins"], dtype=torch.int64, device="cuda"), "step": seed % 1000}
    if case["calls"] in ("batch", "exchange"):
        ctx.reserve_batch([tuple(t.grad.shape) if t.grad.dim() == 2 else (1, t.grad.numel()) for t in tensors])
        state["batch"] = edgc.PreparedBatch(tensors)
    return state


# ---------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------
def run(state):
    case, ctx, ts = state["case"], state["ctx"], state["tensors"]
    flats = state["flats"] if len(state["flats"]) > 1 else state["flats"][0]
    ctx.entropy_estimate_async(flats, case["stride"], CHUNK, EST_SEED, state["step"], case["bins"], state["result"],
                               counts_out=state["counts"])
    out = {"entropy": state["result"].view(torch.float64)[:2], "range": state["result"].view(torch.float32)[4:6],
           "n_sampled": state["result"].view(torch.int64)[3:4], "counts": state["counts"]}
    r, deferred = case["rank"], case["residual"] == "deferred"
    if case["calls"] == "single":
        t = ts[0]
        ctx.compress(t.grad, t.residual, t.residual_is_zero, t.Q, t.P, r, power_iters=case["power_iters"])
        ctx.decompress(t.P, t.Q, r, t.residual, t.grad_out)
    elif case["calls"] == "batch":
        ctx.compress_batch(state["batch"], r, power_iters=case["power_iters"], deferred=deferred)
        ctx.decompress_batch(state["batch"], r, deferred=deferred)
    elif case["calls"] == "exchange":       # the all-reduces of P and of Q stand between these calls
        ctx.compress_p_batch(state["batch"], r, deferred=deferred)
        ctx.compress_q_batch(state["batch"], r)
        ctx.decompress_batch(state["batch"], r, deferred=deferred)
    if case["calls"] != "estimate":
        for i, t in enumerate(ts):
            out["t%d" % i] = (t.grad_out if t.Q is None else
                              {"out": t.grad_out, "residual": t.residual, "P": t.P[:, :r], "Q": t.Q[:, :r]})
    return out


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------
def _sampled(n, stride, slot):
    """Elements the sampler takes of a buffer of n: every stride-th chunk from `slot` on."""
    if stride == 1:
        return n
    chunks = -(-n // CHUNK)
    if slot >= chunks:
        return 0
    k = -(-(chunks - slot) // stride)
    last = slot + (k - 1) * stride
    return (k - 1) * CHUNK + min(CHUNK, n - last * CHUNK)


def work(case):
    b = 2 if case["dtype"] == "bf16" else 4
    r, n_bytes, flops = case["rank"], 0, 0
    for s in _shapes(case):
        numel = s[0] * (s[1] if len(s) == 2 else 1)
        if case["calls"] == "estimate":
            n_bytes += b * _sampled(numel, case["stride"], 0)
            continue
        if _sent_as_it_stands(s, r):
            n_bytes += 2 * b * numel
            continue
        m, n = s
        # the sample is part of the gradient, which is read anyway
        n_bytes += numel * (2 * b + (4 if case["residual"] == "zero" else 8))
        n_bytes += 4 * r * (2 * n + m + (m if case["residual"] == "deferred" else 0))
        products = 2 * case["power_iters"] + 1 + (1 if case["residual"] == "deferred" else 0)
        flops += 2 * numel * r * products
    return {"bytes": n_bytes + 8 * case["bins"], "flops": flops}


def tolerance(case):
    if case["calls"] == "estimate":
        return {"rel": 1e-9, "max": 1e-9, "differ": 0.0}
    # against 64 bits the listed and some drawn cases show up to 2e-5 (operands in two bf16 planes, 17 bits) and, with
    # bf16 gradients, 6e-3 (operands and the reconstruction rounded to bf16)
    return {"rel": 1e-4} if case["dtype"] == "f32" else {"rel": 2.4e-2}


# ---------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------
def _mix64(seed, ctr):
    """The published splitmix64 output function: the sampler's slot is drawn from it."""
    mask = (1 << 64) - 1
    z = (seed + 0x9E3779B97F4A7C15 * (ctr + 1)) & mask
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & mask
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & mask
    return z ^ (z >> 31)


def _exact_estimate(case, tensors, step):
    stride, bins = case["stride"], case["bins"]
    slot = _mix64(EST_SEED, step) % stride
    parts = []
    for t in tensors:
        x = t["G"].reshape(-1)
        if stride > 1:
            chunks = torch.arange(slot, max(slot, -(-x.numel() // CHUNK)), stride, device=x.device)
            at = (chunks[:, None] * CHUNK + torch.arange(CHUNK, device=x.device)[None, :]).reshape(-1)
            x = x[at[at < x.numel()]]
        parts.append(x.float())
    x = torch.cat(parts)
    lo, hi = x.min(), x.max()
    width = (hi - lo).cpu()
    scale = torch.tensor(float(bins), dtype=torch.float32) / width      # one correctly rounded division
    # the definition of a bin is in 32 bits, each operation rounded by itself
    at = ((x - lo) * scale.to(x.device)).long().clamp_(0, bins - 1)
    counts = torch.bincount(at, minlength=bins)
    p = counts[counts > 0].double() / x.numel()
    bits = float(-(p * torch.log2(p)).sum())
    diff = bits * math.log(2.0) + math.log(float(width.double()) / bins)
    return {"entropy": torch.tensor([bits, diff], dtype=torch.float64), "range": torch.stack([lo, hi]).cpu(),
            "n_sampled": torch.tensor([x.numel()], dtype=torch.int64), "counts": counts}


def exact(case, seed):
    tensors = _inputs(case, seed)
    out = _exact_estimate(case, tensors, seed % 1000)
    if case["calls"] == "estimate":
        return out
    as_sent = lambda x: x.to(_tdtype(case)).double()      # the residual is taken against what was sent
    for i, t in enumerate(tensors):
        if "Q" not in t:
            out["t%d" % i] = t["G"]
            continue
        Q = t["Q"].double()
        D = t["G"].double()
        if "R" in t:
            D = D + t["R"].double()
        if case["residual"] == "deferred":
            D -= as_sent(t["P"].double() @ t["Q"].double().t())
        for _ in range(case["power_iters"]):
            P, R = torch.linalg.qr(D @ Q)
            P = P * torch.sign(torch.diagonal(R))          # positive diagonal: the factor is unique
            Q = D.t() @ P
        M = P @ Q.t()
        if case["residual"] != "deferred":
            D = D - as_sent(M)
        out["t%d" % i] = {"out": M, "residual": D, "P": P, "Q": Q}
    return out
