"""The work that is measured: what a program that uses this library has it do.

Each case is one call (or, for a training step, the pair of calls) of the public binding
`paper_2506_05233_amd.libmesa` on inputs that live on the GPU: the sequence forward (prefill and
evaluation), the states-only prefill, the decode step, the training step (forward and backward) and the
layer's two ends around them.  Sizes are those of the library's own workloads (the small fp32 layers at
d 64, the 1B-shaped layer at d 128, the long context, batched decode) and ragged ones between them.
Values follow the layer's front end: unit-norm queries and keys, Gaussian values, sigmoid gates whose
logits have mean 3 to 5, a regulariser in [0.25, 1].
"""
import math

import torch

from paper_2506_05233_amd import libmesa

PRECISION = {"auto": libmesa.MESA_PREC_AUTO, "single": libmesa.MESA_PREC_BF16}
RING = 8  # tokens that a decode case feeds in turn


def _seq(name, batch, heads, tokens, d_k, d_v, dtype, steps, mu, chunk=64, precision="auto", eps=0.0):
    return {"name": name, "kind": "forward", "batch": batch, "heads": heads, "tokens": tokens, "d_k": d_k, "d_v": d_v,
            "dtype": dtype, "steps": steps, "mu": mu, "chunk": chunk, "precision": precision, "eps": eps}


def _train(name, batch, heads, tokens, d_k, d_v, dtype, steps, mu):
    return dict(_seq(name, batch, heads, tokens, d_k, d_v, dtype, steps, mu), kind="train")


def _prefill(name, batch, heads, tokens, d_k, d_v, dtype, mu):
    return {"name": name, "kind": "prefill", "batch": batch, "heads": heads, "tokens": tokens, "d_k": d_k, "d_v": d_v,
            "dtype": dtype, "mu": mu}


def _decode(name, batch, heads, d_k, d_v, dtype, steps, packed, mu=4.0):
    return {"name": name, "kind": "decode", "batch": batch, "heads": heads, "d_k": d_k, "d_v": d_v, "dtype": dtype,
            "steps": steps, "packed": packed, "mu": mu}


def _ends(name, batch, heads, tokens, d_k, d_v, dtype, conv_v):
    return {"name": name, "kind": "ends", "batch": batch, "heads": heads, "tokens": tokens, "d_k": d_k, "d_v": d_v,
            "dtype": dtype, "conv_v": conv_v}


def listed():
    return [
        # one short fp32 sequence with two heads: an interactive or test-sized call, all latency
        _seq("forward_tiny_f32", 1, 2, 256, 64, 64, "f32", 10, 3.0),
        # a small fp32 model's layer
        _seq("forward_small_f32", 4, 8, 2048, 64, 64, "f32", 15, 3.0),
        # the 1B-shaped layer with the default precision for bf16 inputs
        _seq("forward_1b_bf16", 8, 16, 2048, 128, 128, "bf16", 15, 4.0),
        # the same in the single-pass mode, which trades accuracy for speed
        _seq("forward_1b_bf16_single", 8, 16, 2048, 128, 128, "bf16", 15, 4.0, precision="single"),
        # one long document: few sequences, gates near one
        _seq("forward_long_bf16", 1, 16, 16384, 128, 128, "bf16", 20, 5.0),
        # evaluation of a few prompts with the solver's relative tolerance; a ragged length, narrower values
        _seq("forward_tol_ragged_bf16", 3, 8, 1000, 128, 64, "bf16", 30, 4.0, eps=1e-4),
        # prompts to recurrent states before decoding, ragged length
        _prefill("prefill_ragged_bf16", 4, 16, 4001, 128, 128, "bf16", 4.0),
        # one decode step of a large serving batch
        _decode("decode_batch_bf16", 256, 16, 128, 128, "bf16", 15, False),
        # one decode step of three users, on the packed state
        _decode("decode_few_packed_bf16", 3, 16, 128, 128, "bf16", 15, True),
        # a training step of the 1B-shaped layer: forward with q*, then the gradients
        _train("train_1b_bf16", 8, 16, 2048, 128, 128, "bf16", 15, 4.0),
        # a training step of a small fp32 layer at a ragged length
        _train("train_ragged_f32", 2, 4, 777, 64, 64, "f32", 10, 3.0),
        # the layer's ends at the 1B shape: projections to inputs, outputs through the norm
        _ends("ends_1b_bf16", 8, 16, 2048, 128, 128, "bf16", False),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "prefill", "decode", "decode", "train", "ends"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    d_k = rng.choice([64, 128])
    d_v = rng.choice([d_k, d_k, 64, 128])
    heads = rng.choice([1, 2, 4, 6, 8, 12, 16])
    mu = rng.choice([3.0, 4.0, 5.0])
    if kind == "decode":
        c = _decode("", _spread(rng, 1, 256), heads, d_k, d_v, dtype, rng.randint(5, 20), rng.random() < 0.4, mu)
    else:
        # fp32 products at d 128 cost several times the bf16 ones: fewer tokens keep them under the largest
        most = 262144 if dtype == "bf16" or kind in ("prefill", "ends") else 32768
        if kind == "train" and dtype == "f32":
            most = 16384
        rows = _spread(rng, 256, most)  # tokens over all sequences and heads
        heads = min(heads, max(1, rows // 64))
        tokens = _spread(rng, 48, min(16384, max(48, rows // heads)))
        batch = max(1, rows // (heads * tokens))
        if kind == "forward":
            single = dtype == "bf16" and rng.random() < 0.3
            tol = rng.random() < 0.25
            chunk = 64 if dtype == "bf16" or rng.random() < 0.8 else 32
            c = _seq("", batch, heads, tokens, d_k, d_v, dtype, 30 if tol else rng.randint(5, 20), mu, chunk,
                     "single" if single else "auto", 1e-4 if tol else 0.0)
            if tol and batch * heads * tokens > most // 2:
                c["steps"] = 15
        elif kind == "train":
            c = _train("", batch, heads, tokens, d_k, d_v, dtype, rng.randint(5, 15), mu)
        elif kind == "prefill":
            c = _prefill("", batch, heads, tokens, d_k, d_v, dtype, mu)
        else:
            c = _ends("", batch, heads, tokens, d_k, d_v, dtype, rng.random() < 0.5)
    del c["name"]
    return c


def _device():
    return torch.device("cuda")


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _sequence_inputs(case, seed):
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(seed)
    b, h, t, dk, dv = case["batch"], case["heads"], case["tokens"], case["d_k"], case["d_v"]

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev)

    def unit(*shape):
        x = normal(*shape)
        return x / x.norm(dim=-1, keepdim=True)

    dt = _dtype(case)
    return {"q": unit(b, h, t, dk).to(dt), "k": unit(b, h, t, dk).to(dt), "v": normal(b, h, t, dv).to(dt),
            "gamma": torch.sigmoid(normal(b, h, t) + case["mu"]), "beta": torch.sigmoid(normal(b, h, t)),
            "lam": torch.rand((h, dk), generator=g, device=dev) * 0.75 + 0.25, "dout": normal(b, h, t, dv)}


def _decode_inputs(case, seed):
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(seed)
    n, h, dk, dv = case["batch"], case["heads"], case["d_k"], case["d_v"]

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev)

    def unit(*shape):
        x = normal(*shape)
        return x / x.norm(dim=-1, keepdim=True)

    # the states after a prompt: gated sums over keys whose weights have decayed
    m = 2 * dk
    w = torch.exp(-torch.rand((n, h, m, 1), generator=g, device=dev) * 4.0)
    k, v = unit(n, h, m, dk), normal(n, h, m, dv)
    state_h = torch.matmul((w * k).transpose(-1, -2).contiguous(), k)
    state_h = 0.5 * (state_h + state_h.transpose(-1, -2))
    state_g = torch.matmul((w * v).transpose(-1, -2).contiguous(), k)
    dt = _dtype(case)
    ring = [{"q": unit(n, h, dk).to(dt), "k": unit(n, h, dk).to(dt), "v": normal(n, h, dv).to(dt),
             "gamma": torch.sigmoid(normal(n, h) + case["mu"]), "beta": torch.sigmoid(normal(n, h))}
            for _ in range(RING)]
    lam = torch.rand((h, dk), generator=g, device=dev) * 0.75 + 0.25
    return state_h.contiguous(), state_g.contiguous(), ring, lam


def _ends_inputs(case, seed):
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(seed)
    b, h, t, dk, dv = case["batch"], case["heads"], case["tokens"], case["d_k"], case["d_v"]

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev)

    dt = _dtype(case)
    return {"qp": normal(b, t, h, dk).to(dt), "kp": normal(b, t, h, dk).to(dt), "vp": normal(b, t, h, dv).to(dt),
            "conv_q": 0.5 * normal(h * dk, 4), "conv_k": 0.5 * normal(h * dk, 4),
            "conv_v": 0.5 * normal(h * dv, 4) if case["conv_v"] else None,
            "a_gamma": normal(b, t, h) + 4.0, "a_beta": normal(b, t, h), "theta": normal(h, dk),
            "o": normal(b, h, t, dv), "weight": 1.0 + 0.1 * normal(h, dv)}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "decode":
        state_h, state_g, ring, lam = _decode_inputs(case, seed)
        if case["packed"]:
            state_h = libmesa.pack_state(state_h)
        return {"case": case, "H": state_h, "G": state_g, "ring": ring, "lam": lam, "at": 0,
                "out": torch.empty((case["batch"], case["heads"], case["d_v"]), device=_device())}
    if kind == "ends":
        return dict(_ends_inputs(case, seed), case=case)
    s = dict(_sequence_inputs(case, seed), case=case)
    b, h, t, dk, dv = case["batch"], case["heads"], case["tokens"], case["d_k"], case["d_v"]
    need = libmesa.forward_workspace_bytes(b, h, t, dk, dv, case.get("chunk", 64))
    s["workspace"] = torch.empty(max(need, 16), dtype=torch.uint8, device=_device())
    if kind == "train":
        need = libmesa.backward_workspace_bytes(b, h, t, dk, dv)
        s["backward_workspace"] = torch.empty(need, dtype=torch.uint8, device=_device())
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "forward":
        tol = {"eps": case["eps"], "want_steps": True} if case["eps"] else {}
        return libmesa.forward(s["q"], s["k"], s["v"], s["gamma"], s["beta"], s["lam"], case["steps"], case["chunk"],
                               PRECISION[case["precision"]], workspace=s["workspace"], **tol)
    if kind == "train":
        f = libmesa.forward(s["q"], s["k"], s["v"], s["gamma"], s["beta"], s["lam"], case["steps"], case["chunk"],
                            want_qstar=True, workspace=s["workspace"])
        g = libmesa.backward(s["k"], s["v"], s["gamma"], s["beta"], s["lam"], f["qstar"], s["dout"], case["steps"],
                             workspace=s["backward_workspace"])
        return dict(g, out=f["out"])
    if kind == "prefill":
        return libmesa.prefill_states(s["k"], s["v"], s["gamma"], s["beta"], workspace=s["workspace"])
    if kind == "decode":
        x = s["ring"][s["at"] % RING]
        s["at"] += 1
        out = libmesa.decode_step(s["H"], s["G"], x["q"], x["k"], x["v"], x["gamma"], x["beta"], s["lam"], case["steps"],
                                  out=s["out"], packed=case["packed"])
        return {"out": out, "G": s["G"], "H": s["H"]}
    f = libmesa.frontend(s["qp"], s["kp"], s["vp"], s["conv_q"], s["conv_k"], s["conv_v"], s["a_gamma"], s["a_beta"],
                         s["theta"])
    return dict(f, y=libmesa.output_norm(s["o"], s["weight"], out_dtype=_dtype(case)))


def work(case):
    """Inputs read once and results written once, and the flops of the sums as the method states them (the
    causal half of the products inside a chunk; one product for the first residual and one a step)."""
    kind, b, h, dk, dv = case["kind"], case["batch"], case["heads"], case["d_k"], case["d_v"]
    es = 2 if case["dtype"] == "bf16" else 4
    if kind == "decode":
        rows_h = dk // 2 + 1 if case["packed"] else dk
        pairs = b * h
        return {"bytes": pairs * (8 * (rows_h + dv) * dk + es * (2 * dk + dv) + 8 + 4 * dv) + 4 * h * dk,
                "flops": pairs * (3 * dk * dk + 5 * dv * dk + (case["steps"] + 1) * 2 * dk * dk)}
    n = b * h * case["tokens"]
    if kind == "ends":
        return {"bytes": n * (2 * es * (2 * dk + dv) + 16 + (4 + es) * dv),
                "flops": n * (2 * (8 + 8) * dk + (8 + 8) * dv * case["conv_v"] + 4 * dv)}
    c = case.get("chunk", 64)
    scan = 2 * (dk + dv) * dk
    if kind == "prefill":
        return {"bytes": n * (es * (dk + dv) + 8) + b * h * 4 * (dk + dv) * dk, "flops": n * scan}
    solve = (case["steps"] + 1) * (2 * dk * dk + 2 * (c + 1) * dk)
    if case["eps"]:
        solve = solve // 3  # the tolerance ends a solve after about a third of the steps allowed
    read = 2 * dv * dk + (c + 1) * (dk + dv)
    size = {"bytes": n * (es * (2 * dk + dv) + 8 + 4 * dv) + 4 * h * dk, "flops": n * (scan + solve + read)}
    if kind == "train":
        # the right-hand side (a read-out), the second solve, the adjoint scan, and the products of the gradients
        size["bytes"] += n * (4 * dv + 4 * (2 * dk + dv) + 8) + 4 * h * dk
        size["flops"] += n * (read + solve + 2 * (dk + dv) * dk + 10 * dk * dv + 2 * (c + 1) * (2 * dk + dv))
    elif case["eps"]:
        size["bytes"] += 4 * n
    return size


def tolerance(case):
    # about four times the error of a pass against the same sums in 64 bits
    kind = case["kind"]
    if kind == "ends":
        return {"rel": 7e-3, "max": 0.05} if case["dtype"] == "bf16" else {"rel": 5e-7}
    if kind == "prefill":
        return {"rel": 1e-5}
    if kind == "decode":
        return {"rel": 1.5e-6}
    if kind == "train":
        return {"rel": 1.7e-2} if case["dtype"] == "bf16" else {"rel": 3e-6}
    if case["precision"] == "single":
        return {"rel": 2e-2, "differ": 0.01}
    if case["eps"]:
        return {"rel": 4e-5, "differ": 0.01}  # a residual at the limit may end a solve one step apart
    return {"rel": 3e-5} if case["dtype"] == "bf16" else {"rel": 2e-6}


def _states(x0, gamma, add):
    """x_t = gamma_t x_{t-1} + add_t over the block's tokens, in place on add [N, T, ...]."""
    for t in range(add.shape[1]):
        torch.addcmul(add[:, t], gamma[:, t, None, None], add[:, t - 1] if t else x0, out=add[:, t])
    return add


def _cg(a, lam, q, steps, eps):
    """Conjugate gradients on (a + diag(lam)) x = q from the Jacobi start, [N, T, d] columns; x and the steps used."""
    def times(p):
        return (a * p[..., None, :]).sum(-1) + lam * p

    x = q / (a.diagonal(dim1=-2, dim2=-1) + lam)
    r = q - times(x)
    p = r.clone()
    d = (r * r).sum(-1, keepdim=True)
    first, used = d, torch.zeros_like(d, dtype=torch.int32)
    going = d > 0
    for _ in range(steps):
        w = times(p)
        pw = (p * w).sum(-1, keepdim=True)
        going = going & (pw > 0)
        al = torch.where(going, d / pw, torch.zeros_like(d))
        x = x + al * p
        r = r - al * w
        used += going
        n = (r * r).sum(-1, keepdim=True)
        p = torch.where(going, r + n / d * p, p)
        d = torch.where(going, n, d)
        going = going & (n > eps * eps * first)
    return x, used[..., 0]


def _blocks(n, t, elems):
    """Token ranges whose [n, range, elems] states in 64 bits stay near a gigabyte."""
    size = max(1, min(t, int(1e9 // (8 * n * elems))))
    return [(lo, min(t, lo + size)) for lo in range(0, t, size)]


def _flat(x):
    return x.reshape(-1, *x.shape[2:]).double()


def exact(case, seed):
    kind = case["kind"]
    if kind == "ends":
        return _exact_ends(case, seed)
    if kind == "decode":
        return _exact_decode(case, seed)
    s = _sequence_inputs(case, seed)
    b, h, t, dk, dv = case["batch"], case["heads"], case["tokens"], case["d_k"], case["d_v"]
    n = b * h
    k, v, gamma, beta = (_flat(s[x]) for x in ("k", "v", "gamma", "beta"))
    bk = beta[..., None] * k
    ranges = _blocks(n, t, dk * max(dk, dv))
    hs = torch.zeros((n, dk, dk), dtype=torch.float64, device=k.device)
    gs = torch.zeros((n, dv, dk), dtype=torch.float64, device=k.device)

    def block(lo, hi, h0, g0):
        hb = _states(h0, gamma[:, lo:hi], bk[:, lo:hi, :, None] * k[:, lo:hi, None, :])
        gb = _states(g0, gamma[:, lo:hi], v[:, lo:hi, :, None] * bk[:, lo:hi, None, :])
        return hb, gb

    starts, out, qstar, used, right = [], [], [], [], []
    if kind != "prefill":
        q = _flat(s["q"])
        lam = s["lam"].double().repeat(b, 1)[:, None, :]
        dout = _flat(s["dout"])
    for lo, hi in ranges:
        starts.append((hs, gs))
        hb, gb = block(lo, hi, hs, gs)
        hs, gs = hb[:, -1].clone(), gb[:, -1].clone()
        if kind == "prefill":
            continue
        x, c = _cg(hb, lam, q[:, lo:hi], case["steps"], case["eps"])
        out.append((gb * x[..., None, :]).sum(-1))
        qstar.append(x)
        used.append(c)
        if kind == "train":
            u = (gb * dout[:, lo:hi, :, None]).sum(-2)
            right.append(_cg(hb, lam, u, case["steps"], 0.0)[0])
        del hb, gb
    if kind == "prefill":
        return hs.reshape(b, h, dk, dk), gs.reshape(b, h, dv, dk)
    out = torch.cat(out, 1).reshape(b, h, t, dv)
    if kind == "forward":
        return {"out": out, "steps": None} if case["eps"] else out
    # the adjoints of the two states, walked backwards
    qs, es = torch.cat(qstar, 1), torch.cat(right, 1)
    grads = {"dk": torch.empty_like(k), "dv": torch.empty_like(v), "dgamma": torch.empty_like(gamma),
             "dbeta": torch.empty_like(beta)}
    ah, ag = torch.zeros_like(hs), torch.zeros_like(gs)
    for (lo, hi), (h0, g0) in reversed(list(zip(ranges, starts))):
        hb, gb = block(lo, hi, h0, g0)
        for i in reversed(range(lo, hi)):
            ah = ah - es[:, i, :, None] * qs[:, i, None, :]
            ag = ag + dout[:, i, :, None] * qs[:, i, None, :]
            hp, gp = (hb[:, i - lo - 1], gb[:, i - lo - 1]) if i > lo else (h0, g0)
            grads["dgamma"][:, i] = (ah * hp).sum((-1, -2)) + (ag * gp).sum((-1, -2))
            gk = (ag * k[:, i, None, :]).sum(-1)
            gv = (ag * v[:, i, :, None]).sum(-2)
            hk = (ah * k[:, i, None, :]).sum(-1)
            kh = (ah * k[:, i, :, None]).sum(-2)
            grads["dv"][:, i] = beta[:, i, None] * gk
            grads["dk"][:, i] = beta[:, i, None] * (gv + hk + kh)
            grads["dbeta"][:, i] = (v[:, i] * gk).sum(-1) + (k[:, i] * hk).sum(-1)
            ah, ag = gamma[:, i, None, None] * ah, gamma[:, i, None, None] * ag
        del hb, gb
    res = {name: x.reshape(b, h, *x.shape[1:]) for name, x in grads.items()}
    return dict(res, dq=es.reshape(b, h, t, dk), dlam=-(qs * es).reshape(b, h, t, dk).sum((0, 2)), out=out)


def _exact_decode(case, seed):
    state_h, state_g, ring, lam = _decode_inputs(case, seed)
    x = {name: y.double() for name, y in ring[0].items()}
    g, be = x["gamma"][..., None, None], x["beta"][..., None, None]
    hs = g * state_h.double() + be * x["k"][..., :, None] * x["k"][..., None, :]
    gs = g * state_g.double() + be * x["v"][..., :, None] * x["k"][..., None, :]
    qs, _ = _cg(hs, lam.double()[None], x["q"], case["steps"], 0.0)
    out = (gs * qs[..., None, :]).sum(-1)
    # the packed state also holds copies that nothing reads, so it has no value of its own here
    return {"out": out, "G": gs, "H": None if case["packed"] else hs}


def _exact_ends(case, seed):
    s = {name: None if x is None else x.double() for name, x in _ends_inputs(case, seed).items()}
    b, h, t, dk, dv = case["batch"], case["heads"], case["tokens"], case["d_k"], case["d_v"]

    def conv(x, w):
        if w is None:
            return x
        w = w.reshape(h, -1, 4)
        y = x * w[..., 0]
        for i in range(1, 4):
            y[:, i:] += w[..., i] * x[:, : max(0, t - i)]
        return y * torch.sigmoid(y)

    def heads_first(x):
        return x.transpose(1, 2)

    def unit(x):
        return x / torch.sqrt((x * x).sum(-1, keepdim=True) + 1e-6)

    beta = torch.sigmoid(s["a_beta"])
    gamma = torch.sigmoid(s["a_gamma"]) * (1.0 - (1.0 - 0.9975) * beta * beta)
    o = s["o"]
    y = o / torch.sqrt((o * o).mean(-1, keepdim=True) + 1e-6) * s["weight"][None, :, None, :]
    return {"q": heads_first(unit(conv(s["qp"], s["conv_q"]))).contiguous(),
            "k": heads_first(unit(conv(s["kp"], s["conv_k"]))).contiguous(),
            "v": heads_first(conv(s["vp"], s["conv_v"])).contiguous(),
            "gamma": heads_first(gamma).contiguous(), "beta": heads_first(beta).contiguous(),
            "lam": 0.25 + torch.nn.functional.softplus(s["theta"]), "y": heads_first(y).contiguous()}
