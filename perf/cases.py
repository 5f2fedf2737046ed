"""The work that a user of the block-diffusion Gated DeltaNet layer has it do, as timed cases.

Three kinds of program use the layer.  A training program runs the two-stream forward and its
backward on long batched or packed sequences (``fwd``, ``bwd``, ``step``) and the ShortConv in
front of them (``conv``).  A serving program runs one block per request against cached states:
the read-only denoise pass many times (``denoise``), the commit pass once per block
(``commit``), or the AR-Trust verify round with its accept step (``verify``).  A developer checks
the same layer in fp32 on small shapes (``step`` with ``dtype`` "f32").

A case is a dict of plain values; ``prepare`` makes what the program holds before the call (on
the GPU, from the seed alone, with the input distributions of ``workloads.py``), ``run`` is one
pass through the public entry points, ``exact`` the same results in float64 by plain torch.
"""
import math

import torch

import paper_2606_01774_amd as bd

# The training workloads are those of paper_2606_01774_amd/workloads.py and of the block-size
# sweep of bench.py; the serving ones have its 32 heads of 128 x 128.
_TRAIN = dict(batch=1, seqlen=4096, docs=0, h_qk=16, h_v=16, d=128, block=32, dtype="bf16", out="f32")


def _train(**kw):
    return {**_TRAIN, **kw}


def listed():
    return [
        # One user's chat at a time: the denoise pass of a single request, called in a loop by
        # the sampler, where the latency of the call is all that counts.
        dict(name="denoise_1_request", kind="denoise", requests=1, h_qk=32, h_v=32, d=128, block=32, out="f32"),
        # A loaded server: 64 concurrent requests, one denoise step.
        dict(name="denoise_64_requests", kind="denoise", requests=64, h_qk=32, h_v=32, d=128, block=32, out="f32"),
        # The same server when the blocks are done: the token-causal pass that advances every
        # cached state, with its outputs.
        dict(name="commit_64_requests", kind="commit", requests=64, h_qk=32, h_v=32, d=128, block=32, out="f32"),
        # An AR-Trust verify round: the anchor and 7 draft tokens per request, the states before
        # each draft position kept, then the accept step that rewinds.
        dict(name="verify_64_requests", kind="verify", requests=64, h_qk=32, h_v=32, d=128, block=8, out="f32"),
        # The layer's training forward on the usual batch (4 sequences of 4096 clean + 4096 noisy
        # tokens), and its backward.
        dict(name="fwd_4x4096", kind="fwd", **_train(batch=4)),
        dict(name="bwd_4x4096", kind="bwd", **_train(batch=4)),
        # A training step with the small diffusion blocks (4 positions) a diffusion model is
        # trained with when it has to decode few tokens at a time.
        dict(name="step_blocks_of_4", kind="step", **_train(block=4)),
        # A training step with grouped value heads, long sequences and large blocks.
        dict(name="step_grouped_16k", kind="step",
             **_train(batch=2, seqlen=16384, h_v=32, block=64, out="bf16")),
        # Document packing: a long packed batch, forward with bf16 outputs; and a step on a
        # short one whose last document ends inside a block, as the end of a data set does.
        dict(name="fwd_packed_128k", kind="fwd", **_train(seqlen=131072, docs=32, out="bf16")),
        dict(name="step_packed_ragged", kind="step", **_train(seqlen=6007, docs=5)),
        # The ShortConv in front of the layer (q, k, v projections side by side), both ways.
        dict(name="conv_4x4096", kind="conv", batch=4, seqlen=4096, channels=6144, width=4, block=32, dtype="bf16"),
        # A developer's fp32 check of forward and gradients on a small shape.
        dict(name="step_f32_small", kind="step",
             **_train(seqlen=256, h_qk=2, h_v=2, d=64, block=16, dtype="f32")),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["denoise", "commit", "verify", "fwd", "bwd", "step", "step", "f32", "conv"])
    heads = rng.choice([(16, 16), (16, 32), (32, 32), (8, 8), (4, 12)])
    out = rng.choice(["f32", "bf16"])
    if kind in ("denoise", "commit"):
        return dict(kind=kind, requests=_log(rng, 1, 64), h_qk=heads[0], h_v=heads[1], d=128,
                    block=rng.choice([4, 8, 16, 24, 32]), out=out)
    if kind == "verify":
        return dict(kind=kind, requests=_log(rng, 1, 64), h_qk=heads[0], h_v=heads[1], d=128,
                    block=rng.randint(2, 8), out="f32")
    if kind == "conv":
        return dict(kind=kind, batch=rng.randint(1, 4), seqlen=_log(rng, 100, 4096),
                    channels=4 * _log(rng, 128, 1536), width=rng.randint(2, 4), block=rng.choice([4, 8, 16, 32, 64]),
                    dtype=rng.choice(["bf16", "bf16", "f32"]))
    if kind == "f32":   # a developer's checks; the smaller head size in bf16 among them
        d = rng.choice([64, 64, 128])
        h_qk = rng.randint(1, 4)
        dtype = rng.choice(["f32", "f32", "bf16"]) if d == 64 else "f32"
        return dict(kind="step", **_train(batch=rng.randint(1, 3), seqlen=_log(rng, 40, 400 * 64 // d), h_qk=h_qk,
                                          h_v=h_qk * rng.randint(1, 2), d=d, block=rng.choice([4, 8, 16, 32]),
                                          dtype=dtype))
    block = rng.choice([1, 2, 4, 4, 8, 8, 16, 16, 32, 32, 32, 32, 48, 64])
    # rows x v-heads: the backward's work grows with the number of blocks
    rows = _log(rng, 300, 16384) if kind == "fwd" else _log(rng, 300, min(16384, 800 * block))
    rows = max(rows * 16 // max(16, heads[1]), 64)
    if rng.random() < 0.4:
        docs = rng.randint(2, max(2, min(24, rows // 128)))
        return dict(kind=kind, **_train(seqlen=max(rows, 2 * docs * block), docs=docs, h_qk=heads[0], h_v=heads[1],
                                        block=block, out=out))
    batch = rng.randint(1, 4)
    return dict(kind=kind, **_train(batch=batch, seqlen=max(rows // batch, 24), h_qk=heads[0], h_v=heads[1],
                                    block=block, out=out))


_DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def _document_offsets(case):
    """Document starts on block boundaries, lengths spread 1 : 4; the last document takes the rest."""
    n, total, L = case["docs"], case["seqlen"], case["block"]
    weights = [1.0 + 3.0 * ((7 * i + 3) % n) / n for i in range(n)]
    cu, acc = [0], 0.0
    for w in weights[:-1]:
        acc += w
        cu.append(max(cu[-1], int(total * acc / sum(weights)) // L * L))
    return cu + [total]


def _stream(gen, rows, h_qk, h_v, d, dtype):
    """q, k L2-normalised normals, v normal, g = -softplus(U(-6, -2)), beta = sigmoid(U(-2, 2))."""
    dev = gen.device

    def normal(h):
        return torch.randn(*rows, h, d, generator=gen, device=dev)

    q, k, v = normal(h_qk), normal(h_qk), normal(h_v)
    q = q / q.norm(dim=-1, keepdim=True)
    k = k / k.norm(dim=-1, keepdim=True)
    g = -torch.nn.functional.softplus(torch.rand(*rows, h_v, generator=gen, device=dev) * 4 - 6)
    beta = torch.sigmoid(torch.rand(*rows, h_v, generator=gen, device=dev) * 4 - 2)
    return [q.to(dtype), k.to(dtype), v.to(dtype), g, beta]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind = case["kind"]
    s = dict(case=case)
    if kind == "conv":
        shape, dt = (case["batch"], case["seqlen"], case["channels"]), _DT[case["dtype"]]
        for name in ("x", "xn", "dy", "dyn"):
            s[name] = torch.randn(shape, generator=gen, device="cuda").to(dt)
        bound = 1 / math.sqrt(case["width"])
        s["w"] = (torch.rand(case["channels"], case["width"], generator=gen, device="cuda") * 2 - 1) * bound
        s["bias"] = (torch.rand(case["channels"], generator=gen, device="cuda") * 2 - 1) * bound
        return s
    h_qk, h_v, d = case["h_qk"], case["h_v"], case["d"]
    if kind in ("denoise", "commit", "verify"):
        R, L = case["requests"], case["block"]
        s["in"] = _stream(gen, (R, L), h_qk, h_v, d, torch.bfloat16)
        # states of a few hundred tokens, in a pool with free slots, at scattered places
        slots = R + max(1, R // 4)
        s["pool"] = torch.randn(slots, h_v, d, d, generator=gen, device="cuda") * 0.15
        s["slot"] = torch.randperm(slots, generator=gen, device="cuda")[:R].to(torch.int32).contiguous()
        s["o"] = torch.empty(R, L, h_v, d, dtype=_DT[case["out"]], device="cuda")
        if kind == "verify":
            s["states"] = torch.empty(R, L - 1, h_v, d, d, device="cuda")
            s["accept"] = torch.randint(0, L, (R,), generator=gen, device="cuda").to(torch.int32)
        return s
    B, T = case["batch"], case["seqlen"]
    s["clean"] = _stream(gen, (B, T), h_qk, h_v, d, _DT[case["dtype"]])
    s["noisy"] = _stream(gen, (B, T), h_qk, h_v, d, _DT[case["dtype"]])
    s["pack"] = {}
    if case["docs"]:
        host = torch.tensor(_document_offsets(case), dtype=torch.int32)
        s["pack"] = dict(cu_seqlens=host.to("cuda"), cu_seqlens_host=host)
    if kind != "fwd":
        # a loss averaged over tokens: small upstream gradients
        for name in ("do", "don"):
            s[name] = (torch.randn(B, T, h_v, d, generator=gen, device="cuda") * 1e-3).to(_DT[case["out"]])
    return s


_GRADS = ("dq", "dk", "dv", "dg", "dbeta", "dqn", "dkn", "dvn", "dgn", "dbetan")


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "conv":
        y, yn = bd.bdgdn_shortconv_fwd(s["x"], s["xn"], s["w"], s["bias"], block=case["block"])
        dx, dxn, dw, db = bd.bdgdn_shortconv_bwd(s["x"], s["xn"], s["w"], s["bias"], s["dy"], s["dyn"],
                                                 block=case["block"])
        return dict(y=y, yn=yn, dx=dx, dxn=dxn, dw=dw, db=db)
    if kind == "denoise":
        return dict(o=bd.bdgdn_denoise_step(s["pool"], *s["in"], slot=s["slot"], o=s["o"]))
    if kind == "commit":
        o = bd.bdgdn_commit(s["pool"], *s["in"], slot=s["slot"], o_causal=s["o"])
        return dict(o=o, pool=s["pool"])
    if kind == "verify":
        states, o = bd.bdgdn_commit_record(s["pool"], *s["in"], n_record=case["block"] - 1, slot=s["slot"],
                                           states=s["states"], o_causal=s["o"])
        bd.bdgdn_accept_states(s["pool"], states, s["accept"], block=case["block"], h_qk=case["h_qk"], slot=s["slot"])
        return dict(o=o, states=states, pool=s["pool"])
    out = {}
    if kind in ("fwd", "step"):
        o, on, ht = bd.bdgdn_fwd_train(*s["clean"], *s["noisy"], block=case["block"], want_ht=True,
                                       out_dtype=_DT[case["out"]], **s["pack"])
        out.update(o=o, on=on, ht=ht)
    if kind in ("bwd", "step"):
        out.update(bd.bdgdn_bwd_train(*s["clean"], *s["noisy"], s["do"], s["don"], block=case["block"], **s["pack"]))
    return out


def work(case):
    kind = case["kind"]
    if kind == "conv":
        n = case["batch"] * case["seqlen"] * case["channels"] * (2 if case["dtype"] == "bf16" else 4)
        rows = case["batch"] * case["seqlen"] * case["channels"]
        # forward x, xn, y, yn; backward x, xn, dy, dyn, dx, dxn
        return dict(bytes=10 * n, flops=2 * rows * (2 * case["width"] + 6 * case["width"]))
    h_qk, h_v, d = case["h_qk"], case["h_v"], case["d"]
    ob = 2 if case["out"] == "bf16" else 4
    if kind in ("denoise", "commit", "verify"):
        R, L = case["requests"], case["block"]
        tok = R * L * (h_qk * 2 * d * 2 + h_v * (2 * d + 8 + ob * d))
        state = R * h_v * d * d * 4
        # verify: the pool in and out, L - 1 states written; the accept step reads and writes
        # one state of a request (none where all drafts are accepted, 1 in L)
        states = {"denoise": 1.0, "commit": 2.0, "verify": 2 + (L - 1) + 2 * (L - 1) / L}[kind]
        return dict(bytes=int(tok + states * state), flops=8 * R * L * h_v * d * d)
    rows = case["batch"] * case["seqlen"]
    ib = 2 if case["dtype"] == "bf16" else 4
    units = case["docs"] or case["batch"]
    inputs = 2 * rows * (h_qk * 2 * d * ib + h_v * (d * ib + 8))
    nbytes = flops = 0
    if kind in ("fwd", "step"):
        nbytes += inputs + 2 * rows * h_v * d * ob + units * h_v * d * d * 4
        flops += 2 * rows * h_v * 8 * d * d
    if kind in ("bwd", "step"):
        nbytes += inputs + 2 * rows * h_v * d * ob + 2 * rows * (h_qk * 2 * d + h_v * (d + 2)) * 4
        flops += 2 * rows * h_v * 16 * d * d
    return dict(bytes=int(nbytes), flops=int(flops))


def tolerance(case):
    """About four times the error against ``exact`` of each precision: fp32 throughout 3e-7, fp16 matrix operands
    under fp32 sums 6e-4 (bf16 inputs, fp32 results), results rounded to bf16 1.7e-3."""
    if case.get("dtype") == "f32":
        rel = 2e-6
    elif case.get("out") == "bf16" or case["kind"] == "conv":
        rel = 7e-3
    else:
        rel = 2.4e-3
    return dict(rel=rel, max=20 * rel)


# ---------------------------------------------------------------- float64 reference
def _tri_inverse(A):
    """(I + A)^-1 of strictly lower triangular A [..., L, L] by doubling."""
    L = A.shape[-1]
    eye = torch.eye(L, dtype=A.dtype, device=A.device)
    inv, p = eye - A, A @ A
    n = 2
    while n < L:
        inv = inv @ (eye + p)
        p = p @ p
        n *= 2
    return inv


def _intra(k, g, beta):
    """Per block [..., L, d]: gamma [..., L], decays D = gamma_n / gamma, T = (I + A)^-1 diag(beta)."""
    G = g.cumsum(-1)
    low = torch.ones(G.shape[-1], G.shape[-1], dtype=torch.bool, device=G.device).tril(-1)
    dec = torch.exp((G[..., :, None] - G[..., None, :]).masked_fill(~low, 0.0))
    A = (beta[..., :, None] * dec * (k @ k.transpose(-1, -2))).masked_fill(~low, 0.0)
    return G, torch.exp(G[..., -1:] - G), _tri_inverse(A) * beta[..., None, :]


def _two_streams(clean, noisy, block, scale, h0):
    """clean, noisy: q, k, v [N, H, nb, L, d], g, beta [N, H, nb, L] float64 -> o, on, ht."""
    q, k, v, g, beta = clean
    G, D, T = _intra(k, g, beta)
    gam = torch.exp(G)
    S, seeds, deltas = h0, [], []
    kd = k * D[..., None]
    for b in range(k.shape[2]):
        seeds.append(S)
        delta = T[:, :, b] @ (v[:, :, b] - gam[:, :, b, :, None] * (k[:, :, b] @ S))
        deltas.append(delta)
        S = gam[:, :, b, -1, None, None] * S + kd[:, :, b].transpose(-1, -2) @ delta
    seed, delta = torch.stack(seeds, 2), torch.stack(deltas, 2)
    low = torch.ones(block, block, dtype=torch.bool, device=q.device).tril()
    dec = torch.exp((G[..., :, None] - G[..., None, :]).masked_fill(~low, 0.0))
    P = (dec * (q @ k.transpose(-1, -2))).masked_fill(~low, 0.0)
    o = scale * (gam[..., None] * (q @ seed) + P @ delta)
    qn, kn, vn, gn, betan = noisy
    Gn, Dn, Tn = _intra(kn, gn, betan)
    deltan = Tn @ (vn - torch.exp(Gn)[..., None] * (kn @ seed))
    on = scale * (torch.exp(Gn[..., -1])[..., None, None] * (qn @ seed)
                  + (qn @ kn.transpose(-1, -2)) @ (Dn[..., None] * deltan))
    return o, on, S


def _spans(case):
    if case["docs"]:
        cu = _document_offsets(case)
        return [(0, cu[i], cu[i + 1]) for i in range(case["docs"])]
    return [(b, 0, case["seqlen"]) for b in range(case["batch"])]


def _to_blocks(x, spans, L, heads):
    """[B, T, h(, d)] -> [N, heads, nb, L(, d)] float64, sequences padded with zeros, heads repeated."""
    nb = max(-(-(e - s) // L) for _, s, e in spans)
    y = torch.zeros(len(spans), nb * L, *x.shape[2:], dtype=torch.float64, device=x.device)
    for i, (b, s, e) in enumerate(spans):
        y[i, :e - s] = x[b, s:e]
    y = y.reshape(len(spans), nb, L, *x.shape[2:]).transpose(2, 3).transpose(1, 2)   # [N, h, nb, L, ...]
    return y.repeat_interleave(heads // x.shape[2], 1).contiguous()


def _from_blocks(y, spans, B, T, h):
    """The inverse, repeated heads summed."""
    y = y.reshape(y.shape[0], h, y.shape[1] // h, *y.shape[2:]).sum(2)
    y = y.transpose(1, 2).transpose(2, 3)
    y = y.reshape(y.shape[0], y.shape[1] * y.shape[2], *y.shape[3:])
    x = torch.zeros(B, T, *y.shape[2:], dtype=torch.float64, device=y.device)
    for i, (b, s, e) in enumerate(spans):
        x[b, s:e] = y[i, :e - s]
    return x


def _exact_train(case, s):
    L, H, B, T, d = case["block"], case["h_v"], case["batch"], case["seqlen"], case["d"]
    spans, grad = _spans(case), case["kind"] != "fwd"
    sides = [[_to_blocks(x, spans, L, H).requires_grad_(grad) for x in s[key]] for key in ("clean", "noisy")]
    scale = float(torch.tensor(1 / math.sqrt(d), dtype=torch.float32))
    h0 = torch.zeros(len(spans), H, d, d, dtype=torch.float64, device="cuda")
    o, on, ht = _two_streams(*sides, L, scale, h0)
    out = {}
    if case["kind"] in ("fwd", "step"):
        out.update(o=_from_blocks(o.detach(), spans, B, T, H), on=_from_blocks(on.detach(), spans, B, T, H),
                   ht=ht.detach())
    if grad:
        do, don = (_to_blocks(s[key], spans, L, H) for key in ("do", "don"))
        grads = torch.autograd.grad([o, on], sides[0] + sides[1], [do, don])
        for name, x, gr in zip(_GRADS, s["clean"] + s["noisy"], grads):
            out[name] = _from_blocks(gr, spans, B, T, x.shape[2])
    return out


def _exact_serve(case, s):
    H, L, kind = case["h_v"], case["block"], case["kind"]
    pool, slot = s["pool"].double(), s["slot"].long()
    q, k, v, g, beta = (x.double() for x in s["in"])
    q, k = (x.repeat_interleave(H // x.shape[2], 2) for x in (q, k))
    scale = float(torch.tensor(1 / math.sqrt(case["d"]), dtype=torch.float32))
    S, o, states = pool[slot], [], []
    for t in range(L):
        states.append(S)
        S = torch.exp(g[:, t])[..., None, None] * S
        u = v[:, t] - (k[:, t, :, None] @ S)[:, :, 0]
        S = S + (beta[:, t, :, None] * k[:, t])[..., None] * u[:, :, None]
        o.append(scale * (q[:, t, :, None] @ S)[:, :, 0])
    if kind == "denoise":
        return dict(o=scale * torch.stack([(q[:, t, :, None] @ S)[:, :, 0] for t in range(L)], 1))
    out = dict(o=torch.stack(o, 1))
    if kind == "verify":
        out["states"] = torch.stack(states[1:], 1)
        kept = torch.stack(states[1:] + [S], 1)
        S = kept[torch.arange(kept.shape[0], device="cuda"), s["accept"].long()]
    pool[slot] = S
    out["pool"] = pool
    return out


def _exact_conv(case, s):
    x, xn = (s[key].double().requires_grad_() for key in ("x", "xn"))
    w, bias = s["w"].double().requires_grad_(), s["bias"].double().requires_grad_()
    T, L = case["seqlen"], case["block"]
    t = torch.arange(T, device="cuda")
    y = yn = bias
    for i in range(case["width"]):
        back = lambda z: torch.nn.functional.pad(z, (0, 0, i, 0))[:, :T]   # noqa: E731
        same = (t % L >= i)[:, None]
        y = y + w[:, i] * back(x)
        yn = yn + w[:, i] * torch.where(same, back(xn), back(x))
    y, yn = torch.nn.functional.silu(y), torch.nn.functional.silu(yn)
    dx, dxn, dw, db = torch.autograd.grad([y, yn], [x, xn, w, bias], [s["dy"].double(), s["dyn"].double()])
    return dict(y=y.detach(), yn=yn.detach(), dx=dx, dxn=dxn, dw=dw, db=db)


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "conv":
        return _exact_conv(case, s)
    if case["kind"] in ("denoise", "commit", "verify"):
        return _exact_serve(case, s)
    return _exact_train(case, s)
