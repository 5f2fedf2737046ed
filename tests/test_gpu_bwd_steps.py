"""GPU parity of the per-step backward's two schedules against the fp64 oracle: parallel over
blocks (the default, with two fp32 states per (block, v-head) of workspace) and the serial
walk that a smaller workspace selects.  Sizes at the edges of what the kernels cut: spans of 4
positions, chunks of 8 rows and 64 gates, the state kept at a block's middle (blocks from 8
positions on), d_k != d_v, grouped heads, documents, several views."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2606_01774_amd as bd
from paper_2606_01774_amd import workloads as W
from parity_utils import TOL, draw_gates, rel_err, unit_errors

pytestmark = pytest.mark.gpu

NAMES = ("dq", "dk", "dv", "dg", "dbeta", "dqn", "dkn", "dvn", "dgn", "dbetan", "dh0")
KEYS = ("q", "k", "v", "g", "beta")


def _walk_bytes(n_seq, blocks, hv, dk, dv):
    """The serial walk's workspace: a state per started group of eight blocks and chain, and
    eight 16-column tile states per (chain, tile)."""
    up = lambda x: -(-x // 256) * 256   # noqa: E731
    return up((blocks // 8 + n_seq) * hv * dk * dv * 4) + up(n_seq * hv * (dv // 16) * 8 * dk * 16 * 4)


def _inputs(B, T, hqk, hv, dk, dv, dtype, seed, lengths):
    inp = W.make_custom_train(B, T, hqk, hv, dk, dv, dtype, seed=seed, lengths=lengths)
    rng = np.random.default_rng(seed + 1)
    n = B if lengths is None else len(lengths)
    do, don = (torch.from_numpy(rng.standard_normal((B, T, hv, dv)).astype(np.float32)) for _ in range(2))
    h0 = torch.from_numpy((0.3 * rng.standard_normal((n, hv, dk, dv))).astype(np.float32))
    dht = torch.from_numpy(rng.standard_normal((n, hv, dk, dv)).astype(np.float32))
    cu = None if lengths is None else torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32)
    return inp, do, don, h0, dht, cu


@pytest.mark.parametrize("walk", [False, True])
@pytest.mark.parametrize("B,T,hqk,hv,dk,dv,L,dtype,lengths", [
    (1, 1, 1, 1, 64, 64, 1, "f32", None),             # one position
    (2, 67, 1, 2, 64, 128, 4, "f32", None),           # one span per block, 64 gates and 3 more
    (1, 63, 2, 4, 128, 64, 7, "f32", None),           # a short second span, no middle state
    (1, 130, 1, 1, 128, 128, 9, "f32", None),         # a middle state, one position past a span
    (3, 33, 1, 1, 64, 64, 32, "f32", None),           # a one-position tail block
    (1, 300, 1, 2, 64, 64, 8, "f32", [64, 0, 8, 228]),    # documents, an empty one
    (1, 129, 1, 1, 64, 64, 64, "bf16", None),         # the longest blocks
    (1, 250, 1, 2, 128, 128, 63, "bf16", [126, 124]),     # odd blocks, the largest LDS
])
def test_both_schedules_match_oracle(B, T, hqk, hv, dk, dv, L, dtype, lengths, walk):
    inp, do, don, h0, dht, cu = _inputs(B, T, hqk, hv, dk, dv, dtype, 40 + T + L, lengths)
    n, blocks = (B, B * -(-T // L)) if lengths is None else (len(lengths), -(-T // L))
    d = {k: v.cuda() for k, v in inp.items()}
    desc = bd.make_fwd_desc(d["q"], d["v"], block=L, num_seqs=0 if cu is None else n)
    steps = 2 * (-(-blocks * hv * dk * dv * 4 // 256) * 256)
    small = _walk_bytes(n, blocks, hv, dk, dv)
    assert bd.bdgdn_bwd_train_workspace(desc) == max(small, steps)
    if walk and small >= steps:
        small = steps - 256                       # below the parallel schedule: must be refused or walk
    size = small if walk else max(small, steps)
    print(f"steps B={B} T={T} h={hqk}/{hv} d={dk}x{dv} L={L} {dtype} {lengths} workspace {size}", flush=True)
    args = ([d[k] for k in KEYS] + [d[k + "n"] for k in KEYS] + [do.cuda(), don.cuda()])
    kw = dict(block=L, cu_seqlens=None if cu is None else cu.cuda(), cu_seqlens_host=cu, h0=h0.cuda(),
              dht=dht.cuda(), want_dh0=True, workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
    if walk and size < _walk_bytes(n, blocks, hv, dk, dv):
        with pytest.raises(bd.BdgdnError):        # less than both schedules need
            bd.bdgdn_bwd_train(*args, **kw)
        return
    got = bd.bdgdn_bwd_train(*args, **kw)
    torch.cuda.synchronize()
    ref = oracle.bwd_train(*[inp[k] for k in KEYS], *[inp[k + "n"] for k in KEYS], do, don, block=L,
                           scale=1 / math.sqrt(dk), cu_seqlens=None if cu is None else cu.numpy(), h0=h0, dht=dht)
    for name in NAMES:
        e = rel_err(got[name], ref[name])
        assert e <= TOL["f32"], f"{name}: {e:.2e}"   # everything is fp32 whatever the input type


@pytest.mark.parametrize("walk", [False, True])
@pytest.mark.parametrize("T,dk,dv,L,dtype", [
    (9, 64, 64, 1, "f32"),
    (23, 64, 128, 4, "f32"),
    (82, 64, 64, 16, "f32"),            # a middle state, a short tail block
    (108, 128, 64, 21, "f32"),          # a middle state off the block's middle
    (322, 64, 64, 64, "bf16"),          # the longest blocks
    (190, 128, 128, 37, "bf16"),
])
def test_strong_decays(T, dk, dv, L, dtype, walk):
    """Gates from weak to -20, others in each head and in the two streams: every gradient of every
    head, dg of order exp(g) among them, is as exact as with weak ones."""
    clean = [None, -1.0, -3.0, -5.0, -8.0, -20.0, ("single", -12.0), -8.0]
    noisy = [-5.0, None, -8.0, None, -1.0, ("single", -12.0), -20.0, -8.0]
    H = len(clean)
    inp, do, don, h0, dht, _ = _inputs(1, T, H, H, dk, dv, dtype, 90 + T, None)
    rng = np.random.default_rng(T)
    inp["g"], inp["gn"] = draw_gates(rng, inp["g"], clean), draw_gates(rng, inp["gn"], noisy)
    d = {k: v.cuda() for k, v in inp.items()}
    blocks = -(-T // L)
    size = _walk_bytes(1, blocks, H, dk, dv)
    assert size < 2 * blocks * H * dk * dv * 4   # the walk's, and not the parallel schedule's
    print(f"steps, strong decays: T={T} d={dk}x{dv} L={L} {dtype} walk={walk}", flush=True)
    got = bd.bdgdn_bwd_train(*[d[k] for k in KEYS], *[d[k + "n"] for k in KEYS], do.cuda(), don.cuda(), block=L,
                             h0=h0.cuda(), dht=dht.cuda(), want_dh0=True,
                             workspace=torch.empty(size, dtype=torch.uint8, device="cuda") if walk else None)
    torch.cuda.synchronize()
    ref = oracle.bwd_train(*[inp[k] for k in KEYS], *[inp[k + "n"] for k in KEYS], do, don, block=L,
                           scale=1 / math.sqrt(dk), h0=h0, dht=dht)
    for name in NAMES:
        per_token = None if name == "dh0" else got[name].dim() == 3
        e, unit, n = unit_errors(got[name], ref[name], per_token=per_token)
        assert n == H and e <= TOL["f32"], f"{name} {unit}: {e:.2e}"


def test_views_deterministic_and_match_oracle():
    """Four noisy views of grouped heads in fp32: against the oracle, and twice the same bits."""
    B, T, hqk, hv, d, L = 1, 90, 1, 2, 64, 16
    base, do, _, h0, dht, _ = _inputs(B, T, hqk, hv, d, d, "f32", 7, None)
    views = []
    for i in range(4):
        src, dv = W.make_custom_train(B, T, hqk, hv, d, d, "f32", seed=70 + i), np.random.default_rng(80 + i)
        w = {k: src[k + "n"] for k in KEYS}
        w["do"] = torch.from_numpy(dv.standard_normal((B, T, hv, d)).astype(np.float32))
        views.append(w)
    print("steps: four views", flush=True)
    dv = [{k: x.cuda() for k, x in w.items()} for w in views]
    runs = [bd.bdgdn_bwd_train_views(*[base[k].cuda() for k in KEYS], dv, do.cuda(), block=L, h0=h0.cuda(),
                                     dht=dht.cuda(), want_dh0=True) for _ in range(2)]
    torch.cuda.synchronize()
    ref_c, ref_v = oracle.bwd_train_views(*[base[k] for k in KEYS], views, do, block=L, scale=1 / math.sqrt(d),
                                          h0=h0, dht=dht)
    for n in ("dq", "dk", "dv", "dg", "dbeta", "dh0"):
        assert rel_err(runs[0][0][n], ref_c[n]) <= TOL["f32"], n
        assert torch.equal(runs[0][0][n], runs[1][0][n]), n
    for i in range(4):
        for n in ("dq", "dk", "dv", "dg", "dbeta"):
            assert rel_err(runs[0][1][i][n], ref_v[i][n]) <= TOL["f32"], (i, n)
            assert torch.equal(runs[0][1][i][n], runs[1][1][i][n]), (i, n)


@pytest.mark.parametrize("T,d,L,dtype", [
    (70, 64, 16, "f32"),       # per-step
    (70, 128, 32, "bf16"),     # block form, and on chunks, and in halves
    (70, 128, 4, "bf16"),
    (70, 128, 64, "bf16"),
])
def test_gradients_at_any_float(T, d, L, dtype):
    """The gradient buffers need no more alignment than a float: one float past a 16-byte boundary the
    results are the same bits."""
    inp, do, don, h0, dht, _ = _inputs(1, T, 1, 2, d, d, dtype, 60 + L, None)
    dev = {k: v.cuda() for k, v in inp.items()}
    args = [dev[k] for k in KEYS] + [dev[k + "n"] for k in KEYS] + [do.cuda(), don.cuda()]
    kw = dict(block=L, h0=h0.cuda(), dht=dht.cuda(), want_dh0=True)
    print(f"gradients one float off: d={d} L={L} {dtype}", flush=True)
    want = bd.bdgdn_bwd_train(*args, **kw)
    grads = {}
    for name, x in want.items():
        grads[name] = torch.empty(x.numel() + 4, device="cuda")[1:1 + x.numel()].view(x.shape)
        assert grads[name].data_ptr() % 16 == 4
    got = bd.bdgdn_bwd_train(*args, grads=grads, **kw)
    torch.cuda.synchronize()
    for name in NAMES:
        assert got[name].data_ptr() == grads[name].data_ptr()
        assert torch.equal(got[name], want[name]), name
