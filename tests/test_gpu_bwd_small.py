"""GPU parity of the backward for noisy blocks of 1, 2, 4, 8 and 16 positions on clean chunks of
32 (one noisy view): against the fp64 oracle at the edges of a chunk, in time segments bit for
bit, and the per-block schedule where there are too few blocks to gain by chunks."""
import math
import time

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


def _case(B, T, hqk, hv, L, lengths=None, out=torch.float32, gates=None, end=0.1):
    inp = W.make_custom_train(B, T, hqk, hv, 128, 128, "bf16", seed=T + L, lengths=lengths)
    rng = np.random.default_rng(T + L + 1)
    if gates is not None:
        inp["g"], inp["gn"] = draw_gates(rng, inp["g"], gates[0]), draw_gates(rng, inp["gn"], gates[1])
    n = B if lengths is None else len(lengths)
    do, don = (torch.from_numpy(rng.standard_normal((B, T, hv, 128)).astype(np.float32)).to(out) for _ in range(2))
    h0 = torch.from_numpy((0.3 * rng.standard_normal((n, hv, 128, 128))).astype(np.float32))
    # dht reaches the last positions only: at N(0, 1) their dv is up to 34 times the RMS over a
    # sequence of 1500, and its fp16 rounding alone (2^-11 of the entry, twice) 3.3e-2 of that RMS;
    # a tenth of it keeps that part under 4e-3
    dht = torch.from_numpy((end * rng.standard_normal((n, hv, 128, 128))).astype(np.float32))
    cu = None if lengths is None else torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32)

    def run(workspace=None):
        got = bd.bdgdn_bwd_train(*[inp[k].cuda() for k in KEYS], *[inp[k + "n"].cuda() for k in KEYS], do.cuda(),
                                 don.cuda(), block=L, cu_seqlens=None if cu is None else cu.cuda(),
                                 cu_seqlens_host=cu, h0=h0.cuda(), dht=dht.cuda(), want_dh0=True,
                                 workspace=workspace)
        torch.cuda.synchronize()
        return got
    desc = bd.make_fwd_desc(inp["q"], inp["v"], block=L, num_seqs=0 if cu is None else n, out_dtype=out)
    ref = oracle.bwd_train(*[inp[k] for k in KEYS], *[inp[k + "n"] for k in KEYS], do, don, block=L,
                           scale=1 / math.sqrt(128), cu_seqlens=None if cu is None else cu.numpy(), h0=h0, dht=dht)
    return run, desc, cu, ref


def _on_chunks(workspace, T, cu, B):
    """Whether a call ran on chunks in one pass: its segment table, the chunks of the sequences before
    each one, is then what the workspace starts with."""
    lens = [T] * B if cu is None else np.diff(cu.numpy())
    table = np.concatenate([[0], np.cumsum([-(-int(x) // 32) for x in lens])])
    return bool((workspace[:4 * len(table)].cpu().numpy().view(np.int32) == table).all())


def _check(got, ref):
    for name in NAMES:
        e = rel_err(got[name], ref[name])
        assert e <= TOL["bf16"], f"{name}: {e:.2e}"


@pytest.mark.parametrize("B,T,hqk,hv,L,lengths,out,more,chunks", [
    (1, 32, 1, 1, 1, None, torch.float32, 0, True),                     # one chunk, 32 noisy blocks
    (1, 15, 1, 1, 1, None, torch.float32, 0, True),                     # less than half a chunk
    (1, 33, 1, 2, 2, None, torch.float32, 0, True),                     # one position into a second chunk, grouped heads
    (2, 100, 2, 2, 4, None, torch.bfloat16, 0, True),                   # the last chunk one block, bf16 upstream gradients
    (1, 95, 1, 4, 8, None, torch.float32, 0, True),                     # a block short of its last position
    (1, 272, 1, 1, 16, None, torch.float32, 0, True),                   # half a chunk at the end
    (3, 48, 1, 1, 16, None, torch.float32, 0, False),                   # too few blocks to gain by chunks
    (1, 203, 1, 2, 8, [40, 0, 8, 64, 91], torch.float32, 0, True),      # documents across, inside and on chunks, an empty one
    (1, 65, 1, 1, 2, [16, 2, 0, 30, 17], torch.float32, 0, True),       # all shorter than a chunk
    (1, 9, 1, 1, 16, None, torch.float32, 1 << 16, False),              # less than a block, a larger workspace than queried
    (1, 96, 1, 1, 16, [16] * 6, torch.float32, 1 << 18, False),         # documents of one block, the same
    # around the rule: seven steps saved or six; more units than CUs, halved or not
    (1, 240, 1, 1, 16, None, torch.float32, 0, True),
    (1, 208, 1, 1, 16, None, torch.float32, 0, False),
    (44, 12, 2, 2, 4, None, torch.float32, 0, True),
    (42, 12, 2, 2, 4, None, torch.float32, 0, False),
    (44, 48, 2, 2, 16, None, torch.float32, 0, False),
])
def test_small_blocks_match_oracle(B, T, hqk, hv, L, lengths, out, more, chunks):
    print(f"small blocks B={B} T={T} h={hqk}/{hv} L={L} {lengths}", flush=True)
    run, desc, cu, ref = _case(B, T, hqk, hv, L, lengths, out)
    ws = torch.full((bd.bdgdn_bwd_train_workspace(desc) + more,), 255, dtype=torch.uint8, device="cuda")
    _check(run(ws), ref)
    assert _on_chunks(ws, T, cu, B) == chunks


@pytest.mark.parametrize("L", [1, 4, 16])
def test_strong_decays(L):
    """Clean gates from weak to -8, others in each head, beside weak and strong noisy ones: every
    gradient of every head, the clean dg of order exp(g) among them, within the tolerance."""
    # no head has both streams below -5: its dh0, of order exp(-8) / 128, would be at fp16's spacing
    clean = [None, -1.0, -2.0, -5.0, -8.0, ("single", -8.0), -5.0, -3.0]
    noisy = [-5.0, None, None, None, None, None, -5.0, -1.0]
    print(f"small blocks, strong decays: L={L}", flush=True)
    # at g = -1 and below dht reaches the last few positions alone: at a tenth of N(0, 1) their dv is up to
    # 40 times the RMS, which falls with the length, and two fp16 roundings of it 2e-2; a fifth of that here
    run, _, _, ref = _case(1, 264, 8, 8, L, gates=(clean, noisy), end=0.02)
    got = run()
    for name in NAMES:
        e, unit, n = unit_errors(got[name], ref[name], per_token=None if name == "dh0" else got[name].dim() == 3)
        assert n == 8 and e <= TOL["bf16"], f"{name} {unit}: {e:.2e}"


@pytest.mark.parametrize("B,T,hqk,hv,L,lengths", [
    (1, 2050, 1, 1, 4, None),
    (2, 1500, 1, 2, 16, None),
    (1, 2800, 1, 1, 16, [2400, 0, 48, 352]),
])
def test_small_blocks_segments_bitwise(B, T, hqk, hv, L, lengths):
    """The smallest workspace the segmented queries name holds only some of the chunks: the same
    bits as in one pass."""
    run, desc, cu, ref = _case(B, T, hqk, hv, L, lengths)
    size = min(bd.bdgdn_bwd_train_workspace_segmented(desc, cu, k) for k in range(2, 40))
    chunks = sum(-(-int(x) // 32) for x in (np.diff(cu.numpy()) if cu is not None else [T] * B)) * hv
    assert size < chunks * (2 * 128 + 2 * 32) * 128 * 2
    print(f"small blocks in segments, B={B} T={T} L={L} {lengths}: {size} bytes", flush=True)
    one, seg = run(), run(torch.empty(size, dtype=torch.uint8, device="cuda"))
    for name in NAMES:
        assert torch.equal(one[name], seg[name]), name
    _check(seg, ref)


def test_documents_shorter_than_a_chunk_keep_their_workspace():
    """Documents of one block of 16: chunks would need more than the queried workspace and save nothing,
    so blocks run one by one."""
    run, desc, cu, ref = _case(1, 96, 1, 1, 16, [16] * 6)
    print("small blocks: documents of one block", flush=True)
    ws = torch.full((bd.bdgdn_bwd_train_workspace(desc),), 255, dtype=torch.uint8, device="cuda")
    _check(run(ws), ref)
    assert not _on_chunks(ws, 96, cu, 1)


def test_short_documents_beside_a_long_one_are_planned_at_once():
    """Chunks do not fit the queried workspace here in any number of segments: finding that out takes a
    few passes over the documents, not one for every number of segments of the long one (over 50 ms)."""
    lengths = [16] * 12000 + [6000 * 16]
    T, L = sum(lengths), 16
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32)
    gen = torch.Generator(device="cuda").manual_seed(0)
    x = [torch.randn(1, T, 1, 128, generator=gen, device="cuda").mul_(0.1).bfloat16() for _ in range(3)]
    gate = torch.full((1, T, 1), -0.05, device="cuda")
    beta = torch.full((1, T, 1), 0.5, device="cuda")
    do = torch.zeros(1, T, 1, 128, device="cuda")
    ws = torch.empty(bd.bdgdn_bwd_train_workspace(bd.make_fwd_desc(x[0], x[2], block=L, num_seqs=len(lengths))),
                     dtype=torch.uint8, device="cuda")
    print("small blocks: many short documents and a long one", flush=True)
    times = []
    for _ in range(3):
        torch.cuda.synchronize()
        t = time.perf_counter()
        bd.bdgdn_bwd_train(*x, gate, beta, *x, gate, beta, do, do, block=L, cu_seqlens=cu.cuda(), cu_seqlens_host=cu,
                           workspace=ws)
        times.append(time.perf_counter() - t)
    torch.cuda.synchronize()
    assert not _on_chunks(ws, T, cu, 1)
    assert min(times) < 0.02, times
