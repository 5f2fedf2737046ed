"""GPU parity of the backward for noisy blocks of two halves (even blocks of 34 .. 64 positions)
against the fp64 oracle: the last block's rows around a half, the smallest and largest halves,
one to four v-heads per q/k head (their q/k gradients summed by one workgroup)."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2606_01774_amd as bd
from paper_2606_01774_amd import workloads as W
from parity_utils import TOL, rel_err

pytestmark = pytest.mark.gpu

NAMES = ("dq", "dk", "dv", "dg", "dbeta", "dqn", "dkn", "dvn", "dgn", "dbetan", "dh0")
KEYS = ("q", "k", "v", "g", "beta")


@pytest.mark.parametrize("B,T,hqk,hv,L,lengths,out", [
    (1, 64, 1, 1, 64, None, torch.float32),                    # one whole block
    (1, 65, 1, 2, 64, None, torch.float32),                    # one row in a second block
    (2, 95, 2, 2, 64, None, torch.bfloat16),                   # a row short of a half
    (2, 97, 1, 3, 64, None, torch.float32),                    # one row in the second half
    (1, 34, 1, 4, 34, None, torch.float32),                    # the smallest halves (17 rows)
    (1, 16, 1, 2, 34, None, torch.bfloat16),                   # less than a half
    (1, 225, 2, 4, 50, [50, 0, 100, 75], torch.float32),       # documents of one, two, one and a half blocks
])
def test_halves(B, T, hqk, hv, L, lengths, out):
    inp = W.make_custom_train(B, T, hqk, hv, 128, 128, "bf16", seed=T + L, lengths=lengths)
    rng = np.random.default_rng(T + L + 1)
    n = B if lengths is None else len(lengths)
    do, don = (torch.from_numpy(rng.standard_normal((B, T, hv, 128)).astype(np.float32)).to(out) for _ in range(2))
    h0 = torch.from_numpy((0.3 * rng.standard_normal((n, hv, 128, 128))).astype(np.float32))
    cu = None if lengths is None else torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32)
    got = bd.bdgdn_bwd_train(*[inp[k].cuda() for k in KEYS], *[inp[k + "n"].cuda() for k in KEYS], do.cuda(),
                             don.cuda(), block=L, cu_seqlens=None if cu is None else cu.cuda(),
                             cu_seqlens_host=cu, h0=h0.cuda(), want_dh0=True)
    torch.cuda.synchronize()
    ref = oracle.bwd_train(*[inp[k] for k in KEYS], *[inp[k + "n"] for k in KEYS], do, don, block=L,
                           scale=1 / math.sqrt(128), cu_seqlens=None if cu is None else cu.numpy(), h0=h0, dht=None)
    for name in NAMES:
        e = rel_err(got[name], ref[name])
        print(f"{name} {e:.2e}", flush=True)
        assert e <= TOL["bf16"], f"{name}: {e:.2e}"
