"""Roundings on the way to a gradient of the block-form backward, by the 2-norm of its error
against the fp64 oracle: with bf16 upstream gradients (exact in fp16) the error is that of the
fp16 roundings in between, each of relative RMS 2^-11 / sqrt(3) times the RMS of 1 / x over a
binade of log-uniform x, 2.1e-4, and independent ones add in squares."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2606_01774_amd as bd
from paper_2606_01774_amd import workloads as W
from parity_utils import draw_gates

pytestmark = pytest.mark.gpu

KEYS = ("q", "k", "v", "g", "beta")
ONE = 2.0 ** -11 / math.sqrt(3) * math.sqrt(0.375 / math.log(2))


def _errors(L, clean, noisy, with_clean, T=256, seeds=4, with_dht=False):
    """Relative 2-norm error of every gradient over all heads and seeds; the clean readout's
    upstream gradient zero unless with_clean, that of the final state without with_dht."""
    H, num, den = len(clean), {}, {}
    for seed in range(seeds):
        inp = W.make_custom_train(1, T, H, H, 128, 128, "bf16", seed=300 + seed)
        rng = np.random.default_rng(400 + seed)
        inp["g"], inp["gn"] = draw_gates(rng, inp["g"], clean), draw_gates(rng, inp["gn"], noisy)
        do, don = (torch.from_numpy(rng.standard_normal((1, T, H, 128)).astype(np.float32)).bfloat16()
                   for _ in range(2))
        if not with_clean:
            do = torch.zeros_like(do)
        dht = torch.from_numpy(0.1 * rng.standard_normal((1, H, 128, 128)).astype(np.float32)) if with_dht else None
        got = bd.bdgdn_bwd_train(*[inp[k].cuda() for k in KEYS], *[inp[k + "n"].cuda() for k in KEYS], do.cuda(),
                                 don.cuda(), block=L, dht=None if dht is None else dht.cuda(), want_dh0=True)
        torch.cuda.synchronize()
        ref = oracle.bwd_train(*[inp[k] for k in KEYS], *[inp[k + "n"] for k in KEYS], do, don, block=L,
                               scale=1 / math.sqrt(128), dht=dht)
        for name, x in ref.items():
            axes = tuple(i for i in range(x.ndim) if i != (1 if name == "dh0" else 2))
            d = got[name].double().cpu().numpy() - x
            scale, e = (x * x).mean(axis=axes), (d * d).mean(axis=axes)
            if not scale.all():
                continue   # zero: dq without a clean readout, dh0 behind a reset
            num[name] = num.get(name, 0) + (e / scale).mean() / seeds   # each head by its own size
    err = {name: math.sqrt(x) for name, x in num.items()}
    print(f"L={L}", {name: f"{x:.2e}" for name, x in err.items()}, flush=True)
    return err


@pytest.mark.parametrize("L", [2, 16, 32])
def test_seed_gradient_rounds_the_upstream_rows_once(L):
    """dh0 from the noisy readout under strong clean decays, s gamma~_n Q~^T dO~ and a part through the
    keys a few times smaller: one rounding, of the sum.  Scaling the rows in fp16 was a second one."""
    err = _errors(L, [-4.0] * 4, [None] * 4, False)
    assert err["dh0"] <= 1.2 * ONE


@pytest.mark.parametrize("L", [2, 16])
def test_noisy_blocks_in_a_chunk_round_once_per_factor(L):
    """dv from the noisy readout under strong clean decays, mostly the share of the noisy blocks of
    the same chunk (Q~ K^T)^T a: three roundings (the Gram entries, the sum, its part through the
    noisy keys' own) and smaller ones.  Rounding a = s gamma~_n dO~ to fp16 was a fourth."""
    err = _errors(L, [-4.0] * 4, [None] * 4, False)
    assert err["dv"] <= 1.9 * ONE


@pytest.mark.parametrize("L", [1, 4, 16, 32, 64])
def test_clean_dg_keeps_entries_of_the_decays_order(L):
    """dg at clean gates of -8, where every term is of order exp(-8): Delta, dDelta and R~ are rounded
    once each, and the terms' Gram entries not at all (in fp16 they were below its normal range)."""
    err = _errors(L, [-8.0] * 4, [None] * 4, True)
    assert err["dg"] <= 2.5 * ONE


@pytest.mark.parametrize("L", [4, 7, 32, 64])
def test_clean_dg_of_a_short_last_block(L):
    """The same with a last block of fewer positions than its padding (of 7 all are): the state
    gradient's term on the last position, of order one, would be added to a sum and taken off again."""
    err = _errors(L, [-8.0] * 4, [None] * 4, True, T=86, with_dht=True)
    assert err["dg"] <= 2.5 * ONE


@pytest.mark.parametrize("reset", [-1e4, -1e7])
@pytest.mark.parametrize("L", [1, 4, 16, 32, 64])
def test_a_gate_of_any_size_costs_the_others_nothing(L, reset):
    """One position in sixteen forgets everything, by whatever gate: the decays of the others come from
    differences of cumulative gates, in which the large one's rounding (0.5 at -1e7) must not stay."""
    err = _errors(L, [("single", reset)] * 2, [None, ("single", reset)], True)
    for name in ("dq", "dk", "dv", "dbeta", "dqn", "dkn", "dvn", "dbetan"):
        assert err[name] <= 4 * ONE, (name, err[name])
