"""Partition, merge and re-sampling bit for bit against the oracle where the shared copy launch and the index tables have
their edges: rows of several 4096-column pieces with ragged ends, blocks of unequal width, a hidden layer wider than one
window of the table kernel (262144 ids), more subnets than one level of the bias mean, a last layer with rows enough for a
launch of its own, a large bf16 middle layer, more layers than one launch takes."""
import numpy as np
import pytest
import torch

import ist_inputs as gen
from oracle import ist_oracle as orc

import ist_harness as H

pytestmark = pytest.mark.gpu
C = gen.CONFIGS

CASES = {   # name: (dtype, dims, S)
    "pieces-f32": ("f32", (5, 9001, 4099, 3), 3),
    "pieces-bf16": ("bf16", (4100, 4104, 8200, 12), 8),
    "odd-bf16": ("bf16", (7, 4097, 515, 9), 5),
    "window-f32": ("f32", (3, 300001, 2), 2),
    "many-subnets-bf16": ("bf16", (6, 150, 77, 5), 70),
    "tall-last-f32": ("f32", (4, 48, 4500), 4),
    "tall-last-uneven-bf16": ("bf16", (4, 51, 4200), 7),
    "tall-last-uneven-aligned-f32": ("f32", (4, 52, 4200), 7),
    "large-middle-bf16": ("bf16", (8, 8192, 4096, 4), 4),
    "many-layers-f32": ("f32", (9,) + (24, 17) * 5 + (3,), 3),
}


@pytest.mark.parametrize("name", list(CASES))
def test_copies_match_oracle_bit_for_bit(name):
    dtype, dims, S = CASES[name]
    cfg = gen.scaled(C["cfg3" if dtype == "bf16" else "cfg2"], name=name, dims=dims, S=S, B=2, k=1, dtype=dtype)
    P = H.Problem(cfg, dev="cuda:0")
    ctx = P.context()
    ctx.set_checked(True)
    W, b = [w.clone() for w in P.dW], [x.clone() for x in P.db]
    full_W = [H.np_bits(w, dtype).copy() for w in P.Ws]
    full_b = [H.np_bits(x, dtype).copy() for x in P.bs]
    ctx.partition(W, b, P.dperm)
    perms = P.perms
    for rnd in (1, 2):
        subs = H.export_all(ctx, cfg)
        want = orc.partition(full_W, full_b, perms, S)
        for s in range(S):
            for l in range(cfg.t):
                assert np.array_equal(H.bits(subs[s][0][l]), want[s][0][l]), (name, rnd, s, l)
                assert np.array_equal(H.bits(subs[s][1][l]), want[s][1][l]), (name, rnd, s, l, "bias")
        # what the subnets do not own must keep its bits, what they own must return: into poisoned matrices
        poison = [torch.full_like(w, 7.0) for w in W]
        pb = [torch.full_like(x, 7.0) for x in b]
        ctx.merge(poison, pb)
        torch.cuda.synchronize()
        seven = H.np_bits(np.float32([7.0]), dtype)[0]
        expect = [np.full(w.shape, seven, dtype=full_W[0].dtype) for w in full_W]
        orc.merge(expect, None, perms, S, want)
        for l in range(cfg.t):
            assert np.array_equal(H.bits(poison[l]), expect[l]), (name, rnd, l, "merge")
            if l < cfg.t - 1:
                assert np.array_equal(H.bits(pb[l]), full_b[l]), (name, rnd, l, "bias")
        # merging untouched subnets and cutting by the next permutation leaves W as it is (the mean of S equal output
        # biases may differ in the last bit when S is no power of two)
        perms = gen.make_perms(cfg, rnd)
        ctx.resample(W, b, [torch.from_numpy(p).to("cuda:0") for p in perms])
        torch.cuda.synchronize()
        for l in range(cfg.t):
            assert np.array_equal(H.bits(W[l]), full_W[l]), (name, rnd, l, "re-sampling")
        full_b[-1] = H.bits(b[-1]).copy()
    ctx.close()
