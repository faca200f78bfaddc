"""Networks whose subnets fit the LDS of one compute unit (all local steps in one launch) against the oracle, at the edges
of that kernel's tiles: batches and widths around its 16-row tiles and 16 / 32-deep k-steps, two to eight layers, one sample,
one class, more than 64 and more than 256 classes, mini-batches longer than what a wave holds ahead in registers, no
biases, layer factors, a batch below the context's largest, more steps than one row-loss reduction of the other path."""
import pytest

import ist_inputs as gen

import ist_harness as H

pytestmark = pytest.mark.gpu
C = gen.CONFIGS

CASES = {   # name: (dtype, dims, S, B, k, bias, scale)
    "edges-16": ("f32", (16, 32, 32, 16), 2, 16, 2, True, None),
    "edges-17": ("f32", (17, 34, 66, 17), 2, 17, 2, True, None),
    "edges-bf16-32": ("bf16", (32, 64, 64, 32), 2, 32, 2, True, None),
    "edges-bf16-33": ("bf16", (33, 66, 130, 33), 2, 33, 2, True, None),
    "one-sample": ("f32", (20, 48, 6), 3, 1, 2, True, None),
    "one-hidden-wide-out": ("bf16", (12, 60, 257), 4, 30, 2, True, None),
    "classes-65-nobias": ("f32", (15, 51, 65), 3, 40, 3, False, None),
    "long-batch": ("f32", (40, 32, 3), 4, 260, 2, True, None),          # 260 pieces of 64 values, 128 held ahead
    "wide-input": ("bf16", (601, 45, 21, 9), 3, 60, 2, True, None),     # 10 pieces per sample
    "eight-layers": ("f32", (12, 32, 24, 40, 32, 24, 32, 40, 7), 2, 9, 2, True, None),
    "factors": ("f32", (30, 40, 60, 11), 2, 25, 2, True, (1.0, 4.0, 2.0)),
    "many-steps": ("bf16", (24, 40, 10), 2, 21, 35, True, None),
}


@pytest.mark.parametrize("name", list(CASES))
def test_small_network_matches_oracle(name):
    dtype, dims, S, B, k, bias, scale = CASES[name]
    cfg = gen.scaled(C["cfg3" if dtype == "bf16" else "cfg2"], name=name, dims=dims, S=S, B=B, k=k, lr=0.05, dtype=dtype,
                     init_gain=1.5 if len(dims) > 5 else 1.0)
    P = H.Problem(cfg, has_bias=bias, dev="cuda:0", **({} if scale is None else {"scale": scale}))
    ctx = P.context()
    ctx.partition(P.dW, P.db, P.dperm)
    ctx.profile_enable(True)
    H.check_training(P, ctx)
    labels = {r["label"] for r in ctx.profile_kernels()}
    ctx.profile_enable(False)
    assert any(s.startswith("k_small_steps") for s in labels), labels   # the shape does take the kernel under test
    ctx.close()
