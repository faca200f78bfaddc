"""Full forward pass of at most 32 samples: the product kernel with 16 rows of W per workgroup, at the edges of its sample
tiles (1, 15, 16, 17, 31, 32; 33 is beyond it), of its neuron tiles and of the waves' shares of k, against 64-bit sums over
the same stored values."""
import pytest
import torch

from paper_1910_02120_amd import ISTContext

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B", [1, 15, 16, 17, 31, 32, 33])
# rows of W: the shortest the kernel takes, one piece less, a remainder of a stage, one piece into a third stage; widths
# that 16 divides and not, fewer classes than a tile
@pytest.mark.parametrize("K,N,classes", [(1024, 1016, 5), (1016, 1040, 16), (2056, 1048, 17), (4104, 2008, 101)])
def test_logits_against_64_bit_sums(dtype, B, K, N, classes):
    td, u = (torch.float32, 2.0 ** -24) if dtype == "f32" else (torch.bfloat16, 2.0 ** -9)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(B * 7919 + K)
    W = [(torch.randn((o, i), generator=g, device="cuda:0") / i ** 0.5).to(td) for i, o in ((K, N), (N, classes))]
    b = [torch.randn(o, generator=g, device="cuda:0").to(td) for o in (N, classes)]
    X = torch.randn((B, K), generator=g, device="cuda:0").to(td)
    ctx = ISTContext([K, N, classes], 2, dtype, "dense", True, max_B=B, device="cuda:0", bind=False)
    got = torch.full((B, classes), float("nan"), dtype=torch.float32, device="cuda:0")
    ctx.forward_full(W, b, B, X=X, logits=got, static=True)
    torch.cuda.synchronize()
    Wd, bd, Xd = [w.double().cpu() for w in W], [v.double().cpu() for v in b], X.double().cpu()
    h = (Xd @ Wd[0].T + bd[0]).clamp(min=0.0)
    want = h @ Wd[1].T + bd[1]
    # worst case of both sums in fp32 ((terms + 1) roundings each) and of storing the hidden layer in the storage type
    e32 = 2.0 ** -24
    eh = (K + 1) * e32 * (Xd.abs() @ Wd[0].abs().T + bd[0].abs())
    eh = eh + u * (h + eh)
    bound = eh @ Wd[1].abs().T + (N + 1) * e32 * ((h + eh) @ Wd[1].abs().T + bd[1].abs())
    assert bool(((got.double().cpu() - want).abs() <= bound).all())
    ctx.close()
