"""The forms of the layout transform in: a thread per site (up to two workgroups
per CU, 512 pairs of a block and a right-hand side on the card), through LDS, and
through LDS past the caches (input and output over 256 MB), on both sides of
each line, bit for bit against the transform's definition."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def blocked(canon, dims):
    """(n, V, 12) -> the blocked layout, flat (torch)."""
    lx, ly, lz, lt = dims
    n = canon.shape[0]
    v = canon.reshape(n, lt // 4, 4, lz // 4, 4, ly // 4, 4, lx // 4, 4, 12)
    return v.permute(1, 3, 5, 7, 0, 9, 2, 4, 6, 8).contiguous().reshape(-1)


@pytest.mark.parametrize("dims,prec,nrhs", [
    ((16, 16, 16, 32), "f64", 1), ((16, 16, 16, 32), "f32", 1), ((16, 16, 16, 32), "f16", 1),  # 512 pairs
    ((16, 16, 16, 40), "f64", 1), ((16, 16, 16, 40), "f32", 1), ((16, 16, 16, 40), "f16", 1),  # 640
    ((4, 16, 24, 48), "f64", 9), ((4, 16, 24, 48), "f64", 10),  # 255 and 283 MB
    ((4, 16, 24, 48), "f32", 12), ((4, 16, 24, 48), "f32", 13),
    ((4, 16, 24, 48), "f16", 15), ((4, 16, 24, 48), "f16", 16),
])
def test_pack_forms(dims, prec, nrhs):
    import torch
    from paper_1710_07041_amd import ddsap
    ctx = ddsap.Context(dims)
    scalar = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}[prec]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    # exact in every precision: what is tested is where each number goes
    x = torch.randint(-1024, 1025, (nrhs, int(np.prod(dims)), 12, 2), generator=gen, device="cuda").to(torch.float64)
    canon = torch.view_as_complex(x).contiguous()
    out = ctx.empty_blocked(prec, nrhs)
    ctx.pack(canon, out, prec, nrhs)
    ctx.synchronize()
    want = torch.view_as_real(blocked(canon, dims)).reshape(-1).to(scalar)
    assert torch.equal(out.view(scalar)[: want.numel()], want)
