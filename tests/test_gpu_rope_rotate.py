"""GPU: pic_rope_rotate rounds as (x c - (y s), x s + (y c)) with the bracketed product
rounded to float32 first, whatever the size of the call (the pairs per thread follow it),
the pairing and the rotary width."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_13126_amd  # noqa: F401  (fails loudly if the library is missing)


@pytest.mark.parametrize("n,heads,D", [(1, 3, 64), (33, 8, 128), (256, 16, 128), (257, 16, 128), (1500, 9, 64)])
@pytest.mark.parametrize("style,rotary", [(0, 0), (1, 0), (1, 30), (0, 32), (1, 2)])
@pytest.mark.parametrize("f32", [False, True])
def test_rotate_rounding(n, heads, D, style, rotary, f32):
    import paper_2606_13126_amd as P
    dt = torch.float32 if f32 else torch.bfloat16
    cfg = P.make_config(heads, heads, D, dtype=P.PIC_F32 if f32 else P.PIC_BF16, rope_style=style, rotary_dim=rotary, rope_theta=5e5)
    tab = torch.empty((n, D // 2, 2) if f32 else (n, D // 2), dtype=torch.float32, device="cuda")
    P.pic_rope_table_build(cfg, tab)
    gen = torch.Generator().manual_seed(97)
    x = torch.randn((n, heads, D), generator=gen).to(dt)
    pos = torch.randperm(n, generator=gen).to(torch.int32)
    got = x.cuda()
    P.pic_rope_rotate(cfg, got, pos.cuda(), table=tab)
    torch.cuda.synchronize()
    cs = tab.cpu() if f32 else tab.cpu().view(torch.bfloat16).view(n, D // 2, 2)
    cs = cs.double().numpy()[pos.numpy()][:, None, :, :]
    r = rotary or D
    c, s = cs[..., : r // 2, 0], cs[..., : r // 2, 1]
    xd = x.double().numpy()
    a, b = (xd[..., : r // 2], xd[..., r // 2:r]) if style == 0 else (xd[..., 0:r:2], xd[..., 1:r:2])
    lo = (a * c - (b * s).astype(np.float32)).astype(np.float32)
    hi = (a * s + (b * c).astype(np.float32)).astype(np.float32)
    want = x.float().numpy().copy()
    if style == 0:
        want[..., : r // 2], want[..., r // 2:r] = lo, hi
    else:
        want[..., 0:r:2], want[..., 1:r:2] = lo, hi
    want = torch.from_numpy(want).to(dt)
    differ = int((got.cpu() != want).sum())
    # the 64-bit sum here rounds twice: it may differ from the fused one once in 2^29 values
    assert differ <= (1 if f32 else 0), differ
