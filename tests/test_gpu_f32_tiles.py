"""GPU: the float32 kernel at the edges of its tiles (16 query rows per wave, 64 per
workgroup, 16- and 32-key tiles, 128-key splits), with and without room for split
partials, with the groups in the kernel arguments and in the workspace, and with
infinities that only some rows see."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import workload_oracle as WO
from tests.gpu_util import assert_close, gpu_run, say, to_np

pytestmark = pytest.mark.gpu

S, Pd, Q, Sp = W.SSEP, W.PDEP, W.QUERY, W.Span


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_13126_amd  # noqa: F401  (fails loudly if the library is missing)


@pytest.mark.parametrize("Hq,Hkv,D,cached,fresh,style", [
    (4, 1, 128, 0, 4, 0),      # 16 rows: one-wave workgroups, one partial 16-key tile
    (4, 1, 128, 112, 17, 1),   # 68 rows: a second row tile of four rows; 129 keys: two splits
    (2, 2, 64, 96, 32, 0),     # 32 rows, 128 keys: one split exactly
    (8, 2, 64, 480, 33, 1),    # 132 rows, 513 keys: splits whose last tile holds one key
    (3, 3, 128, 16, 1, 0),     # one row per KV head, 17 keys: two 16-key tiles
    (16, 1, 64, 240, 9, 0),    # 144 rows of one KV head, three row tiles
])
def test_f32_tile_edges(Hq, Hkv, D, cached, fresh, style):
    spans = ([Sp(cached, S, key="a")] if cached else []) + [Sp(fresh, Pd | Q, fresh=True)]
    wl = W.small_case(f"f32_{Hq}_{Hkv}_{D}_{cached}_{fresh}", [spans], Hq=Hq, Hkv=Hkv, D=D, dtype=torch.float32, seed=91)
    db = gpu_run(wl, rope_style=style)
    ref = WO.run(wl, style="neox" if style == 0 else "gptj")
    assert_close(to_np(db.o), ref, wl.dtype, wl.name)
    # a workspace without room for partials is accepted: the keys stay unsplit
    db.workspace = None
    db.o.fill_(float("nan"))
    db.attend()
    torch.cuda.synchronize()
    assert_close(to_np(db.o), ref, wl.dtype, wl.name + " without workspace")


@pytest.mark.parametrize("decode", [False, True])
def test_f32_splits_of_many_groups(decode):
    # 66 requests: groups and merge map travel through the workspace, beside the partials
    from paper_2606_13126_amd import _binding as B
    lens = [40] * 64 + [700, 1500]
    reqs = [[Sp(n, S), Sp(1, Pd, fresh=True) if decode else Sp(3 + 20 * (n > 600), Pd | Q, fresh=True)] for n in lens]
    wl = W.build(f"f32_many_{decode}", reqs, num_q_heads=6, num_kv_heads=2, head_dim=64, rope_theta=1e4, dtype=torch.float32,
                 seed=98, num_blocks=sum(lens) // 16 + 4 * len(lens) + 16, decode=decode)
    db = gpu_run(wl, rope_style=1)
    shape = B.pic_plan_shape(db.cfg, db.host, decode)
    assert shape["upload_launches"] == 1 and shape["merge_blocks"] > 0
    ref = WO.run(wl, style="gptj")
    assert_close(to_np(db.o), ref, wl.dtype, wl.name)
    # room for the table and the attention map alone: unsplit
    db.workspace = db.workspace[:66 * 48 + 256 + 4 * 1024]
    db.o.fill_(float("nan"))
    db.attend()
    torch.cuda.synchronize()
    assert_close(to_np(db.o), ref, wl.dtype, wl.name + " unsplit")


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("at", [16, 40, 63])
def test_f32_non_finite_values_reach_only_rows_that_see_them(bad, at):
    # the value row of token `at` of a 70-token causal span: earlier tokens stay finite
    # and unchanged (a probability of zero times infinity must not reach them)
    wl = W.small_case("f32_bad", [[Sp(70, S | Q, fresh=True)]], Hq=4, Hkv=2, D=64, dtype=torch.float32, seed=92)
    clean = gpu_run(wl).o.clone()
    wl.v_new[at, :, 5] = bad
    got = gpu_run(wl).o
    say(f"[gpu] f32 V row {at} = {bad}")
    assert torch.equal(got[:at], clean[:at])
    assert not torch.isfinite(got[at:, :, 5]).any()
    keep = np.arange(64) != 5
    assert torch.allclose(got[at:][..., keep], clean[at:][..., keep], rtol=0, atol=1e-5)
