"""GPU: decode at the edges of its split policy (chunks of four cache blocks) and of the
three forms of its merge (up to 8 splits, up to 64, more)."""
import pytest
import torch

import workloads as W
from oracle import workload_oracle as WO
from tests.gpu_util import assert_close, gpu_run, to_np

pytestmark = pytest.mark.gpu

S, Pd, Sp = W.SSEP, W.PDEP, W.Span


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_13126_amd  # noqa: F401  (fails loudly if the library is missing)


@pytest.mark.parametrize("Hq,Hkv,D,lens", [
    (8, 2, 128, [32]),             # 33 keys: three cache blocks, unsplit
    (8, 8, 64, [255]),             # 16 blocks: four splits
    (4, 1, 128, [256, 5]),         # 17 blocks: five splits of up to four blocks, and one request unsplit
    (8, 8, 64, [511]),             # 32 blocks: eight splits, merged by one thread row
    (4, 1, 128, [512, 5]),         # 33 blocks: nine splits, eight thread rows
    (32, 8, 128, [2047]),          # 128 blocks: 32 splits
    (8, 2, 64, [2048, 300]),       # 129 and 19 blocks: 33 and 5 splits
    (32, 8, 128, [4095]),          # 256 blocks: 64 splits
    (28, 4, 128, [4096, 40]),      # 257 blocks: 65 splits, thirty-two thread rows
    (12, 12, 64, [6000]),          # 94 splits of heads that fill two workgroups
    (28, 4, 128, [9000, 700, 150, 40]),   # thirty-two, eight and one thread row in one launch
    (40, 8, 64, [900, 200]),       # eight and one, the last block of one half empty
])
def test_decode_split_and_merge_edges(Hq, Hkv, D, lens):
    # the partials and their sums are float32 in every form: the tolerance of any bf16 decode
    reqs = [[Sp(n, S), Sp(1, Pd, fresh=True)] for n in lens]
    wl = W.build(f"decode_merge_{Hq}_{Hkv}_{D}_{lens[0]}", reqs, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=D, rope_theta=5e5,
                 dtype=torch.bfloat16, seed=93, value_scale=0.5, num_blocks=sum(lens) // 16 + 3 * len(lens) + 16, decode=True)
    db = gpu_run(wl)
    ref = WO.run(wl)
    assert_close(to_np(db.o), ref, wl.dtype, wl.name)
    if lens[0] < 256 and D == 128:
        # an unsplit call needs no workspace
        db.workspace = None
        db.o.fill_(float("nan"))
        db.attend()
        torch.cuda.synchronize()
        assert_close(to_np(db.o), ref, wl.dtype, wl.name + " without workspace")


def test_decode_merge_without_room_for_its_map():
    # 66 requests: their merge map travels through the workspace.  One that ends before the
    # wider merge's entries is accepted, with one thread row per query head
    from paper_2606_13126_amd import _binding as B
    lens = [70] * 65 + [3200]
    wl = W.build("decode_merge_map", [[Sp(n, S), Sp(1, Pd, fresh=True)] for n in lens], num_q_heads=32, num_kv_heads=8,
                 head_dim=64, rope_theta=5e5, dtype=torch.bfloat16, seed=94, value_scale=0.5,
                 num_blocks=sum(lens) // 16 + 3 * len(lens) + 16, decode=True)
    db = gpu_run(wl)
    shape = B.pic_plan_shape(db.cfg, db.host, True)
    assert shape["upload_launches"] == 1 and shape["merge_blocks"] == 65 * 4 + 32
    ref = WO.run(wl)
    assert_close(to_np(db.o), ref, wl.dtype, wl.name)
    db.workspace = db.workspace[:-64]
    db.o.fill_(float("nan"))
    db.attend()
    torch.cuda.synchronize()
    assert_close(to_np(db.o), ref, wl.dtype, wl.name + " one row per head")
