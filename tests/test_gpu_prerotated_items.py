"""GPU: prefill over rotated keys on both sides of the rule that picks its kernel (items of
few key tiles or few rows against longer ones), with ragged windows and last tiles.  All
positions are 0, so that the rotation is the identity."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import workload_oracle as WO
from tests.gpu_util import assert_close, to_np

pytestmark = pytest.mark.gpu

S, Pd, Q, Sp = W.SSEP, W.PDEP, W.QUERY, W.Span


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_13126_amd  # noqa: F401  (fails loudly if the library is missing)


@pytest.mark.parametrize("Hq,Hkv,D,docs,tail,n,short", [
    (32, 8, 128, (21, 170), 64, 32, True),      # 255 keys, four tiles for each of 256 items (unsplit)
    (32, 8, 128, (21, 172), 64, 32, False),     # 257 keys, five tiles, one key in the last
    (8, 2, 128, (1,), 33, 2, True),             # 132 rows, one tile
    (12, 12, 128, (37, 300), 64, 22, True),     # seven tiles, but 64 rows
    (12, 12, 128, (37, 300), 129, 22, False),   # 129 rows, eight tiles
    (32, 8, 64, (50, 333), 64, 32, True),       # 447 keys, seven tiles: short at D = 64
    (32, 8, 64, (50, 335), 64, 32, False),      # 449 keys, eight
    (32, 8, 128, (2800,), 250, 1, False),       # splits of six tiles
    (16, 4, 64, (7,), 300, 2, True),            # causal row tiles of one to five tiles
])
@pytest.mark.parametrize("style", [0, 1])
def test_prerotated_prefill_items(Hq, Hkv, D, docs, tail, n, short, style):
    from paper_2606_13126_amd import _binding as B
    from paper_2606_13126_amd.runner import DeviceBatch
    # the same number of keys from the start of the request, and from inside a cache block
    # (a tail that keeps its document's window)
    reqs = [[Sp(n, S) for n in docs] + [Sp(tail, Pd | Q, fresh=True)], [Sp(21, S), Sp(sum(docs), S), Sp(tail, Q, fresh=True)]]
    reqs = [reqs[i % 2] for i in range(n)]
    wl = W.small_case(f"prerotated_{Hq}_{D}_{sum(docs)}_{tail}", reqs, Hq=Hq, Hkv=Hkv, D=D, dtype=torch.bfloat16, seed=96,
                      value_scale=0.5)
    wl.positions = np.zeros_like(wl.positions)
    db = DeviceBatch(wl, rope_style=style, k_prerotated=True, table_positions=None)
    items = B.pic_plan_debug(db.cfg, db.host, False)
    tiles = sum((int(i[5]) - int(i[4]) + 63) // 64 for i in items if i[3] - i[2] > 128)
    assert (tiles < len(items) * (5 if D == 128 else 8)) == short
    db.write()
    db.o.fill_(float("nan"))
    db.attend()
    torch.cuda.synchronize()
    assert_close(to_np(db.o), WO.run(wl), wl.dtype, f"{wl.name} style={style}")
