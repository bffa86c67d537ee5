"""GPU: a prefill whose keys are seen by many row tiles rotates them once, into a copy
in the workspace.  Windows that start and end inside cache blocks, two segments that
share a block, positions outside the cos/sin table, both pairings and head sizes,
partial rotary width; and the same call with a workspace that ends before the copy."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import workload_oracle as WO
from tests.gpu_util import assert_close, say, to_np

pytestmark = pytest.mark.gpu

S, Pd, Q, Sp = W.SSEP, W.PDEP, W.QUERY, W.Span


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_13126_amd  # noqa: F401  (fails loudly if the library is missing)


def case(D, tail, docs):
    # request 0: cached documents of odd lengths and a tail over all of them (one
    # segment); request 1: detached query spans in one block with an unqueried span
    # between them (segments that share a cache block), nothing else visible
    reqs = [[Sp(n, S) for n in docs] + [Sp(tail, Pd | Q, fresh=True)],
            [Sp(21, S), Sp(70, S | Q, fresh=True), Sp(3, S), Sp(65, S | Q, fresh=True), Sp(64, S)]]
    return W.small_case(f"key_copy_d{D}", reqs, Hq=128, Hkv=8, D=D, theta=5e5, dtype=torch.bfloat16, seed=95,
                        value_scale=0.5, position_offsets=[0, 7000])


@pytest.mark.parametrize("D,style,tail,docs,table_len,rotary", [
    (128, 0, 208, (37, 1999, 705), None, None),   # 2,949 keys: the last key tile holds five
    (128, 1, 201, (1024, 1024, 1024), 1500, None),  # half of the positions outside the table
    (64, 0, 240, (511, 2050), 0, None),           # computed cos/sin
    (64, 1, 208, (37, 1999, 705), None, 30),
    (128, 0, 225, (16, 2736), None, 64),          # partial rotary: chunks in kernel order
])
def test_key_copy(D, style, tail, docs, table_len, rotary):
    from paper_2606_13126_amd import _binding as B
    from paper_2606_13126_amd.runner import DeviceBatch
    wl = case(D, tail, docs)
    wl.rotary_dim = rotary
    n_tab = None if table_len == 0 else table_len or int(wl.positions.max()) + 1
    db = DeviceBatch(wl, rope_style=style, table_positions=n_tab)
    shape = B.pic_plan_shape(db.cfg, db.host, False)
    need = shape["partial_slots"] * 256 * (D + 2) * 4
    assert shape["upload_launches"] == 0
    keys = sum(docs) + tail
    size = db.workspace.numel()
    say(f"[gpu] key copy D={D} style={style}: workspace {size}, partials {need}, {keys} keys in request 0")
    assert size >= need + keys * 8 * D * 2          # the copy is planned
    db.write()
    db.attend()
    torch.cuda.synchronize()
    ref = WO.run(wl, style="neox" if style == 0 else "gptj")
    assert_close(to_np(db.o), ref, wl.dtype, f"key copy D={D} style={style} rotary={rotary}")
    # a workspace with room for the partials alone is accepted: rotation in the kernel
    db.workspace = db.workspace[:need]
    db.o.fill_(float("nan"))
    db.attend()
    torch.cuda.synchronize()
    assert_close(to_np(db.o), ref, wl.dtype, f"no key copy D={D} style={style} rotary={rotary}")


def test_key_copy_reads_no_key_outside_the_windows():
    # keys and values that no query sees are NaN: in the pool they reach neither the
    # copy's visible rows nor the outputs
    from paper_2606_13126_amd.runner import DeviceBatch
    wl = case(128, 208, (37, 1999, 705))
    ref = WO.run(wl)
    unseen = list(range(0, 21)) + list(range(91, 94)) + list(range(159, 223))
    for t in unseen:
        b = int(wl.block_tables[1, t // 16])
        wl.k_pool[b, :, t % 16] = float("nan")
        wl.v_pool[b, :, t % 16] = float("nan")
    db = DeviceBatch(wl, table_positions=int(wl.positions.max()) + 1)
    db.workspace.view(torch.uint8).fill_(255)       # NaN wherever nothing is written
    db.write()
    db.attend()
    torch.cuda.synchronize()
    assert_close(to_np(db.o), ref, wl.dtype, "key copy with NaN outside the windows")
