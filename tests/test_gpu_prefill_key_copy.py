"""GPU: a prefill whose keys are seen by many row tiles rotates them once, into a copy
in the workspace.  Windows that start and end inside cache blocks, two segments that
share a block, positions outside the cos/sin table, both pairings and head sizes,
partial rotary width; more groups than the kernel arguments hold; the most segments a copy
has; a captured call; and the same calls with a workspace that ends before the copy."""
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


def was_copied(db, copy_bytes):
    """Whether a call writes the copy at the end of its workspace."""
    db.workspace.fill_(255)
    db.attend()
    torch.cuda.synchronize()
    return not bool((db.workspace[-copy_bytes:] == 255).all())


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
    assert was_copied(db, keys * 8 * D * 2)
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


def attend_both(db, wl, copy_bytes, rows=None):
    """The outputs with the copy and with a workspace that ends just before it."""
    out = []
    full = db.workspace
    for ws in (full, full[: full.numel() - copy_bytes]):
        db.workspace = ws
        db.o.fill_(float("nan"))
        db.attend()
        torch.cuda.synchronize()
        out.append(to_np(db.o))
    db.workspace = full
    return out


def test_key_copy_with_groups_in_the_workspace():
    # 66 short fresh documents between the cached ones and the tail: 67 groups go through the
    # workspace's table, and with them where each finds its keys in the copy
    from paper_2606_13126_amd import _binding as B
    from paper_2606_13126_amd.runner import DeviceBatch
    spans = [Sp(n, S) for n in (37, 1999, 705)] + [Sp(5, S | Q, fresh=True) for _ in range(66)]
    wl = W.small_case("key_copy_many", [spans + [Sp(208, Pd | Q, fresh=True)]], Hq=128, Hkv=8, D=128, theta=5e5,
                      dtype=torch.bfloat16, seed=100, value_scale=0.5)
    db = DeviceBatch(wl, table_positions=int(wl.positions.max()) + 1)
    shape = B.pic_plan_shape(db.cfg, db.host, False)
    assert shape["groups"] == 67 and shape["upload_launches"] == 1
    copy = -(-int(wl.seq_lens[0]) // 16) * 8 * 16 * 128 * 2
    before = shape["partial_slots"] * 256 * (128 + 2) * 4 + 67 * 48 + 4 * (shape["attention_blocks"] + shape["merge_blocks"])
    assert before + copy <= db.workspace.numel() <= before + copy + 4 * 256    # the copy comes last
    db.write()
    assert was_copied(db, copy)
    ref = WO.run(wl)
    for got, what in zip(attend_both(db, wl, copy), ("copy", "no copy")):
        assert_close(got, ref, wl.dtype, f"{wl.name} {what}")


@pytest.mark.parametrize("n,copied", [(64, True), (65, False)])
def test_key_copy_segments(n, copied):
    # documents that see themselves, apart from each other: a segment each, at most 64
    from paper_2606_13126_amd.runner import DeviceBatch
    spans = []
    for _ in range(n):
        spans += [Sp(3, S), Sp(208, S | Q, fresh=True)]
    wl = W.small_case(f"key_copy_{n}_segments", [spans], Hq=128, Hkv=8, D=64, theta=5e5, dtype=torch.bfloat16, seed=101,
                      value_scale=0.5)
    db = DeviceBatch(wl, table_positions=int(wl.positions.max()) + 1)
    at = [211 * i + 3 for i in range(n)]
    copy = sum((a + 207) // 16 - a // 16 + 1 for a in at) * 8 * 16 * 64 * 2
    assert (db.workspace.numel() >= copy) == copied
    db.write()
    assert not copied or was_copied(db, copy)
    rows = list(range(0, 208 * n, 499))
    ref = WO.run(wl, rows=rows)
    for got, what in zip(attend_both(db, wl, copy if copied else 0), ("copy", "no copy")):
        assert np.isfinite(got).all()
        assert_close(got[rows], ref, wl.dtype, f"{wl.name} {what}")


def test_key_copy_captured():
    from paper_2606_13126_amd.runner import DeviceBatch
    wl = case(128, 208, (37, 1999, 705))
    db = DeviceBatch(wl, table_positions=int(wl.positions.max()) + 1)
    db.write()
    assert was_copied(db, 4096)
    db.attend()
    torch.cuda.synchronize()
    ref = db.o.clone()
    g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            db.write()
            db.attend()
    for r in range(3):
        torch.cuda.synchronize()
        db.o.fill_(7.0)
        db.workspace.fill_(255)
        junk = torch.randn(1 << 20, device="cuda").sum()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        say(f"  replay {r}: junk={float(junk):.3f}")
        assert torch.equal(db.o.view(torch.int16), ref.view(torch.int16))


@pytest.mark.parametrize("table,copied", [(True, False), (False, True)])
def test_key_copy_of_many_short_items(table, copied):
    # 190 one-token documents beside the tail: 1,900 items, which the alternating kernel would
    # slow down by more than the copy saves, unless every item computed its cos/sin
    from paper_2606_13126_amd.runner import DeviceBatch
    spans = [Sp(n, S) for n in (37, 1999, 705)] + [Sp(1, S | Q, fresh=True) for _ in range(190)]
    wl = W.small_case("key_copy_short_items", [spans + [Sp(208, Pd | Q, fresh=True)]], Hq=128, Hkv=8, D=128, theta=5e5,
                      dtype=torch.bfloat16, seed=102, value_scale=0.5)
    db = DeviceBatch(wl, table_positions=int(wl.positions.max()) + 1 if table else None)
    copy = -(-int(wl.seq_lens[0]) // 16) * 8 * 16 * 128 * 2
    assert db.workspace.numel() > copy
    db.write()
    assert was_copied(db, copy) == copied
    rows = list(range(0, 190, 9)) + list(range(190, 398, 7))
    assert_close(to_np(db.o)[rows], WO.run(wl, rows=rows), wl.dtype, f"{wl.name} table={table}")
