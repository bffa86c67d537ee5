"""The entry point that allocates nothing (pic_attn_decode_noalloc) against
pic_attn_decode with a caller workspace: same kernels, so the outputs must agree
bit for bit, on two calls in a row (the second with a smaller batch that reuses the
library's scratch), and both within the oracle tolerance."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W
from oracle import workload_oracle as WO
from tests.cases import many_requests_decode
from tests.gpu_util import assert_close, say, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_13126_amd  # noqa: F401  (fails loudly if the library is missing)


def _noalloc(db):
    """Call the C entry point through ctypes with the batch of a DeviceBatch."""
    from paper_2606_13126_amd import _binding as B
    lib = B.lib()
    dev = B._dev(db.block_tables, db.positions)
    rope = B._rope(db.table)
    rc = lib.pic_attn_decode_noalloc(ctypes.byref(db.cfg), ctypes.byref(db.host.c), ctypes.byref(dev),
                                     ctypes.byref(rope), db.q.data_ptr(), db.o.data_ptr(), db.k_pool.data_ptr(),
                                     db.v_pool.data_ptr(), int(db.k_pool.shape[0]),
                                     torch.cuda.current_stream().cuda_stream)
    assert rc == B.PIC_OK, lib.pic_last_error().decode()


def _case(wl):
    from paper_2606_13126_amd.runner import DeviceBatch
    db = DeviceBatch(wl, table_positions=int(wl.positions.max()) + 1)
    db.write()
    db.attend()                     # pic_attn_decode with its own workspace
    torch.cuda.synchronize()
    ref = db.o.clone()
    db.o.fill_(float("nan"))
    _noalloc(db)
    torch.cuda.synchronize()
    return db, ref


def test_noalloc_decode_matches_workspace_decode_two_calls():
    # first call: 64 requests of 8193 keys (4 key splits each: the scratch holds the
    # split partials); second call: a smaller batch of 256 short requests, whose group
    # table also goes through the scratch, reading what the first call left there
    first = W.decode_64req()
    second = many_requests_decode(num_reqs=96)
    for wl in (first, second):
        say(f"[gpu] noalloc decode {wl.name}: {wl.num_reqs} requests, {int(wl.seq_lens.sum())} keys")
        db, ref = _case(wl)
        assert torch.equal(db.o.view(torch.int16), ref.view(torch.int16)), wl.name
        assert_close(to_np(db.o), WO.run(wl), wl.dtype, f"noalloc {wl.name} vs oracle")
        del db
        torch.cuda.empty_cache()


@pytest.mark.parametrize("lens", [[1500, 90], [40] * 64 + [700, 1500]])
def test_noalloc_decode_float32(lens):
    # the key splits' partials live in the scratch, for more than 64 requests after the
    # previous call's and beside the group table
    S, Pd, Sp = W.SSEP, W.PDEP, W.Span
    wl = W.build(f"noalloc_f32_{len(lens)}", [[Sp(n, S), Sp(1, Pd, fresh=True)] for n in lens], num_q_heads=8, num_kv_heads=2,
                 head_dim=128, rope_theta=1e4, dtype=torch.float32, seed=99, num_blocks=sum(lens) // 16 + 4 * len(lens) + 16,
                 decode=True)
    say(f"[gpu] noalloc float32 decode of {len(lens)} requests")
    db, ref = _case(wl)
    assert torch.equal(db.o.view(torch.int32), ref.view(torch.int32))
    assert_close(to_np(db.o), WO.run(wl), wl.dtype, f"{wl.name} vs oracle")


def test_noalloc_decode_narrow_workgroups():
    # models with one or two KV heads decode with 2- and 4-wave workgroups (three or
    # two per CU, more key splits): the scratch holds their partials too
    for hq, hkv in ((32, 1), (64, 2)):
        wl = many_requests_decode(num_reqs=64, Hq=hq, Hkv=hkv, D=128)
        say(f"[gpu] noalloc decode Hq={hq} Hkv={hkv}: {wl.num_reqs} requests, {int(wl.seq_lens.sum())} keys")
        db, ref = _case(wl)
        assert torch.equal(db.o.view(torch.int16), ref.view(torch.int16)), (hq, hkv)
        assert_close(to_np(db.o), WO.run(wl), wl.dtype, f"noalloc Hq={hq} Hkv={hkv} vs oracle")
        del db
        torch.cuda.empty_cache()
