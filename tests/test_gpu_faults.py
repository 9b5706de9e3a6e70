"""Failure handling forced from the host (msc_debug_inject): an allocation
or a HIP runtime call is made to report failure, every kernel still runs
and exits normally.  The failing call reports MSC_ENOMEM / MSC_EHIP, the
requests it touched fail alone, and the context and the queue go on to give
exact results."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2409_03771_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def msc():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_03771_amd import msc as m
    yield m
    m.debug_inject(m.INJECT_ENOMEM, -1)
    m.debug_inject(m.INJECT_EHIP, -1)


def _segment_raw(msc, ctx, t):
    outs = tuple(torch.empty(t.numel(), dtype=torch.int32, device="cuda")
                 for _ in range(3))
    dims = (ctypes.c_int64 * 3)(*msc.grid_dims(t.shape))
    rc = msc._lib.msc_segment(ctx, ctypes.c_void_p(t.data_ptr()), dims,
                              *(ctypes.c_void_p(o.data_ptr()) for o in outs),
                              None)
    return rc, outs


def test_allocation_failures(msc):
    f = synth.gaussian_field((45, 38, 30), 8, 81)
    t = torch.from_numpy(f).cuda()
    # Context creation.
    ctx = ctypes.c_void_p()
    msc.debug_inject(msc.INJECT_ENOMEM, 0)
    assert msc._lib.msc_create(ctypes.byref(ctx), 0) == msc.MSC_ENOMEM
    assert not ctx.value
    assert msc._lib.msc_create(ctypes.byref(ctx), 0) == msc.MSC_OK
    try:
        # The first call of a fresh context allocates its records and its
        # workspace: each failing allocation fails the call cleanly.
        for after in (0, 1, 2):
            msc.debug_inject(msc.INJECT_ENOMEM, after)
            rc, _ = _segment_raw(msc, ctx, t)
            msc.debug_inject(msc.INJECT_ENOMEM, -1)
            assert rc in (msc.MSC_OK, msc.MSC_ENOMEM), rc
        rc, outs = _segment_raw(msc, ctx, t)
        assert rc == msc.MSC_OK
        torch.cuda.synchronize()
        for name, g, w in zip(("asc", "desc", "ms"), outs, O.segment(f)):
            np.testing.assert_array_equal(g.cpu().numpy(), w, err_msg=name)
    finally:
        msc._lib.msc_destroy(ctx)
    # Queue creation.
    msc.debug_inject(msc.INJECT_ENOMEM, 0)
    with pytest.raises(msc.MscError) as e:
        msc.Server(hbm_budget=64 << 20, max_batch=4)
    assert e.value.code == msc.MSC_ENOMEM
    msc.debug_inject(msc.INJECT_ENOMEM, -1)


def test_runtime_failure_in_a_plain_call(msc):
    f = synth.gaussian_field((50, 41, 33), 8, 82)
    t = torch.from_numpy(f).cuda()
    msc.debug_inject(msc.INJECT_EHIP, 0)
    with pytest.raises(msc.MscError) as e:
        msc.segment(t)
    assert e.value.code == msc.MSC_EHIP
    msc.debug_inject(msc.INJECT_EHIP, -1)
    got = msc.segment(t)
    torch.cuda.synchronize()
    for name, g, w in zip(("asc", "desc", "ms"), got, O.segment(f)):
        np.testing.assert_array_equal(g.cpu().numpy(), w, err_msg=name)


@pytest.mark.parametrize("after", [1, 3, 9, 20])
def test_runtime_failure_in_the_queue(msc, after):
    """A runtime failure somewhere in the queue's threads (a copy, a launch)
    fails the requests it touched with MSC_EHIP; every other request is
    exact, and the queue serves new requests afterwards."""
    fields = [synth.gaussian_field((30 + i, 26, 21), 5, 90 + i)
              for i in range(8)]
    reqs = [(1, f) if i % 3 else (2, synth.threshold_mask(f, 0.6))
            for i, f in enumerate(fields)]
    with msc.Server(hbm_budget=256 << 20, max_batch=4) as srv:
        msc.debug_inject(msc.INJECT_EHIP, after)
        tickets = [srv.submit(k, a) for k, a in reqs]
        codes = [srv.wait(t) for t in tickets]
        # Disarmed before any result is copied back (the copy is a checked
        # call of this thread).
        msc.debug_inject(msc.INJECT_EHIP, -1)
        for t, (k, a), rc in zip(tickets, reqs, codes):
            assert rc in (msc.MSC_OK, msc.MSC_EHIP), rc
            if rc == msc.MSC_OK:
                got = srv.fetch(t)
                if k == 1:
                    for g, w in zip(got, O.segment(a)):
                        np.testing.assert_array_equal(g, w)
                else:
                    np.testing.assert_array_equal(got, O.cc_grid(a)[0])
            srv.release(t)
        assert msc.MSC_EHIP in codes
        for k, a in reqs[:3]:
            t = srv.submit(k, a)
            assert srv.wait(t) == msc.MSC_OK
            got = srv.fetch(t)
            if k == 1:
                for g, w in zip(got, O.segment(a)):
                    np.testing.assert_array_equal(g, w)
            else:
                np.testing.assert_array_equal(got, O.cc_grid(a)[0])
            srv.release(t)
        assert srv.info()["arena_used"] == 0


@pytest.mark.parametrize("kind,after", [
    (1, 1),    # the pair table's allocation, with the compression queued
    (2, 6),    # a runtime call after the kernels' launches
])
def test_csr_call_that_fails_leaves_nothing_running(msc, kind, after):
    """A CSR segmentation that fails between its passes returns with its
    stream drained, and a call on another stream, which carves the same
    memory, is exact."""
    n = 120
    d = synth.kuhn_csr(n, seed=3, nbumps=9, permute=False)
    rng = np.random.default_rng(2)
    big = [torch.from_numpy(a).cuda() for a in
           (d["row_ptr"], d["col_idx"],
            rng.permutation(n ** 3).astype(np.float32))]
    s = synth.kuhn_csr(24, seed=4, nbumps=6)
    f = np.empty_like(s["field"])
    f[s["perm"]] = s["field"]
    small = [torch.from_numpy(a).cuda() for a in
             (s["row_ptr"], s["col_idx"], f)]
    one, two = torch.cuda.Stream(), torch.cuda.Stream()

    def call(ctx, g, stream):
        outs = [torch.empty(g[2].numel(), dtype=torch.int32, device="cuda")
                for _ in range(3)]
        torch.cuda.synchronize()
        rc = msc._lib.msc_segment_csr(
            ctx, g[2].numel(), *(ctypes.c_void_p(t.data_ptr())
                                 for t in (*g, *outs)),
            ctypes.c_void_p(stream.cuda_stream))
        return rc, outs

    ctx = ctypes.c_void_p()
    assert msc._lib.msc_create(ctypes.byref(ctx), 0) == msc.MSC_OK
    try:
        msc.debug_inject(kind, after)
        rc, _ = call(ctx, big, one)
        idle = one.query()
        msc.debug_inject(kind, -1)
        assert rc == (msc.MSC_ENOMEM if kind == 1 else msc.MSC_EHIP)
        assert idle, "kernels of the failed call still run"
        rc, outs = call(ctx, small, two)
        assert rc == msc.MSC_OK
        torch.cuda.synchronize()
        for name, g, w in zip(("asc", "desc", "ms"), outs,
                              O.segment_csr(s["row_ptr"], s["col_idx"], f)):
            np.testing.assert_array_equal(g.cpu().numpy(), w, err_msg=name)
    finally:
        msc._lib.msc_destroy(ctx)


@pytest.mark.parametrize("X,Y,Z,ranks", [(513, 513, 33, 2), (513, 513, 50, 3)])
def test_slabs_of_a_rank_call_share_one_workspace(msc, X, Y, Z, ranks):
    """Slabs that cover different numbers of tile layers: the workspace is
    taken once for the thickest, never grown with an earlier slab's kernels
    queued on it (a second allocation would fail here)."""
    mask = synth.random_field((X, Y, Z), seed=X + Z) > 0.4
    t = torch.from_numpy(mask.astype(np.uint8)).cuda()
    want = msc.cc_label_grid(t)
    got = torch.empty(t.numel(), dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    dims = (ctypes.c_int64 * 3)(X, Y, Z)
    ctx = ctypes.c_void_p()
    assert msc._lib.msc_create(ctypes.byref(ctx), 0) == msc.MSC_OK
    try:
        msc.debug_inject(msc.INJECT_ENOMEM, 1)
        rc = msc._lib.cc_label_grid_ranks(
            ctx, ctypes.c_void_p(t.data_ptr()), dims, ranks,
            ctypes.c_void_p(got.data_ptr()), None)
        msc.debug_inject(msc.INJECT_ENOMEM, -1)
        assert rc == msc.MSC_OK
        assert torch.equal(got, want)
    finally:
        msc._lib.msc_destroy(ctx)
