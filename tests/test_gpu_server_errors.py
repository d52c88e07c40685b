"""Requests of a batch that could not be started stay in the server's queue.
The error is one an earlier HIP call of the program left behind (a hipMalloc
without an output pointer): the batch call reports it, and a later poll runs
the batch."""
import ctypes as C
import time

import numpy as np
import pytest

from paper_2512_10386_amd import synth

pytestmark = pytest.mark.gpu


def test_requests_wait_after_a_failed_poll():
    import torch
    from paper_2512_10386_amd import binding as B
    from paper_2512_10386_amd.serve import Server
    prm = dict(k=16, leaf_cap=256)
    frames = [torch.from_numpy(synth.sphere_plane(seed=s, n_sphere=3000, n_plane=900, n_out=600)[0]).cuda()
              for s in (1, 2, 3)]
    torch.cuda.synchronize()
    den = B.Denoiser(0, **prm)
    srv = Server(0, hbm_budget=1 << 30, max_slots=1, slot_points=10_000, slot_frames=2, **prm)
    try:
        outs = [srv.alloc(len(f)) for f in frames]
        left = {srv.submit(f, o) for f, o in zip(frames, outs)}
        # the HIP runtime the library is linked with
        hip = C.CDLL(B.LIB_PATH)
        assert hip.hipMalloc(None, C.c_size_t(16)) != 0
        failed = 0
        t0 = time.time()
        while left:
            assert time.time() - t0 < 20.0, f"tickets {sorted(left)} never finish"
            try:
                left.difference_update(srv.poll()[0])
            except B.GdnError as e:
                assert e.status == B.GDN_EHIP
                failed += 1
        print("[server] failed polls:", failed, flush=True)
        torch.cuda.synchronize()
        for f, o in zip(frames, outs):
            ref = den(f)
            assert torch.equal(o.keep[:len(f)], ref.keep) and torch.equal(o.score[:len(f)], ref.score)
            assert np.array_equal(o.n_kept.cpu().numpy()[:1], ref.n_kept.cpu().numpy()[:1])
    finally:
        hip.hipGetLastError()
        den.close()
        srv.close()


def test_failed_polls_between_batches():
    """Two slots, batches that differ, an error before every other poll: what
    a failed poll had enqueued has ended when it returns, so the next batch of
    that slot, and inputs overwritten once their ticket is done, meet nothing
    of it."""
    import torch
    from paper_2512_10386_amd import binding as B
    from paper_2512_10386_amd.serve import Server
    prm = dict(k=16, leaf_cap=256)
    frames = [torch.from_numpy(synth.sphere_plane(seed=s, n_sphere=900 * s, n_plane=200 * s + 7, n_out=300)[0]).cuda()
              for s in range(1, 9)]
    torch.cuda.synchronize()
    den = B.Denoiser(0, **prm)
    srv = Server(0, hbm_budget=1 << 30, max_slots=2, slot_points=12_000, slot_frames=3, **prm)
    try:
        refs = [(r.keep.cpu(), r.score.cpu()) for r in (den(f) for f in frames)]
        inputs = [f.clone() for f in frames]
        outs = [srv.alloc(len(f)) for f in frames]
        torch.cuda.synchronize()
        tickets = {srv.submit(x, o): i for i, (x, o) in enumerate(zip(inputs, outs))}
        left = set(tickets)
        hip = C.CDLL(B.LIB_PATH)
        failed = polls = 0
        t0 = time.time()
        while left:
            assert time.time() - t0 < 20.0, f"tickets {sorted(left)} never finish"
            polls += 1
            if polls % 2:
                assert hip.hipMalloc(None, C.c_size_t(16)) != 0
            try:
                done = srv.poll()[0]
            except B.GdnError as e:
                assert e.status == B.GDN_EHIP
                failed += 1
                continue
            finally:
                hip.hipGetLastError()  # where the poll started nothing
            for t in done:
                left.remove(t)
                inputs[tickets[t]].zero_()
        torch.cuda.synchronize()
        assert failed > 0
        for (keep, score), o in zip(refs, outs):
            assert torch.equal(o.keep[:len(keep)].cpu(), keep) and torch.equal(o.score[:len(score)].cpu(), score)
    finally:
        hip.hipGetLastError()
        den.close()
        srv.close()
