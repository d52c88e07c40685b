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
