"""Workspace sizes never fall as inputs grow: a workspace made for the largest
frame (or for a server's slot) takes every smaller one. Host side only."""
import pytest

# the tile of the radix passes changes at 2^14, 7 * 2^14 and 2^20 points, the
# tile of the scans at 2^20
EDGES = [1 << 14, 7 << 14, 1 << 20]


@pytest.mark.parametrize("k", [1, 12, 32, 64])
@pytest.mark.parametrize("frames", [1, 2, 300])
def test_workspace_never_falls_as_points_grow(k, frames):
    from paper_2512_10386_amd import binding as B
    p = B.make_params(k=k)
    for edge in EDGES:
        sizes = [B.gdn_workspace_size_batch(0, p, n, frames) for n in range(edge - 3, edge + 4)]
        sizes += [B.gdn_workspace_size_batch(0, p, edge + d, frames) for d in (100, 1000, 3000, 10_000)]
        assert sizes == sorted(sizes), (edge, sizes)


def test_workspace_of_a_slot_takes_fewer_frames():
    from paper_2512_10386_amd import binding as B
    p = B.make_params(k=32)
    for points in (16_400, 114_800, 1_048_700):
        slot = B.gdn_workspace_size_batch(0, p, points, 8)
        for n in (points, points - 150, points - 16, EDGES[0], points // 2):
            for frames in (1, 2, 7, 8):
                if n <= points:
                    assert B.gdn_workspace_size_batch(0, p, n, frames) <= slot, (points, n, frames)


@pytest.mark.parametrize("other", [1000, 0, 3_000_000])
def test_eval_workspace_never_falls_as_clouds_grow(other):
    """Sizes around the edges, against a small, an equal and a large cloud."""
    from paper_2512_10386_amd import binding as B
    for edge in EDGES + [1 << 15]:
        ns = list(range(edge - 3, edge + 4)) + [edge + d for d in (100, 1000, 3000, 10_000)]
        for pair in (lambda n: (n, other or n), lambda n: (other or n, n)):
            sizes = [B.gdn_eval_workspace_size(0, *pair(n)) for n in ns]
            assert sizes == sorted(sizes), (edge, sizes)


@pytest.mark.gpu
def test_server_slot_runs_a_slightly_smaller_batch():
    """A slot of 114,800 points takes a batch of 114,650, on the other side of
    an edge; its frames equal the same frames denoised alone."""
    import time

    import numpy as np
    import torch

    from paper_2512_10386_amd import synth
    from paper_2512_10386_amd.binding import Denoiser
    from paper_2512_10386_amd.serve import Server
    x = torch.from_numpy(synth.lidar_frame(seed=5, n_az=1800)[0][:114_650].astype(np.float32)).cuda()
    frames = [x[:60_000].contiguous(), x[60_000:].contiguous()]
    torch.cuda.synchronize()
    srv = Server(0, hbm_budget=8 << 30, max_slots=1, slot_points=114_800, slot_frames=8, k=32, leaf_cap=512)
    den = Denoiser(0, k=32, leaf_cap=512)
    try:
        outs = [srv.alloc(len(f)) for f in frames]
        left = {srv.submit(f, o) for f, o in zip(frames, outs)}
        t0 = time.time()
        while left:
            assert time.time() - t0 < 30.0, "server did not finish"
            left.difference_update(srv.poll()[0])
        torch.cuda.synchronize()
        for f, o in zip(frames, outs):
            ref = den(f)
            for a, b in ((o.keep, ref.keep), (o.score, ref.score), (o.stage, ref.stage)):
                assert torch.equal(a[:len(f)], b[:len(f)])
    finally:
        den.close()
        srv.close()


def test_nearest_workspace_is_the_least_where_every_pair_is_evaluated():
    """Few queries or few reference points do not pay for sorting millions of
    others, and ask for no room to do it."""
    from paper_2512_10386_amd import binding as B
    for na, nb in ((1, 200_000_000), (2, 120_000_000), (200, 2_000_000), (2_000_000, 200), (20_000_000, 16),
                   (1_000_000, 1000), (3000, 100_000), (5000, 5000)):
        assert B.gdn_nearest_best_workspace_size(0, na, nb) == B.gdn_nearest_workspace_size(0, na), (na, nb)
    for n in (500, 1_000_000):
        least = 2 * (-(-8 * n // 256) * 256) + 2 * 65536
        assert B.gdn_eval_workspace_size(0, 1_000_000, 16) < 2 * 8 * 1_000_000
        assert (B.gdn_eval_workspace_size(0, n, n) > least) == (n > 500)
    for na, nb in ((20_000, 20_000), (1_000_000, 3000), (3000, 1_000_000)):
        best = B.gdn_nearest_best_workspace_size(0, na, nb)
        assert B.gdn_nearest_workspace_size(0, na) < best <= B.gdn_eval_workspace_size(0, na, nb)


def test_nearest_workspace_never_falls_as_clouds_grow():
    from paper_2512_10386_amd import binding as B
    ns = sorted({int(16 * 1.13 ** i) for i in range(110)} | {e + d for e in EDGES for d in (-1, 0, 1)})
    for size in (B.gdn_nearest_best_workspace_size, B.gdn_eval_workspace_size):
        for other in (5, 300, 2500, 16_000, 200_000, 5_000_000):
            for pair in (lambda n: (n, other), lambda n: (other, n), lambda n: (n, n)):
                sizes = [size(0, *pair(n)) for n in ns]
                assert sizes == sorted(sizes), (size.__name__, other)
