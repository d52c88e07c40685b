"""Nearest neighbours and metrics of clouds of unequal sizes: the two directions
of the brute-force search have grids of their own (few queries take the
reference in many chunks), one point on a side among them. Against the oracle,
tolerances as in test_gpu_eval.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ev():
    from paper_2512_10386_amd.evaluate import Evaluator
    e = Evaluator(0)
    yield e
    e.close()


def cloud(n, seed):
    x = np.random.default_rng(seed).normal(size=(n, 3)).astype(np.float32)
    x[n // 2:n // 2 + 3] = x[:1]  # copies: equal distances go to the smaller index
    return x


@pytest.mark.parametrize("na,nb", [(1, 70_001), (70_001, 1), (2, 255), (257, 3), (256, 40_000), (255, 40_193),
                                   (40_193, 257), (3_000, 20_000), (524_289, 5), (5, 600_000), (300, 300_000)])
def test_unequal_clouds_vs_oracle(ev, oracle, na, nb):
    import torch
    from paper_2512_10386_amd import binding as B
    a, b = cloud(na, 1), cloud(nb, 2)
    at, bt = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    print(f"[unequal] {na} {nb}", flush=True)
    idx, d2 = ev.nearest(at, bt)
    ri, rd = oracle.nearest(a, b)
    assert np.array_equal(idx.cpu().numpy().view(np.uint32), ri)
    assert np.array_equal(d2.cpu().numpy().view(np.uint32), rd.view(np.uint32))
    exp = oracle.eval_metrics(a, b)
    assert np.allclose(ev.metrics(at, bt).cpu().numpy(), exp, rtol=1e-12, atol=0)
    # the smallest workspace accepted
    least = -(-8 * na // 256) * 256 + -(-8 * nb // 256) * 256 + 2 * 65536
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    out = torch.empty(4, dtype=torch.float64, device="cuda")
    B.gdn_eval_metrics(ev.ctx, at.data_ptr(), na, bt.data_ptr(), nb, ws.data_ptr(), least, out.data_ptr(),
                       torch.cuda.current_stream().cuda_stream)
    assert np.allclose(out.cpu().numpy(), exp, rtol=1e-12, atol=0)


# both sides of the lines between sorting and evaluating every pair, the key
# widths (2^15 points) and the radix tiles (7 * 2^14 and 2^20) with uneven clouds
@pytest.mark.parametrize("na,nb,sorts", [
    (32_768, 12_000, True), (32_769, 12_001, True), (1_048_577, 3_000, True), (3_000, 1_048_577, True),
    (114_689, 4_500, True), (4_500, 114_688, True), (16_400, 16_400, True), (15_000, 15_000, False),
    (100_000, 3_000, False), (3_000, 100_000, False), (1_048_577, 301, False)])
def test_sorted_search_of_uneven_clouds(ev, na, nb, sorts):
    import torch
    from paper_2512_10386_amd import binding as B
    at, bt = torch.from_numpy(cloud(na, 3)).cuda(), torch.from_numpy(cloud(nb, 4)).cuda()
    least = B.gdn_nearest_workspace_size(ev.ctx, na)
    assert (B.gdn_nearest_best_workspace_size(ev.ctx, na, nb) > least) == sorts
    print(f"[unequal] {na} {nb}", flush=True)
    idx, d2 = ev.nearest(at, bt)
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")  # every pair
    ri, rd = torch.empty_like(idx), torch.empty_like(d2)
    B.gdn_nearest(ev.ctx, at.data_ptr(), na, bt.data_ptr(), nb, ws.data_ptr(), least, ri.data_ptr(), rd.data_ptr(),
                  torch.cuda.current_stream().cuda_stream)
    assert torch.equal(idx, ri) and torch.equal(d2.view(torch.int32), rd.view(torch.int32))


def test_lost_order_answers_every_query(ev, oracle):
    """Where a wait of the sort expires there is no order to go by: each query
    is still answered once, and the metrics sum each point once."""
    import torch
    from paper_2512_10386_amd import binding as B
    a, b = cloud(18_003, 5), cloud(17_001, 6)
    a[7, 1] = np.nan
    at, bt = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    at2 = at[8:].contiguous()
    assert B.gdn_nearest_best_workspace_size(ev.ctx, len(a), len(b)) > B.gdn_nearest_workspace_size(ev.ctx, len(a))
    want, metrics = ev.nearest(at, bt), ev.metrics(at2, bt).cpu().numpy()
    need = B.gdn_eval_workspace_size(ev.ctx, len(a), len(b))
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")  # no order of an earlier call
    idx = torch.full((len(a),), -1, dtype=torch.int32, device="cuda")
    d2 = torch.full((len(a),), -1.0, dtype=torch.float32, device="cuda")
    out = torch.empty(4, dtype=torch.float64, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    B.gdn_debug_lose_order(ev.ctx, True)
    try:
        print("[lost order]", flush=True)
        B.gdn_nearest(ev.ctx, at.data_ptr(), len(a), bt.data_ptr(), len(b), ws.data_ptr(), need, idx.data_ptr(),
                      d2.data_ptr(), st)
        ws2 = torch.zeros_like(ws)
        B.gdn_eval_metrics(ev.ctx, at2.data_ptr(), len(at2), bt.data_ptr(), len(b), ws2.data_ptr(), need,
                           out.data_ptr(), st)
    finally:
        B.gdn_debug_lose_order(ev.ctx, False)
    assert torch.equal(idx, want[0]) and torch.equal(d2.view(torch.int32), want[1].view(torch.int32))
    assert np.allclose(out.cpu().numpy(), metrics, rtol=1e-12, atol=0)
    assert np.allclose(out.cpu().numpy(), oracle.eval_metrics(a[8:], b), rtol=1e-12, atol=0)


# queries that have the reference at about one distance all around them: the
# search of near groups first gives up, and the workgroup takes all points
@pytest.mark.parametrize("na,nb", [(18_001, 18_003), (16_387, 40_000), (40_003, 16_385), (3_001, 200_003)])
@pytest.mark.parametrize("what", ["middle", "copies", "some"])
def test_reference_at_one_distance(ev, na, nb, what):
    import torch
    from paper_2512_10386_amd import binding as B
    rng = np.random.default_rng(na + nb)
    b = rng.normal(size=(nb, 3))
    b = (b / np.linalg.norm(b, axis=1, keepdims=True)).astype(np.float32)
    a = (1e-3 * rng.normal(size=(na, 3))).astype(np.float32)
    if what == "copies":  # equal distances: the axis points, many times, from the centre
        b = np.round(b / np.abs(b).max(1, keepdims=True)).astype(np.float32)
        b[(b != 0).sum(1) != 1] = [0, 0, 1]
        a[:: 3] = 0
        a[5] = [np.nan, 0, 0]
        a[7] = [np.inf, 0, 0]
    elif what == "some":  # a few queries of a tile each
        a[np.arange(na) % 5 != 0] += b[rng.integers(0, nb, int((np.arange(na) % 5 != 0).sum()))]
    at, bt = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    least = B.gdn_nearest_workspace_size(ev.ctx, na)
    assert B.gdn_nearest_best_workspace_size(ev.ctx, na, nb) > least
    print(f"[one distance] {what} {na} {nb}", flush=True)
    idx, d2 = ev.nearest(at, bt)
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")  # every pair
    ri, rd = torch.empty_like(idx), torch.empty_like(d2)
    st = torch.cuda.current_stream().cuda_stream
    B.gdn_nearest(ev.ctx, at.data_ptr(), na, bt.data_ptr(), nb, ws.data_ptr(), least, ri.data_ptr(), rd.data_ptr(), st)
    assert torch.equal(idx, ri) and torch.equal(d2.view(torch.int32), rd.view(torch.int32))
    if what != "copies":
        least = -(-8 * na // 256) * 256 + -(-8 * nb // 256) * 256 + 2 * 65536
        ws = torch.empty(least, dtype=torch.uint8, device="cuda")
        out = torch.empty(4, dtype=torch.float64, device="cuda")
        B.gdn_eval_metrics(ev.ctx, at.data_ptr(), na, bt.data_ptr(), nb, ws.data_ptr(), least, out.data_ptr(), st)
        assert np.allclose(ev.metrics(at, bt).cpu().numpy(), out.cpu().numpy(), rtol=1e-12, atol=0)


# a few points, or many, far outside the others: the cells of the sort grow with
# the distance from the middle; copies, and clouds of which a half is not finite
@pytest.mark.parametrize("na,nb", [(18_003, 17_001), (40_001, 36_003)])
@pytest.mark.parametrize("what", ["one", "one_b", "many", "flat", "copies", "overflow", "nan"])
def test_stray_points(ev, na, nb, what):
    import torch
    from paper_2512_10386_amd import binding as B
    rng = np.random.default_rng(na)
    a, b = cloud(na, 7), cloud(nb, 8)
    if what == "one":
        a[3] = [1e6, -2e5, 1e6]
    elif what == "one_b":
        b[nb - 1] = [-40.0, 300.0, 0.0]
    elif what == "many":
        a[::40], b[::50] = 1e4 * rng.normal(size=a[::40].shape), 1e5 * rng.normal(size=b[::50].shape)
    elif what == "flat":
        a[:, 2] = b[:, 2] = 1.5
        b[0, 2] = 1e5
    elif what == "copies":  # no extent of the middle half
        a[: na * 3 // 4], b[: nb * 3 // 4] = a[0], a[0]
        b[5] = 1e3
    elif what == "overflow":
        a[0], b[0] = 3e38, -3e38
    else:
        a[::2, 0], b[1::2, 1] = np.nan, np.inf
        b[0] = 1e4
    at, bt = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    least = B.gdn_nearest_workspace_size(ev.ctx, na)
    assert B.gdn_nearest_best_workspace_size(ev.ctx, na, nb) > least
    print(f"[stray] {what} {na} {nb}", flush=True)
    idx, d2 = ev.nearest(at, bt)
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")  # every pair
    ri, rd = torch.empty_like(idx), torch.empty_like(d2)
    B.gdn_nearest(ev.ctx, at.data_ptr(), na, bt.data_ptr(), nb, ws.data_ptr(), least, ri.data_ptr(), rd.data_ptr(),
                  torch.cuda.current_stream().cuda_stream)
    assert torch.equal(idx, ri) and torch.equal(d2.view(torch.int32), rd.view(torch.int32))
