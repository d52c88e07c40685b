"""The largest cloud the search takes, 2^30 - 1 queries: every query is answered,
and a sample of them, the ends among it, as all pairs give it."""
import pytest

pytestmark = pytest.mark.gpu


def test_most_queries():
    import torch
    from paper_2512_10386_amd import binding as B
    na, nb = (1 << 30) - 1, 5_000
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GiB of device memory")
    g = torch.Generator("cuda").manual_seed(1)
    a = torch.rand(3 * na, generator=g, device="cuda").view(na, 3)
    b = torch.rand(nb, 3, generator=g, device="cuda")
    ctx = B.gdn_create(0)
    try:
        need = B.gdn_nearest_best_workspace_size(ctx, na, nb)
        assert need > B.gdn_nearest_workspace_size(ctx, na)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        idx = torch.full((na,), -1, dtype=torch.int32, device="cuda")
        d2 = torch.empty(na, dtype=torch.float32, device="cuda")
        print(f"[largest] {na} queries, workspace {need >> 20} MiB", flush=True)
        B.gdn_nearest(ctx, a.data_ptr(), na, b.data_ptr(), nb, ws.data_ptr(), need, idx.data_ptr(), d2.data_ptr(),
                      torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        del ws
        assert int(idx.min()) >= 0 and int(idx.max()) < nb
        s = torch.cat([torch.arange(100, device="cuda"), torch.arange(na - 100, na, device="cuda"),
                       torch.randint(0, na, (2000,), generator=g, device="cuda")])
        e = b[None] - a[s][:, None]
        e = e * e
        d = (e[..., 0] + e[..., 1]) + e[..., 2]
        best = d.min(1).values
        assert torch.equal(d2[s], best)
        assert torch.equal(d.gather(1, idx[s].long()[:, None])[:, 0], best)
    finally:
        B.gdn_destroy(ctx)
        torch.cuda.empty_cache()
