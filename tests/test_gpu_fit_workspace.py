"""The score fit reads the last pass's workspace and writes nothing there, so
several evaluations (on several streams, each with a workspace and outputs of
its own) share inputs only."""
import numpy as np
import pytest

from paper_2512_10386_amd import synth

pytestmark = pytest.mark.gpu


def fit_call(B, ctx, th, x, lab, ws, out, stream):
    fp = B.gdn_fit_params(alpha=th[0], sigma=th[1], gamma=th[2], tau=th[3], temperature=1.0)
    B.gdn_fit_loss_grad(ctx, fp, x.data_ptr(), lab.data_ptr(), len(x), ws.data_ptr(), ws.numel(), out.data_ptr(), stream)


@pytest.mark.parametrize("k", [1, 2, 3, 16, 40])
def test_fit_leaves_the_pass_untouched(k):
    import torch
    from paper_2512_10386_amd import binding as B
    xyz, lab = synth.torus_bumpy(7, 0.01, n_torus=4000, n_bumpy=4000, n_out=900)
    x, l = torch.from_numpy(xyz).cuda(), torch.from_numpy(lab).cuda()
    den = B.Denoiser(0, k=k, leaf_cap=512)
    try:
        den(x)
        torch.cuda.synchronize()
        before = den._ws.clone()
        need = B.gdn_fit_workspace_size(den.ctx, len(x))
        assert need <= 8 * len(x) + 256 + 65536  # one double per point, and the blocks' sums
        thetas = [(1.0, 1.0, 2.0, 8.0), (0.3, 1.4, 2.5, 7.0)]
        alone, both = [], []
        for th in thetas:
            ws, out = torch.empty(need, dtype=torch.uint8, device="cuda"), torch.empty(6, dtype=torch.float64, device="cuda")
            fit_call(B, den.ctx, th, x, l, ws, out, torch.cuda.current_stream().cuda_stream)
            alone.append((ws, out))
        torch.cuda.synchronize()
        assert torch.equal(before, den._ws)
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        for th, s in zip(thetas, streams):
            ws, out = torch.empty(need, dtype=torch.uint8, device="cuda"), torch.empty(6, dtype=torch.float64, device="cuda")
            torch.cuda.synchronize()
            both.append((ws, out))
        for rep in range(3):
            for th, s, (ws, out) in zip(thetas, streams, both):
                fit_call(B, den.ctx, th, x, l, ws, out, s.cuda_stream)
        torch.cuda.synchronize()
        for (_, a), (_, b) in zip(alone, both):
            assert np.array_equal(a.cpu().numpy().view(np.uint64), b.cpu().numpy().view(np.uint64))
        assert float(alone[0][1][5]) > 0
    finally:
        den.close()
