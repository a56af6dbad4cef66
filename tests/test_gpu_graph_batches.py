"""A graph captured on one batch stays valid while the batch does, whatever else runs on its context:
a batch of fewer roots whose FMM trees have more boxes (1088 roots take 63, 8192 take 255), and
wider blocks of columns on the captured batch itself.  Every replay equals the eager result bit
for bit."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_replay_after_other_batches():
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    ctx = native.Context()
    o = native.default_opts(method=2)
    dev = gp.dev()

    def setup(sizes, seed, m):
        batch, X = gen.small_batch(sizes, seed=seed, m=m)
        b = native.Batch(ctx, batch.off)
        d, z, rho, Xt = (gp.to_dev(a) for a in (batch.d, batch.z, batch.rho, np.asarray(X).T))
        new = lambda t=torch.float64, n=batch.total_n: torch.empty(n, dtype=t, device=dev)
        sol = dict(lam=new(), eta=new(), origin=new(torch.int32), iters=new(torch.int32),
                   status=new(torch.int32, batch.nprob))
        out = dict(sol, zhat=new(), b=new(), Y1=torch.empty_like(Xt), Y0=torch.empty_like(Xt))

        def step():
            native.secular_solve(ctx, b, d, z, rho, opts=o, out=sol)
            f = (out["eta"], out["origin"], out["status"])
            native.loewner(ctx, b, d, z, rho, *f, opts=o, out=(out["zhat"], out["b"]))
            for t in (0, 1):
                native.cauchy_apply(ctx, b, d, out["zhat"], out["b"], *f, Xt, trans=t, opts=o, Y=out[f"Y{t}"])
            g = native.secular_backward(ctx, b, d, z, rho, *f, g_lam=out["lam"], opts=o)
            out.update(zip(("gd", "gz", "gr"), g))

        def wide():
            Xw = Xt[:1].expand(64, -1).contiguous()
            for t in (0, 1):
                native.cauchy_apply(ctx, b, d, out["zhat"], out["b"], out["eta"], out["origin"],
                                    out["status"], Xw, trans=t, opts=o)
        return batch, step, wide, out

    batch, step, wide, out = setup([8192, 8192, 5000, 4097], 121, 5)
    step()
    torch.cuda.synchronize()
    eager = {k: v.clone() for k, v in out.items()}
    assert not eager["status"].any()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        step()
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    captured = dict(out)
    other, ostep, owide, oout = setup([1088] * 20, 122, 5)
    assert other.total_n < batch.total_n
    for rep in range(3):
        ostep()
        owide()
        wide()
        for v in captured.values():
            v.fill_(-7)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for k, v in eager.items():
            assert torch.equal(captured[k], v), (rep, k)
