"""The autotuner times a shape on launches that read it, and leaves one that none reads at its
heuristic: counted through the per-kernel timing.  Lines of an older cache file are not taken."""
import numpy as np
import pytest

from paper_2108_04209_amd import gen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def tune(sizes, **kw):
    from paper_2108_04209_amd import native
    from tests import gpu_pipeline as gp
    ctx = gp.context()
    batch = gen.small_batch(sizes, seed=137)
    b = native.Batch(ctx, batch.off)
    d, z, rho = gp.to_dev(batch.d), gp.to_dev(batch.z), gp.to_dev(batch.rho)
    before = native.batch_shapes(b)
    native.kernel_times()
    native.kernel_timing(True, mode="events")
    try:
        after = native.autotune(ctx, b, d, z, rho, opts=native.default_opts(**kw))
        torch.cuda.synchronize()
        count = {k: v[1] for k, v in native.kernel_times().items()}
    finally:
        native.kernel_timing(False)
    return before, after, count


def test_solver_in_lds_reads_no_shape(monkeypatch):
    monkeypatch.delenv("SUPERDC_TUNE_CACHE", raising=False)
    before, after, count = tune([512] * 16)
    assert count["k_secular"] == 1  # the solution that the other kernels are tuned on
    assert all(after[k] == before[k] for k in ("sec_chunk", "sec_split", "fmm_split"))


def test_scalar_solver(monkeypatch):
    monkeypatch.delenv("SUPERDC_TUNE_CACHE", raising=False)
    _, _, count = tune([5000, 300], method=1)
    assert count["k_secular"] > 3


def test_small_vectors_by_the_launch_that_splits(monkeypatch):
    """zhat and b of problems of at most 192 poles take one launch without a split; the split is that
    of the products alone, which HSS steps run (behind their packing launch)."""
    monkeypatch.delenv("SUPERDC_TUNE_CACHE", raising=False)
    _, _, count = tune([100] * 16)
    assert count["k_pack_ke"] == count["k_loewner"] == 9  # 1, 2, 4 wavefronts, three runs each
    assert "k_bnorm" not in count


def test_no_direct_problem(monkeypatch):
    monkeypatch.delenv("SUPERDC_TUNE_CACHE", raising=False)
    before, after, count = tune([2048] * 20, method=2)
    assert all(after[k] == before[k] for k in ("sec_chunk", "sec_split", "vec_split", "bwd_split"))
    assert after["fmm_split"] in (1, 2, 4, 8) and count["k_secular_fmm"] >= 12
    assert not {"k_secular", "k_loewner", "k_bnorm", "k_bwd"} & set(count)


def test_cache_version(tmp_path, monkeypatch):
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("SUPERDC_TUNE_CACHE", str(path))
    _, first, _ = tune([700] * 3)
    line = path.read_text().split()
    old = line[:-1]
    old[1:] = ["64", "16", "16", "16", "8"]
    path.write_text(" ".join(old) + "\n")
    _, again, count = tune([700] * 3)
    assert count["k_secular"] == 1 and again["sec_split"] == first["sec_split"]
    assert len([x for x in path.read_text().split("\n") if x.strip()]) == 2
    _, taken, count = tune([700] * 3)
    assert taken == again and not count
