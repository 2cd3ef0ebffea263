"""Launch tunings the batching server gives to small requests."""
import pytest

from paper_2605_07621_amd import ecut as E, inputs as I


@pytest.mark.gpu
def test_small_spin_requests_keep_the_default(dev, tmp_path, monkeypatch):
    """Small spin requests of a batching server are not timed one by one: they
    keep the default tuning, whose work groups share one launch per step.
    (The autotuner would leave the shape's entry in its cache file.)"""
    cache = tmp_path / "tunings.json"
    monkeypatch.setenv("ECUT_TUNE_CACHE", str(cache))
    srv = E.Server(1 << 30, max_steps=300, tol=1e-10, autotune=True)
    p = I.Problem(I.xxz_chain(13, 1.0, 0.85), I.Cut("spatial", I.left_mask_first(4)), 5)
    ids = [srv.submit(p, seed=k) for k in range(3)]
    srv.drain()
    res = {r["req_id"]: r for r in srv.poll(8)}
    srv.close()
    assert all(res[i]["status"] == 0 for i in ids)
    assert max(abs(res[i]["energy"] - res[ids[0]]["energy"]) for i in ids) <= 1e-9
    assert not cache.exists() or '"' not in cache.read_text()
