"""No workspace is larger than that of the library before the one-launch merge and
the brick codes: a device buffer or a server pool that held a lattice, a batch
or a set of jobs then holds it still (bytes as sw_workspace_bytes_ex and its
relatives returned them)."""
import numpy as np
import pytest

import paper_2302_14720_amd as sw

SIMS = [
    (dict(L=32), 1319680),
    (dict(L=64), 1325824),
    (dict(L=96), 1372928),
    (dict(L=160, q=5), 1479936),
    (dict(L=224), 1640960),
    (dict(L=288), 1855744),
    (dict(L=320), 1636608),
    (dict(L=416, q=5), 2445312),
    (dict(L=512, tile=32), 3027712),
    (dict(L=576), 2363648),
    (dict(L=832), 3505152),
    (dict(L=1024), 4633344),
    (dict(L=1088), 5062656),
    (dict(L=64, flags=2), 1358848),
    (dict(L=160, flags=2), 1684992),
    (dict(L=320, flags=3, q=3), 2865664),
    (dict(L=1024, flags=3), 17216512),
    (dict(L=4064, flags=2), 241570816),
    (dict(L=32768, flags=2), 11992826880),
    (dict(L=16, dims=3), 1359360),
    (dict(L=32, flags=2, q=3, dims=3), 1954048),
    (dict(L=144, flags=1, dims=3), 35930624),
    (dict(L=1616, dims=3), 48928245760),
]
JOBS = [((32, 0, 1), 9472), ((64, 3, 100), 47104), ((160, 5, 100), 201216), ((320, 0, 1), 326400),
        ((1024, 0, 100), 3354624)]
BATCHES = [([32] * 4095, 0, 39885312), ([160, 320, 1024] * 20, 0, 76442624), ([160, 320, 1024] * 20, 2, 76442624),
           ([64, 96, 1088] * 3, 0, 11501056)]
PHI4 = [((2, 1), 2816), ((20, 0), 9122816)]


@pytest.mark.parametrize("cfg,held", SIMS, ids=str)
def test_sim(cfg, held):
    kw = dict(cfg)
    assert 0 < sw.sw_workspace_bytes_ex(sw.sw_config_init(kw.pop("L"), 0.4, 1.0, 1, **kw)) <= held


@pytest.mark.parametrize("job,held", JOBS, ids=str)
def test_job(job, held):
    L, q, n = job
    assert 0 < sw.Server.job_bytes(L, n, q=q) <= held


@pytest.mark.parametrize("sides,merge,held", BATCHES, ids=lambda v: str(v)[:20])
def test_batch(sides, merge, held):
    assert 0 < sw.sw_batch_workspace_bytes(np.array(sides, dtype=np.int32), merge=merge, ring=1) <= held


@pytest.mark.parametrize("sim,held", PHI4, ids=str)
def test_phi4(sim, held):
    assert 0 < sw.lib().sw_phi4_workspace_bytes(*sim) <= held
