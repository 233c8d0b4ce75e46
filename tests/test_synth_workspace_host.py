"""Workspaces of the probe synthesis hold what the call uses (host sizes, no GPU):
the C operand and the windows, T of the two-stage sum where the positions form
scan columns, the BF16 records where sums are large, and nothing as large as S
otherwise."""
import ctypes

import numpy as np
import pytest

SLACK = 4096


def _setup(n=1024, L=100.0, alpha=0.020, f=4):
    import paper_1706_08563_amd as P
    return P, P.prism_smatrix_plan(P.prism_grid_init((L, L, 20.0), 2.0, n), 200e3, alpha, f)


def _scan(nx, ny, L=100.0):
    y, x = np.meshgrid(np.arange(ny) * (L / ny) + 0.1, np.arange(nx) * (L / nx) + 0.3, indexing="ij")
    return np.stack([x.ravel(), y.ravel()], axis=1)


def _job_bytes(d, probes, beams=None):
    return probes * ((((beams or d.n_beams) + 15) // 16) * 128 + d.m_win ** 2 * 8)


def _records(d, beams):
    return (beams + 15) // 16 * 16 * d.ns ** 2 * 4


class _Plan:                                              # the size query reads only the host plan
    def __init__(self, plan):
        self.plan = plan


def test_positions_without_columns_need_no_scratch():
    P, d = _setup()
    plan = P.prism_probe_plan_init(d, np.random.default_rng(1).uniform(0.0, 100.0, size=(400, 2)))
    assert 0 <= plan.ws_bytes - _job_bytes(d, 400) <= SLACK


def test_scan_columns_need_their_T_up_to_the_size_of_S():
    P, d = _setup()
    rows = len(np.unique(P.prism_beam_list(d)[:, 1]))
    full = (d.n_beams + 15) // 16 * 16 * d.ns ** 2 * 8
    for nx in (1, 20, 128, 300):
        plan = P.prism_probe_plan_init(d, _scan(nx, 10))
        T = nx * rows * d.ns * d.m_win * 8
        assert 0 <= plan.ws_bytes - _job_bytes(d, 10 * nx) - min(T, full) <= SLACK


def test_large_sums_need_the_records():
    P, d = _setup()
    plan = P.prism_probe_plan_init(d, np.random.default_rng(2).uniform(0.0, 100.0, size=(16384, 2)))
    assert 0 <= plan.ws_bytes - _job_bytes(d, 16384) - _records(d, d.n_beams) <= SLACK


@pytest.mark.parametrize("probes,large", [(400, False), (16384, True)])
def test_beam_chunks_need_the_records_only(probes, large):
    P, d = _setup()
    xy = np.random.default_rng(3).uniform(0.0, 100.0, size=(probes, 2))
    plan, chunk = _Plan(P.prism_probe_plan_init(d, xy)), 320
    base = _job_bytes(d, probes, chunk) + (_records(d, chunk) if large else 0)
    assert 0 <= P.prism_probe_chunked_workspace(d, plan, chunk) - base <= SLACK
    assert 0 <= P.prism_probe_streaming_workspace(d, plan, chunk) - base - 2 * chunk * d.ns ** 2 * 8 <= SLACK
    few = _Plan(P.prism_probe_plan_init(d, _scan(64, 16)))   # scan columns: beam chunks take the direct sum
    assert 0 <= P.prism_probe_chunked_workspace(d, few, chunk) - _job_bytes(d, 1024, chunk) <= SLACK


def test_batches_share_the_scratch_of_one_s_matrix():
    """Jobs on one S-matrix, none of which would convert it alone, and the
    footprint that the server takes for them."""
    P, d = _setup()
    from paper_1706_08563_amd import serve
    from paper_1706_08563_amd._lib import prism_probe_job
    rng = np.random.default_rng(4)
    plans = [P.prism_probe_plan_init(d, rng.uniform(0.0, 100.0, size=(6000, 2))) for _ in range(3)]
    assert all(p.ws_bytes - _job_bytes(d, 6000) <= SLACK for p in plans)
    assert 0 <= serve._batch_ws(d, plans) - 3 * _job_bytes(d, 6000) - _records(d, d.n_beams) <= SLACK
    jobs = (prism_probe_job * 3)()
    for k, (job, plan) in enumerate(zip(jobs, plans)):     # three S-matrices
        job.desc, job.plan, job.out_scale = ctypes.pointer(d), ctypes.pointer(plan), 1.0
        job.S, job.plan_dev, job.out = 256 * (k + 1), 256, 256
    need = ctypes.c_size_t()
    assert P.lib.prism_probe_batch_workspace(jobs, 3, ctypes.byref(need)) == P.PRISM_OK
    assert 0 <= need.value - 3 * _job_bytes(d, 6000) <= SLACK
