"""GPU parity on both sides of the rules that choose a sweep kernel from the
number of blocks of a colour launch: few blocks share four waves each, more
take one wave each.  Configuration, energy and accepted count equal the
oracle's bit for bit."""
import os
import sys

import numpy as np
import pytest

from paper_2509_20949_amd import workloads as W

pytestmark = pytest.mark.gpu

# blocks per colour 6 * 12 * 7 = 504 and 6 * 12 * 8 = 576 around the rule's
# 512; widths 12 (whole rounds), 2 (the narrowest) and 5..6 (partial lanes)
FEW = dict(L=(144, 48, 77), block=(12, 2, 6), blocks=504)
MANY = dict(L=(144, 48, 89), block=(12, 2, 6), blocks=576)
# FCC: 6 * 12 * 10 = 720 and 6 * 12 * 11 = 792 around 768
FCC_FEW = dict(L=(144, 48, 113), block=(12, 2, 6), blocks=720)
FCC_MANY = dict(L=(144, 48, 125), block=(12, 2, 6), blocks=792)


def note(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def smcx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_20949_amd import smcx as m
    m.lib()
    return m


@pytest.fixture(scope="module", autouse=True)
def oracle_threads(orc):
    orc.set_threads(min(16, os.cpu_count() or 1))
    yield
    orc.set_threads(1)


def run(smcx, orc, shape, epi, T, seed, n_sweeps=2, lattice=0):
    K = epi.shape[1]
    rng = np.random.default_rng(seed)
    sigma = W.configuration(W.equiatomic(K, W.n_sites(shape["L"], lattice)), rng)
    note(f"{shape} K={K} S={epi.shape[0]} T={T} lattice={lattice}")
    lat = smcx.Lattice(shape["L"], epi, sigma, seed, T, block=shape["block"], lattice=lattice)
    ref = orc.OracleState(shape["L"], shape["block"], epi, sigma, seed, lattice=lattice)
    try:
        nb = smcx.smcx_plan(lat.desc)[1]
        assert nb[0] * nb[1] * nb[2] // 8 == shape["blocks"]
        lat.sweep(n_sweeps)
        ref.sweep(T, n_sweeps)
        bad = np.nonzero(lat.config() != ref.sigma)[0]
        assert bad.size == 0, f"{bad.size} sites differ, first {bad[:8]}"
        assert lat.energy() == int(ref.E[0])
        assert lat.stats()["accepted"] == int(ref.accepted[0]) > 0
    finally:
        lat.close()


@pytest.mark.parametrize("shape", [FEW, MANY], ids=["few", "many"])
@pytest.mark.parametrize("K,S", [(2, 1), (3, 2), (4, 3), (5, 2), (5, 3), (6, 3), (7, 1), (8, 2), (8, 3)])
def test_bcc_kernels_around_the_rule(smcx, orc, shape, K, S):
    run(smcx, orc, shape, W.epi_table(S, K, 25.0, np.random.default_rng(K + 10 * S)), 900.0, 300 + K)


@pytest.mark.parametrize("shape", [FEW, MANY], ids=["few", "many"])
@pytest.mark.parametrize("K", [5, 6, 8])
def test_bcc_full_rows_around_the_rule(smcx, orc, shape, K):
    """Interactions too large for the folded rows; 1 K and 5000 K."""
    v = np.random.default_rng(K).choice([-(1 << 22) + 1, (1 << 22) - 1, 0, 123456], size=(3, K, K)).astype(np.int32)
    epi = np.triu(v) + np.transpose(np.triu(v, 1), (0, 2, 1))
    run(smcx, orc, shape, epi, 5000.0, 40 + K)
    run(smcx, orc, shape, epi, 1.0, 50 + K, n_sweeps=1)


@pytest.mark.parametrize("shape", [FCC_FEW, FCC_MANY], ids=["few", "many"])
@pytest.mark.parametrize("K,S", [(2, 1), (3, 2), (4, 3), (5, 3)])
def test_fcc_kernels_around_the_rule(smcx, orc, shape, K, S):
    run(smcx, orc, shape, W.epi_table(S, K, 25.0, np.random.default_rng(K + 10 * S)), 900.0, 400 + K, lattice=1)


@pytest.mark.parametrize("shape", [FCC_FEW, FCC_MANY], ids=["few", "many"])
def test_fcc_full_rows_around_the_rule(smcx, orc, shape):
    v = np.random.default_rng(5).choice([-(1 << 22) + 1, (1 << 22) - 1, 0, 123456], size=(3, 5, 5)).astype(np.int32)
    epi = np.triu(v) + np.transpose(np.triu(v, 1), (0, 2, 1))
    run(smcx, orc, shape, epi, 5000.0, 45, n_sweeps=1, lattice=1)


@pytest.mark.parametrize("L,B,blocks", [((48, 48, 72), (2, 2, 12), 432), ((48, 48, 96), (2, 2, 12), 576)])
def test_slab_kernels_around_the_rule(smcx, orc, L, B, blocks):
    import torch
    job = W.lattice_job(L, 5, 3, 30.0, np.full(2, 950.0), stream=150, name="slab")
    note(f"slab L={L} B={B}")
    planes = job.sigma.reshape(L[2], -1)
    buf = torch.from_numpy(np.ascontiguousarray(planes[[k % L[2] for k in range(-2, L[2] + 2)]])).to("cuda:0")
    torch.cuda.synchronize()
    desc = smcx.make_desc(L, 5, 3, B, job.seed)
    nb = smcx.smcx_plan(desc)[1]
    assert nb[0] * nb[1] * nb[2] // 8 == blocks
    ctx = smcx.smcx_create_slab(desc, buf.data_ptr(), 0, job.epi, 950.0)
    ref = orc.OracleState(L, B, job.epi, job.sigma, job.seed, fixed_z=True)
    try:
        smcx.smcx_sweep(ctx, 2)
        ref.sweep(950.0, 2)
        assert smcx.smcx_energy(ctx) == int(ref.E[0])
        assert np.array_equal(buf[2:L[2] + 2].cpu().numpy().ravel(), ref.sigma)
        assert smcx.smcx_get_stats(ctx)["accepted"] == int(ref.accepted[0]) > 0
    finally:
        smcx.smcx_destroy(ctx)


def test_batch_crosses_the_rule(smcx, orc):
    """A batch whose launches start above the rule's count and fall below it
    as replicas finish."""
    rng = np.random.default_rng(8)
    epi = W.epi_table(3, 5, 30.0, rng)
    shapes = [(FEW["L"], FEW["block"], 1), ((26, 25, 27), (12, 12, 12), 3), ((40, 40, 40), (4, 4, 4), 2)]
    sites = [W.configuration(W.equiatomic(5, W.n_sites(L)), rng) for L, _, _ in shapes]
    descs = [smcx.make_desc(L, 5, 3, B, 70 + r) for r, (L, B, _) in enumerate(shapes)]
    note("batch around the rule")
    b = smcx.smcx_batch_create(descs, sites, [epi] * 3, [1000.0, 700.0, 1400.0])
    try:
        smcx.smcx_batch_run(b, [n for _, _, n in shapes])
        for r, ((L, B, n), T) in enumerate(zip(shapes, (1000.0, 700.0, 1400.0))):
            ref = orc.OracleState(L, B, epi, sites[r], 70 + r)
            ref.sweep(T, n)
            v = smcx.smcx_batch_ctx(b, r)
            assert smcx.smcx_energy(v) == int(ref.E[0])
            assert np.array_equal(smcx.smcx_get_config(v, sites[r].size), ref.sigma)
    finally:
        smcx.smcx_batch_destroy(b)
