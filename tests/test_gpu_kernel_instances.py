"""GPU parity of the instances of the sweep kernels.  Above all of those that give
a block one wavefront, on launches of more blocks than the rule gives four
waves (512 a colour on BCC, 768 on FCC): every species and shell count, every
form of the weight rows, blocks 2 to 12 cells wide along each axis on odd and
even rows, single lattices, slabs, batches and served requests; and slabs of
few blocks, whose instances share four waves.  Configuration, energy and
accepted count equal the oracle's bit for bit."""
import os
import sys

import numpy as np
import pytest

from paper_2509_20949_amd import workloads as W

pytestmark = pytest.mark.gpu
FCC = 1

# (cells, block parameter, blocks per colour); the x widths are in the names.
# Odd Lx * Ly: every other plane of the lattice starts at an odd word.
BCC_SHAPES = {
    "x2_3": ((33, 33, 45), (3, 2, 2), 528),
    "x4_5": ((45, 49, 38), (5, 2, 2), 540),
    "x6_7": ((55, 49, 45), (7, 2, 2), 528),
    "x10_11": ((63, 49, 61), (11, 2, 2), 540),
    "x11_12": ((71, 49, 61), (12, 2, 2), 540),
    "y12": ((45, 144, 73), (5, 12, 2), 540),
    "z12": ((45, 73, 144), (5, 2, 12), 540),
}
FCC_SHAPES = {
    "x2_3": ((33, 33, 69), (3, 2, 2), 816),
    "x4_5": ((45, 49, 53), (5, 2, 2), 780),
    "x6_7": ((55, 49, 69), (7, 2, 2), 816),
    "x10_11": ((63, 49, 89), (11, 2, 2), 792),
    "y12": ((36, 95, 140), (3, 12, 2), 840),
    "z12": ((36, 140, 95), (3, 2, 12), 840),
}
# 28^3 / 8 blocks a colour, between 10 and 11 for each of 256 CUs: workgroups of 11 blocks
FCC_ELEVEN = ((56, 56, 56), (2, 2, 2), 2744)
EXTREME = (-(1 << 22) + 1, (1 << 22) - 1, 0, 123456)


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


def folded_epi(K, S):
    return W.epi_table(S, K, 25.0, np.random.default_rng(K + 10 * S))


def full_epi(K, S):
    """Interactions whose folded weights leave the three digits and the 24 bits."""
    v = np.random.default_rng(K + 10 * S).choice(EXTREME, size=(S, K, K)).astype(np.int32)
    v[:, 0, 0], v[:, 0, K - 1], v[:, K - 1, K - 1] = EXTREME[1], EXTREME[0], EXTREME[1]
    return np.triu(v) + np.transpose(np.triu(v, 1), (0, 2, 1))


def blocks_of(smcx, desc):
    nb = smcx.smcx_plan(desc)[1]
    return nb[0] * nb[1] * nb[2] // 8


def equal(got, ref, what):
    bad = np.nonzero(got != ref)[0]
    assert bad.size == 0, f"{what}: {bad.size} sites differ, first {bad[:8]}"


def single(smcx, orc, shape, epi, T, seed, n_sweeps=2, lattice=0):
    L, B, blocks = shape
    S, K = epi.shape[:2]
    rng = np.random.default_rng(seed)
    sigma = W.configuration(W.equiatomic(K, W.n_sites(L, lattice)), rng)
    note(f"L={L} B={B} K={K} S={S} T={T} lattice={lattice}")
    lat = smcx.Lattice(L, epi, sigma, seed, T, block=B, lattice=lattice)
    ref = orc.OracleState(L, B, epi, sigma, seed, lattice=lattice)
    try:
        assert blocks_of(smcx, lat.desc) == blocks
        lat.sweep(n_sweeps)
        ref.sweep(T, n_sweeps)
        equal(lat.config(), ref.sigma, f"L={L} B={B}")
        assert lat.energy() == int(ref.E[0])
        assert lat.stats()["accepted"] == int(ref.accepted[0])
    finally:
        lat.close()


@pytest.mark.parametrize("S", [1, 2, 3])
@pytest.mark.parametrize("K", [2, 3, 4, 5, 6, 7, 8])
def test_bcc_every_species_shell_and_width(smcx, orc, K, S):
    epi = folded_epi(K, S)
    assert smcx.smcx_weight_rows(0, K, S, epi)[0] == (2 if K <= 5 else 1)   # byte digits, or the last species folded in
    for k, shape in enumerate(BCC_SHAPES.values()):
        single(smcx, orc, shape, epi, 900.0, 500 + 10 * K + k)


@pytest.mark.parametrize("S", [1, 2, 3])
@pytest.mark.parametrize("K", [2, 3, 4, 5, 6, 8])
def test_bcc_full_rows_every_species_and_shell(smcx, orc, K, S):
    epi = full_epi(K, S)
    assert smcx.smcx_weight_rows(0, K, S, epi)[0] == 0
    single(smcx, orc, BCC_SHAPES["x6_7"], epi, 5000.0, 600 + K)
    single(smcx, orc, BCC_SHAPES["x11_12"], epi, 1.0, 610 + K, n_sweeps=1)


@pytest.mark.parametrize("S", [1, 2, 3])
@pytest.mark.parametrize("K", [2, 3, 4, 5])
def test_fcc_every_species_shell_and_width(smcx, orc, K, S):
    epi = folded_epi(K, S)
    assert smcx.smcx_weight_rows(1, K, S, epi)[0] == 2
    for k, shape in enumerate(FCC_SHAPES.values()):
        single(smcx, orc, shape, epi, 900.0, 700 + 10 * K + k, lattice=FCC)


@pytest.mark.parametrize("S", [1, 2, 3])
def test_fcc_full_rows(smcx, orc, S):
    epi = full_epi(5, S)
    assert smcx.smcx_weight_rows(1, 5, S, epi)[0] == 0
    single(smcx, orc, FCC_SHAPES["x4_5"], epi, 5000.0, 800 + S, n_sweeps=1, lattice=FCC)


@pytest.mark.parametrize("S", [1, 2, 3])
@pytest.mark.parametrize("rows", ["digits", "full"])
def test_fcc_eleven_blocks_a_workgroup(smcx, orc, rows, S):
    epi = folded_epi(5, S) if rows == "digits" else full_epi(5, S)
    assert smcx.smcx_weight_rows(1, 5, S, epi)[0] == (2 if rows == "digits" else 0)
    single(smcx, orc, FCC_ELEVEN, epi, 1100.0, 820 + S, lattice=FCC)


SLABS = [((69, 49, 60), (12, 2, 2), 540), ((45, 49, 38), (5, 2, 2), 540), ((35, 144, 78), (4, 12, 2), 570)]
FEW_SLABS = [((23, 24, 22), (12, 4, 6), 6), ((17, 15, 48), (3, 5, 12), 12)]


@pytest.mark.parametrize("K,S", [(5, 3), (4, 2), (3, 1), (6, 3), (8, 2)])
@pytest.mark.parametrize("L,B,blocks", SLABS)
def test_slab(smcx, orc, L, B, blocks, K, S):
    run_slab(smcx, orc, L, B, blocks, K, S)


@pytest.mark.parametrize("S", [1, 2, 3])
@pytest.mark.parametrize("K", [2, 3, 4, 5, 6, 8])
def test_slab_of_few_blocks(smcx, orc, K, S):
    for L, B, blocks in FEW_SLABS:
        run_slab(smcx, orc, L, B, blocks, K, S)


def run_slab(smcx, orc, L, B, blocks, K, S):
    import torch
    epi = folded_epi(K, S)
    rng = np.random.default_rng(900 + K)
    sigma = W.configuration(W.equiatomic(K, W.n_sites(L)), rng)
    note(f"slab L={L} B={B} K={K} S={S}")
    planes = sigma.reshape(L[2], -1)
    buf = torch.from_numpy(np.ascontiguousarray(planes[[k % L[2] for k in range(-2, L[2] + 2)]])).to("cuda:0")
    torch.cuda.synchronize()
    desc = smcx.make_desc(L, K, S, B, 71)
    assert blocks_of(smcx, desc) == blocks
    ctx = smcx.smcx_create_slab(desc, buf.data_ptr(), 0, epi, 950.0)
    ref = orc.OracleState(L, B, epi, sigma, 71, fixed_z=True)
    try:
        smcx.smcx_sweep(ctx, 2)
        ref.sweep(950.0, 2)
        assert smcx.smcx_energy(ctx) == int(ref.E[0])
        equal(buf[2:L[2] + 2].cpu().numpy().ravel(), ref.sigma, "slab")
        assert smcx.smcx_get_stats(ctx)["accepted"] == int(ref.accepted[0]) > 0
    finally:
        smcx.smcx_destroy(ctx)


# replicas of a batch (or requests of a server): the first alone is above the
# rule, the others below it, and each runs another number of sweeps
MIXES = {
    "bcc": (0, [(BCC_SHAPES["x6_7"][:2], 2), (((26, 25, 27), (12, 12, 12)), 5), (((14, 9, 11), (5, 4, 3)), 3)]),
    "fcc": (FCC, [(FCC_SHAPES["x4_5"][:2], 2), (((25, 24, 26), (12, 12, 12)), 5), (((13, 9, 10), (5, 4, 3)), 3)]),
}


def mix(smcx, orc, kind, K, S, epi):
    """Descriptors, sites, temperatures, sweeps and the oracle's results."""
    lattice, shapes = MIXES[kind]
    rng = np.random.default_rng(1000 + 10 * K + S)
    out = []
    for r, ((L, B), n) in enumerate(shapes):
        sigma = W.configuration(W.equiatomic(K, W.n_sites(L, lattice)), rng)
        T = 700.0 + 250.0 * r
        ref = orc.OracleState(L, B, epi, sigma, 80 + r, lattice=lattice)
        ref.sweep(T, n)
        out.append((smcx.make_desc(L, K, S, B, 80 + r, lattice), sigma, T, n, ref))
    assert blocks_of(smcx, out[0][0]) > (768 if lattice else 512) > sum(blocks_of(smcx, d[0]) for d in out[1:])
    return out


MIX_CASES = [("bcc", 5, 3, "folded"), ("bcc", 8, 2, "folded"), ("bcc", 3, 1, "folded"), ("bcc", 6, 3, "full"),
             ("fcc", 5, 3, "folded"), ("fcc", 4, 2, "folded"), ("fcc", 2, 1, "folded"), ("fcc", 5, 3, "full")]


@pytest.mark.parametrize("kind,K,S,rows", MIX_CASES)
def test_batch_above_and_below_the_rule(smcx, orc, kind, K, S, rows):
    epi = folded_epi(K, S) if rows == "folded" else full_epi(K, S)
    jobs = mix(smcx, orc, kind, K, S, epi)
    for run in (smcx.smcx_batch_run, smcx.smcx_batch_run_unbatched):
        note(f"{run.__name__} {kind} K={K} S={S} {rows}")
        b = smcx.smcx_batch_create([j[0] for j in jobs], [j[1] for j in jobs], [epi] * len(jobs), [j[2] for j in jobs])
        try:
            run(b, [j[3] for j in jobs])
            for r, (_, sigma, _, _, ref) in enumerate(jobs):
                v = smcx.smcx_batch_ctx(b, r)
                equal(smcx.smcx_get_config(v, sigma.size), ref.sigma, f"replica {r}")
                assert smcx.smcx_energy(v) == int(ref.E[0])
                assert smcx.smcx_get_stats(v)["accepted"] == int(ref.accepted[0])
        finally:
            smcx.smcx_batch_destroy(b)


@pytest.mark.parametrize("kind,K,S,rows", MIX_CASES)
def test_server_above_and_below_the_rule(smcx, orc, kind, K, S, rows):
    epi = folded_epi(K, S) if rows == "folded" else full_epi(K, S)
    jobs = mix(smcx, orc, kind, K, S, epi)
    note(f"server {kind} K={K} S={S} {rows}")
    srv = smcx.smcx_server_create(1 << 28, len(jobs), 2)
    try:
        ids = [smcx.smcx_server_submit(srv, d, sigma, epi, T, n) for d, sigma, T, n, _ in jobs]
        for _ in range(12):
            smcx.smcx_server_step(srv)
        for rid, (_, sigma, _, _, ref) in zip(ids, jobs):
            assert smcx.smcx_server_poll(srv, rid) == 2
            E, accepted, sites = smcx.smcx_server_result(srv, rid, sigma.size)
            equal(sites, ref.sigma, f"request {rid}")
            assert E == int(ref.E[0]) and accepted == int(ref.accepted[0])
    finally:
        smcx.smcx_server_destroy(srv)


@pytest.mark.parametrize("lattice,K", [(0, 2), (0, 3), (0, 4), (0, 5), (1, 2), (1, 3), (1, 4), (1, 5)])
def test_pair_counts_of_species_unions(smcx, orc, lattice, K):
    """Lattices of 2^22 cells and more count unions of two species: random
    sites, without the first or the last species, and all of one species."""
    L = (130, 131, 247)
    assert L[0] * L[1] * L[2] >= 1 << 22
    N = W.n_sites(L, lattice)
    rng = np.random.default_rng(40 + K)
    sites = rng.integers(0, K, N, dtype=np.uint8)
    for S in (1, 2, 3):
        epi = folded_epi(K, S)
        for what, sigma in (("random", sites), ("no first", np.maximum(sites, 1)), ("no last", np.minimum(sites, K - 2)),
                            ("one", np.full(N, K // 2, np.uint8))):
            note(f"pair counts lattice={lattice} K={K} S={S} {what}")
            lat = smcx.Lattice(L, epi, sigma, 1, 900.0, lattice=lattice)
            try:
                assert np.array_equal(lat.sro()[1], orc.sro(L, S, K, sigma, lattice)[1])
            finally:
                lat.close()
