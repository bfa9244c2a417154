"""GPU parity of the per-cell multipole moments against the FP64 oracle.

Both sides take the same float offsets, compute in double and round each
moment once to float; they may sum in a different rounding order, so the bar
is two float ulps of the moment plus 1e-12 of the sum of |terms| (the scale
of any cancellation), and the count moment M_000 is exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_1810_02916_amd import nearfield as nfp
from paper_1810_02916_amd.synth import WORKLOADS, clustered_box, make_box

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _check(pos, K, L, p):
    b = nfp.bin_particles(torch.from_numpy(np.ascontiguousarray(pos)).to(DEV), K, L, 0.01)
    got = nfp.multipoles(b, p).cpu().numpy().astype(np.float64)
    ref, ref32 = oracle.multipoles(pos, K, L, p)
    absm = oracle.abs_moments(pos, K, L, p)
    assert got.shape == ref.shape
    np.testing.assert_array_equal(got[:, 0], ref[:, 0])
    tol = 2.0 ** -22 * np.abs(ref32.astype(np.float64)) + 1e-12 * absm
    bad = np.abs(got - ref32.astype(np.float64)) > tol
    assert not bad.any(), (np.argwhere(bad)[:5], got[bad][:5], ref32[bad][:5])


@pytest.mark.parametrize("p", [0, 1, 4, 8])
@pytest.mark.parametrize("name", ["uniform32k", "clustered262k"])
def test_multipoles_match_oracle(name, p):
    sp = WORKLOADS[name]
    print(f"[multipoles] {name} p={p}", flush=True)
    _check(make_box(sp), sp.K, sp.L, p)


def test_multipoles_dense_cells_and_wrapping():
    """Cells with hundreds of particles (several 64-particle chunks inside one
    batch), empty batches, positions outside [0, L)."""
    K, L = 5, 2.0
    rng = np.random.default_rng(71)
    h = L / K
    base = clustered_box(600, 9, K, L, 1.5, 0.5, seed=71)
    dense = (np.array([1, 3, 4]) + rng.uniform(0, 1, size=(333, 3))) * h
    far = rng.uniform(-3 * L, 4 * L, size=(100, 3))
    pos = np.concatenate([base, dense, far])[rng.permutation(1033)]
    _check(pos, K, L, 8)


def test_multipoles_batched_and_empty_box():
    specs = [(clustered_box(5000, 16, 12, 1.0, 1.5, 0.5, seed=5), 12, 1.0),
             (np.zeros((0, 3)), 7, 1.0),
             (clustered_box(9000, 20, 9, 3.0, 1.0, 0.5, seed=6), 9, 3.0)]
    b = nfp.bin_particles_batched([torch.from_numpy(p).to(DEV) for p, _, _ in specs],
                                  [K for _, K, _ in specs], [L for _, _, L in specs],
                                  [0.01] * len(specs))
    got = nfp.multipoles(b, 6)
    for (pos, K, L), g in zip(specs, got):
        g = g.cpu().numpy().astype(np.float64)
        if len(pos) == 0:
            np.testing.assert_array_equal(g, 0.0)
            assert g.shape == (K ** 3, nfp.multipole_terms(6))
            continue
        ref, ref32 = oracle.multipoles(pos, K, L, 6)
        absm = oracle.abs_moments(pos, K, L, 6)
        tol = 2.0 ** -22 * np.abs(ref32.astype(np.float64)) + 1e-12 * absm
        assert (np.abs(g - ref32) <= tol).all()


@pytest.mark.parametrize("p", [1, 8])
def test_multipoles_big_cells_in_pieces(p):
    """Cells above the piece size are summed in pieces and combined: cells of
    exactly one piece (512), one past it (513), two pieces (1024), one past
    (1025) and many (5000), next to small and empty cells, in two boxes of
    one batch."""
    K, L = 6, 1.0
    h = L / K
    rng = np.random.default_rng(90 + p)
    sizes = {(0, 0, 0): 512, (0, 0, 1): 513, (2, 5, 5): 1024, (3, 3, 3): 1025, (5, 5, 4): 5000,
             (1, 1, 1): 7}
    parts = [(np.array(c) + rng.uniform(0, 1, size=(n, 3))) * h for c, n in sizes.items()]
    pos = np.concatenate(parts + [rng.uniform(0, L, size=(300, 3))])
    pos = pos[rng.permutation(len(pos))]
    _check(pos, K, L, p)
    other = clustered_box(4000, 12, 7, 1.0, 1.5, 0.5, seed=9)
    b = nfp.bin_particles_batched([torch.from_numpy(other).to(DEV), torch.from_numpy(pos).to(DEV)],
                                  [7, K], [1.0, L], [0.01, 0.01])
    got = nfp.multipoles(b, p)
    for (q, KK, LL), g in zip([(other, 7, 1.0), (pos, K, L)], got):
        ref, ref32 = oracle.multipoles(q, KK, LL, p)
        absm = oracle.abs_moments(q, KK, LL, p)
        tol = 2.0 ** -22 * np.abs(ref32.astype(np.float64)) + 1e-12 * absm
        g = g.cpu().numpy().astype(np.float64)
        np.testing.assert_array_equal(g[:, 0], ref[:, 0])
        assert (np.abs(g - ref32) <= tol).all()


@pytest.mark.parametrize("p", [2, 3, 5, 8])
def test_multipoles_cells_around_chunk_run_and_piece_sizes(p):
    """Cell counts around a staged chunk (32), a group of four, and a piece
    (256), between runs of empty cells, and a box without particles."""
    K, L = 6, 1.0
    counts = [0, 1, 3, 4, 5, 0, 0, 31, 32, 33, 63, 65, 0, 255, 256, 257, 0, 511, 512, 513]
    rng = np.random.default_rng(81)
    parts = [(np.array([c // 36, c // 6 % 6, c % 6]) + rng.uniform(0, 1, (counts[c % 20], 3))) / K
             for c in range(60)]
    pos = np.concatenate(parts)
    _check(pos[rng.permutation(len(pos))], K, L, p)
    empty = nfp.bin_particles(torch.empty((0, 3), dtype=torch.float64, device=DEV), K, L, 0.01)
    assert (nfp.multipoles(empty, p) == 0).all()


@pytest.mark.parametrize("K", [6, 104])
def test_multipoles_many_pieces_of_one_cell(K):
    """Cells of 16, 17, 32, 33 and 79 pieces (a thread or its wave lists them,
    16 at a time are added), the largest one first or last, on a coarse grid
    and on one whose planning blocks cover 4096 cells."""
    rng = np.random.default_rng(83)
    cells = {0: 20000, 1: 4096, 2: 4097, K: 8192, K + 1: 8193, K ** 3 - 2: 257,
             K ** 3 - 1: 20000, K ** 3 // 2: 300}
    parts = [(np.array([c // K ** 2, c // K % K, c % K]) + rng.uniform(0, 1, (n, 3))) / K
             for c, n in cells.items()]
    pos = np.concatenate(parts + [rng.uniform(0, 1, (3000, 3))])
    print(f"[multipoles] pieces K={K}", flush=True)
    _check(pos[rng.permutation(len(pos))], K, 1.0, 2)


def test_multipoles_of_uneven_boxes_equal_the_single_calls_bitwise():
    """A batch of empty, tiny, sparse, large and one-cell boxes in any order:
    every box's moments are those of the box alone."""
    one_cell = (np.array([5, 0, 5]) + np.random.default_rng(3).uniform(0, 1, (700, 3))) / 6
    specs = [(np.zeros((0, 3)), 7), (clustered_box(5000, 16, 12, 1.0, 1.5, 0.5, seed=5), 12),
             (np.full((1, 3), 0.3), 5), (np.zeros((0, 3)), 5),
             (clustered_box(200000, 58, 32, 1.0, 1.5, 0.5, seed=6), 32), (one_cell, 6),
             (np.random.default_rng(4).uniform(0, 1, (900, 3)), 40), (np.zeros((0, 3)), 20)]
    for order in (specs, specs[::-1]):
        pos = [torch.from_numpy(np.ascontiguousarray(p)).to(DEV) for p, _ in order]
        Ks = [K for _, K in order]
        got = nfp.multipoles(nfp.bin_particles_batched(pos, Ks, [1.0] * len(Ks),
                                                       [0.01] * len(Ks)), 4)
        for x, K, g in zip(pos, Ks, got):
            assert torch.equal(g, nfp.multipoles(nfp.bin_particles(x, K, 1.0, 0.01), 4))


def test_multipoles_of_the_finest_grids():
    """1024^3 cells: the launch passes what one grid dimension can hold (33 GB
    of cell starts, moments and workspace)."""
    K = 1024
    rng = np.random.default_rng(82)
    pos = np.concatenate([rng.uniform(0, 1, (3000, 3)),
                          (np.array([1023, 1023, 1023]) + rng.uniform(0, 1, (300, 3))) / K,
                          (np.array([0, 0, 0]) + rng.uniform(0, 1, (7, 3))) / K])
    print(f"[multipoles] K={K}", flush=True)
    b = nfp.bin_particles(torch.from_numpy(pos).to(DEV), K, 1.0, 1e-4)
    got = nfp.multipoles(b, 0)
    c = np.floor(pos * K).astype(np.int64)
    cell, n = np.unique((c[:, 0] * K + c[:, 1]) * K + c[:, 2], return_counts=True)
    assert int(torch.count_nonzero(got)) == len(cell)
    np.testing.assert_array_equal(got[torch.from_numpy(cell).to(DEV), 0].cpu().numpy(), n)
    del b, got
    torch.cuda.empty_cache()
