"""The list builder's row kernel at the edges of its staging: more candidates
than it holds at a time, more centre atoms per cell than it takes at a time,
few cells (split over work-groups) and many, inner cells (which skip the
periodic fold) and boundary ones, both entry formats."""
import numpy as np
import pytest

import synth
from oracle.neighbors import neighbors_of
from tests.gpu_helpers import compare_rows, log, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("n,edges,species", [
    (60000, (52.5, 52.5, 52.5), 2),    # 8^3 cells of 117 atoms, 3,164 candidates
    (900, (13.0, 14.0, 40.0), 3),      # two cells a side, six along z
    (5000, (33.0, 39.5, 26.1), 6),     # 5 x 6 x 4: inner cells along two sides only
    (3, (60.0, 60.0, 60.0), 1),        # more cells than the key space: mostly empty
])
def test_rows_match_definition(n, edges, species, fmt):
    from paper_2608_16329_amd import Potential
    rng = np.random.default_rng(n)
    box = np.array(edges)
    # also outside [0, L): the builder wraps
    pos = rng.uniform(-0.5, 1.5, (n, 3)) * box
    types = rng.integers(0, species, n).astype(np.int32)
    hp = synth.HParams(n_species=species)
    pot = Potential(hp, synth.random_weights(hp, 1))
    pot.set_list_format(fmt)
    pot.build_neighbors(to_dev(pos), to_dev(types), box)
    st = pot.stats()
    log(f"[rows] {n} atoms, {st['n_cells']} cells, {st['n_listed_pairs']} entries of {st['list_entry_bytes']} bytes")
    assert st["list_entry_bytes"] == (4 if fmt else 2)
    atoms = np.unique(np.linspace(0, n - 1, 400).astype(np.int64))
    got = pot.neighbor_rows(atoms)
    compare_rows(got, neighbors_of(pos, box, hp.cutoff + hp.skin, atoms), atoms)
    for row in got:   # grouped by species, each entry once
        assert np.all(np.diff(types[row]) >= 0) and len(np.unique(row)) == len(row)
    pot.close()


def test_longest_row_and_total():
    """Row lengths: the longest and their sum against the definition."""
    from paper_2608_16329_amd import Potential
    rng = np.random.default_rng(5)
    box = np.array([20.0, 21.0, 22.0])
    pos = rng.uniform(0.0, 1.0, (700, 3)) * box
    types = rng.integers(0, 4, 700).astype(np.int32)
    hp = synth.HParams(n_species=4)
    pot = Potential(hp, synth.random_weights(hp, 1))
    pot.build_neighbors(to_dev(pos), to_dev(types), box)
    rows = neighbors_of(pos, box, 6.5, range(700))
    st = pot.stats()
    pot.close()
    assert st["max_row"] == max(len(r) for r in rows)
    assert st["n_listed_pairs"] == sum(len(r) for r in rows)


def test_more_cells_than_one_launch_dimension():
    """Work-groups of 256 threads for each of 17 million cells are more threads
    than a launch dimension takes."""
    from paper_2608_16329_amd import Potential
    rng = np.random.default_rng(6)
    n, edge = 4_300_000, 1672.0
    box = np.full(3, edge)
    pos = np.repeat(rng.uniform(0.0, edge, (n // 4, 3)), 4, axis=0) + rng.normal(0.0, 1.5, (n, 3))
    hp = synth.HParams(n_species=1)
    pot = Potential(hp, synth.random_weights(hp, 1))
    pot.build_neighbors(to_dev(pos), to_dev(np.zeros(n, np.int32)), box)
    st = pot.stats()
    log(f"[rows] {n} atoms, {st['n_cells']} cells")
    assert st["n_cells"] * 256 > 2**32
    atoms = np.argsort(pos[:, 2])[np.linspace(0, n - 1, 25).astype(np.int64)]
    got = pot.neighbor_rows(atoms)
    pot.close()
    compare_rows(got, neighbors_of(pos, box, hp.cutoff + hp.skin, atoms), atoms)
    assert sum(len(r) for r in got) >= 50
