"""The list builder's row kernel at the edges of its staging: more candidates
than it holds at a time, more centre atoms per cell than it takes at a time,
few cells (split over work-groups) and many, inner cells (which skip the
periodic fold) and boundary ones, both entry formats."""
import time

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
    (560000, (270.0, 270.0, 270.0), 2),  # 41^3 cells: work-groups in two layers of the grid
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


def _gas_and_drop(n, edge, species, seed):
    """Half of the atoms spread over the box, half in a drop at its corner (so
    that it reaches across the boundary), some cells in between."""
    rng = np.random.default_rng(seed)
    pos = rng.uniform(0.0, edge, (n, 3))
    drop = n // 2
    pos[:drop] = rng.normal(0.0, 25.0, (drop, 3))
    order = rng.permutation(n)
    return pos[order], rng.integers(0, species, n).astype(np.int32), np.full(3, edge)


@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("n,edge,species", [
    (20000, 270.0, 1),     # 41^3 cells, the first past those that always get a work-group each
    (60000, 270.0, 3),
    (110000, 270.0, 6),
])
def test_rows_of_mostly_empty_cells(n, edge, species, fmt):
    """Many cells with few atoms on average: centres by thread or, where cells
    or neighbourhoods are full, by work-group; every row has to come from one
    of the two."""
    from paper_2608_16329_amd import Potential
    pos, types, box = _gas_and_drop(n, edge, species, n + species)
    hp = synth.HParams(n_species=species)
    pot = Potential(hp, synth.random_weights(hp, 1))
    pot.set_list_format(fmt)
    pot.build_neighbors(to_dev(pos), to_dev(types), box)
    st = pot.stats()
    off, idx = pot.neighbors()
    pot.close()
    log(f"[rows] {n} atoms, {st['n_cells']} cells, {st['n_listed_pairs']} entries, longest {st['max_row']}")
    assert st["n_cells"] * species <= 4 * n + 4096
    length = np.diff(off)
    assert length.max() == st["max_row"] > 16 and (length < 3).sum() > n // 8
    # each pair listed from both sides
    centre = np.repeat(np.arange(n), length)
    assert np.array_equal(np.sort(centre * n + idx), np.sort(idx.astype(np.int64) * n + centre))
    atoms = np.concatenate([np.argsort(length)[::max(n // 150, 1)], np.argsort(length)[-50:]])
    rows = [idx[off[i]:off[i + 1]] for i in atoms]
    compare_rows(rows, neighbors_of(pos, box, hp.cutoff + hp.skin, atoms), atoms)
    for row in rows:
        assert np.all(np.diff(types[row]) >= 0)


def test_mostly_empty_cells_are_no_dearer():
    """A gas of a million atoms, 2.2 million cells, lists in no more time than a
    crystal of as many atoms, 90 times the pairs (a work-group for every cell took
    four times as long)."""
    import torch
    from paper_2608_16329_amd import Potential
    rng = np.random.default_rng(8)
    w = synth.make_workload("fcc-hea6-128", seed=8, n=64)
    n = len(w.pos)
    took = {}
    for name, pos, types, box, species in (("crystal", w.pos, w.types, w.box, 6),
                                           ("gas", rng.uniform(0.0, 1060.0, (n, 3)), np.zeros(n), np.full(3, 1060.0), 1)):
        hp = synth.HParams(n_species=species)
        pot = Potential(hp, synth.random_weights(hp, 1))
        p, t = to_dev(pos), to_dev(types.astype(np.int32))
        times = []
        for _ in range(6):
            torch.cuda.synchronize()
            begin = time.perf_counter()
            pot.build_neighbors(p, t, box)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - begin)
        took[name] = min(times)
        log(f"[rows] {name}: {pot.stats()['n_cells']} cells, {1e6 * took[name]:.0f} us")
        pot.close()
    assert took["gas"] <= took["crystal"]


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
    """17 million cells: work-groups of 256 threads for each would be more
    threads than a launch dimension takes."""
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
