"""Atoms per tile of the fused kernel: systems that get fewer than the largest
number (fewer tiles than work-groups, or a last round that would be nearly
empty), up to the first that gets full tiles, against the oracle."""
import math

import numpy as np
import pytest

import synth
from oracle.model import Model
from tests.gpu_helpers import gpu_eval, log, oracle_full, oracle_sample

pytestmark = pytest.mark.gpu

TOL64, REL32 = 1e-9, 1e-4


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("edge,over", [(4, {}), (6, {}), (7, {"k": 64}), (7, {"lmax": 5}), (11, {}), (13, {})])
def test_tile_sizes_match_oracle(edge, over, precision):
    w = synth.make_workload("fcc-hea6-128", seed=41, n=edge, hp_overrides=dict(over, precision=precision))
    # an odd atom count: drop a few sites
    keep = np.arange(len(w.pos)) % 97 != 5
    pos, types = w.pos[keep], w.types[keep]
    log(f"[tiles] edge {edge} {over} float{precision}: {len(pos)} atoms")
    g = gpu_eval(w.hp, w.weights, pos, types, w.box)
    st = g["stats"]
    g["pot"].close()
    log(f"[tiles] {st['tile_atoms']} atoms per tile, {st['n_tiles']} tiles on {st['n_blocks']} work-groups")
    counts = np.bincount(types, minlength=6)
    assert st["n_tiles"] == sum(-(-int(c) // st["tile_atoms"]) for c in counts)
    if edge <= 7:
        assert st["n_blocks"] == st["n_tiles"] > len(pos) // 16
    m = Model(w.hp, w.weights)
    if len(pos) < 2000:
        E, F, V, _, _ = oracle_full(m, pos, types, w.box)
        got = (g["E_i"], g["F"], g["virial"])
    else:
        atoms = np.linspace(0, len(pos) - 1, 16).astype(np.int64)
        E, F, V = oracle_sample(m, pos, types, w.box, atoms)
        got = (g["E_i"][atoms], g["F"][atoms], g["virial"][atoms])
    for name, a, b in zip("EFV", got, (E, F, V)):
        err = np.abs(a - b).max() / (1.0 if precision == 64 else np.abs(b).max())
        log(f"[tiles] {name}: {err:.2e}")
        assert err <= (TOL64 if precision == 64 else REL32)
    assert abs(g["totals"][0] - g["E_i"].sum()) <= 1e-9 * np.abs(g["E_i"]).sum()


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("workload,edge", [("bcc-unary-32", 6), ("fcc-binary-4", 4), ("fcc-hea6-128", 9)])
def test_totals_of_many_tiles(workload, edge, precision):
    """The totals are the sums of the per-atom outputs to rounding, whatever the
    number of tiles.  A tile's own sum is six additions deep (a wavefront) at
    most, none where tiles hold one atom, and the result is rounded once; sums
    of hundreds of tiles one after the other were 5 to 15 units of 2^-53 off."""
    w = synth.make_workload(workload, seed=43, n=edge, hp_overrides={"precision": precision})
    g = gpu_eval(w.hp, w.weights, w.pos, w.types, w.box)
    tile = g["stats"]["tile_atoms"]
    g["pot"].close()
    out = np.column_stack([g["E_i"], g["virial"]])
    for k in range(10):
        exact, size = math.fsum(out[:, k]), float(np.abs(out[:, k]).sum())
        err = abs(g["totals"][k] - exact) / size * 2.0**53
        log(f"[tiles] {workload} {edge} float{precision}, {tile} atoms per tile: total {k} off by {err:.2f}")
        assert err <= (2.0 if tile == 1 else 8.0)


@pytest.mark.parametrize("precision,workload,edge,most", [
    (64, "bcc-unary-32", 32, 16),    # 65,536 atoms: 4,096 tiles of 16, 16 rounds
    (32, "bcc-unary-32", 37, 32),    # 101,306 atoms: 3,166 tiles of 32, 12.4 rounds
])
def test_full_tiles_of_a_large_system(precision, workload, edge, most):
    """Systems that give every work-group a dozen full tiles and more: as many
    atoms per tile as fit."""
    w = synth.make_workload(workload, seed=42, n=edge, hp_overrides={"precision": precision})
    g = gpu_eval(w.hp, w.weights, w.pos, w.types, w.box)
    st = g["stats"]
    g["pot"].close()
    log(f"[tiles] {len(w.pos)} atoms float{precision}: {st['tile_atoms']} per tile, {st['n_tiles']} tiles")
    assert -(-len(w.pos) // most) >= 12 * st["n_blocks"]
    assert st["tile_atoms"] == most
    atoms = np.linspace(0, len(w.pos) - 1, 16).astype(np.int64)
    E, F, V = oracle_sample(Model(w.hp, w.weights), w.pos, w.types, w.box, atoms)
    for name, a, b in zip("EFV", (g["E_i"][atoms], g["F"][atoms], g["virial"][atoms]), (E, F, V)):
        err = np.abs(a - b).max() / (1.0 if precision == 64 else np.abs(b).max())
        log(f"[tiles] {name}: {err:.2e}")
        assert err <= (TOL64 if precision == 64 else REL32)
