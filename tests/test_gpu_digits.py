"""The encoder's products on 8-bit integer digits (csrc/fused.hip), and the choice
between them and floating-point products:
weights and activations at the ends of what the digits hold - all zero, all
digits at their extreme, rows of very different size, exponents far from one -
and weights that are not finite.

Bound: a product's rounding is below 128 x 2^-53 of (largest weight of the
row) x (largest activation of the column), 1.4e-14; the outputs pass through
three such layers and sums of partial forces that cancel by at most about ten,
so they agree with the oracle to 1e-12 of an output's largest value.  float32
sums are rounded to 24 bits: 128 x 2^-24 and the same factor, 1e-4."""
import numpy as np
import pytest

import synth
from oracle.model import Model, evaluate
from tests.gpu_helpers import gpu_eval, log, to_dev

pytestmark = pytest.mark.gpu

TOL = {64: 1e-12, 32: 1e-4}


def _edit(hp, weights, change):
    """Blob with change(name, values) applied to each segment."""
    out, pos = np.array(weights, copy=True), 0
    for name, n, _ in synth.weight_segments(hp):
        change(name, out[pos:pos + n])
        pos += n
    return out


def _zero_columns(name, v):
    # a zero first layer gives zero activations, so the digits of a whole chunk are zero
    if name.startswith("enc1.") and name[5:] in ("w0", "b0"):
        v[:] = 0.0


def _zero_rows(name, v):
    if name.startswith("enc") and name.endswith(".W1"):
        v.reshape(128, 128)[::3] = 0.0
    if name.startswith("enc") and name.endswith(".Wout"):
        v.reshape(-1, 128)[1::4] = 0.0


def _extreme_digits(name, v):
    # equal weights of 128/255 = 0.808080...(256) of a row's top, and one top
    # value: every digit of the others is at its most negative
    if name.startswith("enc") and (name.endswith(".W1") or name.endswith(".W2")):
        v[:] = -(128.0 / 255.0) / 64.0
        v.reshape(128, 128)[:, 5] = 0.99 / 64.0


def _uneven_rows(name, v):
    if name.startswith("enc") and name.endswith(".W1"):
        v.reshape(128, 128)[:] *= (10.0 ** np.linspace(-12.0, 1.0, 128))[:, None]


def _small_rows(name, v):
    if name.startswith("enc") and name.endswith(".W1"):
        v.reshape(128, 128)[:] *= (10.0 ** np.linspace(-12.0, 0.0, 128))[:, None]


def _far_exponents(name, v):
    # activations of 1e100, weights that bring them back
    if not name.startswith("enc"):
        return
    if name[5:] in ("w0", "b0"):
        v *= 1e100
    elif name.endswith(".W1") or name.endswith(".W2") or name.endswith(".Wout"):
        v *= 1e-100


@pytest.mark.parametrize("change", [_zero_columns, _zero_rows, _extreme_digits, _uneven_rows, _small_rows,
                                    _far_exponents],
                         ids=lambda f: f.__name__[1:])
@pytest.mark.parametrize("k,fusion,precision", [(16, 0, 64), (32, 0, 64), (32, 1, 64), (64, 0, 64), (16, 0, 32),
                                                (32, 0, 32), (32, 1, 32), (64, 0, 32)])
def test_digits_match_oracle(change, k, fusion, precision):
    if precision == 32 and change is _far_exponents:
        pytest.skip("1e100 is not a float32")
    w = synth.make_workload("fcc-binary-4", seed=31, hp_overrides={"k": k, "precision": precision})
    weights = _edit(w.hp, w.weights, change)
    log(f"[digits] {change.__name__} k={k} fusion={fusion} float{precision}")
    ref = evaluate(Model(w.hp, weights), w.pos, w.types, w.box)
    got = gpu_eval(w.hp, weights, w.pos, w.types, w.box, fusion=fusion)
    got["pot"].close()
    for key in ("E_i", "F", "virial"):
        scale = np.abs(ref[key]).max()
        assert np.isfinite(scale) and scale > 0
        err = np.abs(got[key] - ref[key]).max() / scale
        log(f"[digits] {change.__name__} k={k} {key}: {err:.2e}")
        assert err <= TOL[precision], (key, err)


def _large_unit(layer, factor):
    """One hidden unit made `factor` times as large where it is formed (layer 0:
    the first one, 1: the second) and its weights in the layers after it 1/factor
    times: about the same outputs."""
    def change(name, v):
        if not name.startswith("enc"):
            return
        segment = name.split(".")[1]
        if segment == ("w0", "W1")[layer]:
            v.reshape(128, -1)[7] *= factor
        elif segment == ("b0", "b1")[layer]:
            v[7] *= factor
        elif segment in (("W1", "W2", "Wout"), ("W2", "Wout"))[layer]:
            v.reshape(-1, 128)[:, 7] /= factor
    return change


def _few_weights(name, v):
    # rows that use one hidden unit only, each another one
    if name.startswith("enc") and name.endswith(".W1"):
        m = v.reshape(128, 128)
        m[:] = np.diag(np.linspace(0.1, 1.0, 128))


def _table_bytes(hp, digits):
    row = (128 * (7 if hp.precision == 64 else 4) // (hp.precision // 8) + 2) if digits else 129
    return hp.n_species ** 2 * (2 * 128 + (128 * (hp.enc_hidden - 1) + hp.k) * row) * hp.precision // 8


def _uses_digits(hp, weights):
    """Whether the encoder's products run on digits for these weights, from the
    size of the context's tables against one with ordinary weights."""
    from paper_2608_16329_amd import Potential
    sizes = []
    for w in (weights, synth.random_weights(hp, 3)):
        pot = Potential(hp, w)
        sizes.append(pot.memory_bytes())
        pot.close()
    assert sizes[0] - sizes[1] in (0, _table_bytes(hp, False) - _table_bytes(hp, True))
    return sizes[0] == sizes[1]


# Floating-point products do not care about such a unit: their outputs differ
# from float64 by up to 2.6e-6 (float32) and from the oracle by up to 4.9e-15
# (float64) of their 2-norm, whatever the factor.  Allowed: twice that.
NORM = {32: 5.2e-6, 64: 1e-14}


@pytest.mark.parametrize("layer", [0, 1])
@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("factor", [1.0, 30.0, 1e2, 1e3, 1e4, 1e6])
def test_units_of_unequal_size(precision, factor, layer):
    w = synth.make_workload("fcc-binary-4", seed=31, hp_overrides={"precision": precision})
    weights = _edit(w.hp, w.weights, _large_unit(layer, factor))
    ref = evaluate(Model(w.hp, weights), w.pos, w.types, w.box)
    digits = _uses_digits(w.hp, weights)
    log(f"[digits] unit of layer {layer} x {factor:g} float{precision}: {'digits' if digits else 'floating point'}")
    assert digits or factor > 1.0
    assert not digits or factor < 1e3
    got = gpu_eval(w.hp, weights, w.pos, w.types, w.box)
    got["pot"].close()
    for key in ("E_i", "F", "virial"):
        err = np.linalg.norm(got[key] - ref[key]) / np.linalg.norm(ref[key])
        log(f"[digits] {key}: {err:.2e}")
        assert err <= NORM[precision], (key, err)


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("over,fusion,scatter", [
    ({"k": 16}, 0, 0), ({}, 0, 0), ({"k": 64}, 0, 0), ({"angular": 1}, 0, 0), ({"k": 16, "lmax": 5}, 0, 0),
    ({"lmax": 5}, 0, 0), ({"k": 64, "lmax": 4}, 0, 0), ({}, 1, 0), ({}, 2, 0), ({}, 3, 0), ({}, 0, 1),
    ({"enc_hidden": 1}, 0, 0), ({"enc_hidden": 5}, 0, 0), ({"enc_cond": 1}, 0, 0)])
def test_floating_point_encoder_matches_oracle(over, fusion, scatter, precision):
    """Every instantiation of the kernel with floating-point products, reached
    by one large unit."""
    import torch
    from paper_2608_16329_amd import Potential
    w = synth.make_workload("fcc-binary-4", seed=31, hp_overrides=dict(over, precision=precision))
    weights = _edit(w.hp, w.weights, _large_unit(0, 1e5))
    log(f"[digits] floating point {over} fusion {fusion} scatter {scatter} float{precision}")
    ref = evaluate(Model(w.hp, weights), w.pos, w.types, w.box)
    pot = Potential(w.hp, weights)
    pot.set_fusion(fusion)
    pot.set_scatter(scatter)
    pos = to_dev(w.pos)
    pot.build_neighbors(pos, to_dev(w.types.astype(np.int32)), w.box)
    F = torch.empty_like(pos)
    E = torch.empty(len(pos), dtype=torch.float64, device="cuda:0")
    V = torch.empty((len(pos), 9), dtype=torch.float64, device="cuda:0")
    pot.compute(pos, F, E, V)
    got = {"E_i": E.cpu().numpy(), "F": F.cpu().numpy(), "virial": V.cpu().numpy()}
    pot.close()
    for key, out in got.items():
        err = np.abs(out - ref[key]).max() / np.abs(ref[key]).max()
        log(f"[digits] {key}: {err:.2e}")
        assert err <= TOL[precision], (key, err)


@pytest.mark.parametrize("change,digits", [
    (_zero_columns, (64, 32)), (_zero_rows, (64, 32)), (_extreme_digits, (64, 32)), (_small_rows, (64, 32)),
    (_uneven_rows, (32,)), (_few_weights, ())], ids=lambda f: f.__name__[1:] if callable(f) else None)
def test_choice_of_products(change, digits):
    """What the row and column scales absorb stays on digits; rows up to ten
    times the others leave hidden units of as unequal a size, which float32's
    digits hold; rows that hang on one unit, far from the column's largest, do
    not stay on digits."""
    for precision in (64, 32):
        w = synth.make_workload("fcc-binary-4", seed=31, hp_overrides={"precision": precision})
        used = _uses_digits(w.hp, _edit(w.hp, w.weights, change))
        log(f"[digits] {change.__name__} float{precision}: {used}")
        assert used == (precision in digits)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("segment", ["enc3.W1", "enc3.Wout", "enc3.w0"])
@pytest.mark.parametrize("precision", [64, 32])
def test_non_finite_weights_show(bad, segment, precision):
    """A NaN or infinite weight of the table of pairs (1, 1) makes the energy of
    every atom of species 1 non-finite and leaves species 0 alone."""
    w = synth.make_workload("fcc-binary-4", seed=32, hp_overrides={"precision": precision})

    def change(name, v):
        if name == segment:
            v[7] = bad
    weights = _edit(w.hp, w.weights, change)
    log(f"[digits] {segment} {bad}")
    got = gpu_eval(w.hp, weights, w.pos, w.types, w.box)
    got["pot"].close()
    clean = evaluate(Model(w.hp, w.weights), w.pos, w.types, w.box)
    one = w.types == 1
    assert not np.isfinite(got["E_i"][one]).any()
    assert np.abs(got["E_i"][~one] - clean["E_i"][~one]).max() <= (1e-9 if precision == 64 else 1e-4 * np.abs(clean["E_i"]).max())
