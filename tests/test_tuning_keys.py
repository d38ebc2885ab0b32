"""Keys of the tuning cache (host only): a shape found for a plan with real weights is not given to one with complex
weights, whose kernel has other forms."""
import numpy as np
import pytest

import workloads as W
from paper_2606_02169_amd import _lib as L
from paper_2606_02169_amd import tuning


def key(m, dtype=L.MRMF_DTYPE_Z):
    return tuning.signature(m.sites, m.terms, dtype, "gfx950")


def with_phase(m):
    """The same lattice with a phase on its exchange terms."""
    ph = {W.OP_RAISE: np.exp(0.3j), W.OP_LOWER: np.exp(-0.3j)}
    return W.Model(m.sites, [W.Term(t.site_a, t.op_a, t.site_b, t.op_b, t.param, complex(t.w) * ph.get(t.op_a, 1.0))
                             for t in m.terms], m.theta)


MODELS = {"ring": lambda: W.ferrimagnetic_ring(20), "square": lambda: W.square_lattice_spin1(4, np.random.default_rng(3)),
          "chain": lambda: W.heisenberg_chain(12)}


@pytest.mark.parametrize("name", list(MODELS))
@pytest.mark.parametrize("dtype", [L.MRMF_DTYPE_Z, L.MRMF_DTYPE_C])
def test_shipped_shapes_by_kind_of_weights(name, dtype, tmp_path, monkeypatch):
    monkeypatch.setenv("MRMF_TUNE_CACHE", str(tmp_path / "none.json"))
    m = MODELS[name]()
    real, cplx = tuning.lookup(key(m, dtype)), tuning.lookup(key(with_phase(m), dtype))
    assert real["variant"] == L.MRMF_VARIANT_WINDOW and real["D"] == m.dim
    assert cplx["variant"] in (L.MRMF_VARIANT_MASKED, L.MRMF_VARIANT_LIST) and cplx["D"] == m.dim


def test_weights_change_the_key_only_by_kind():
    m = W.ferrimagnetic_ring(8)
    scaled = W.Model(m.sites, [W.Term(t.site_a, t.op_a, t.site_b, t.op_b, t.param, 2 * t.w) for t in m.terms], m.theta)
    tuples = W.Model(m.sites, [(t.site_a, t.op_a, t.site_b, t.op_b, t.param, t.w) for t in m.terms], m.theta)
    assert key(m) == key(scaled) == key(tuples) != key(with_phase(m))
    assert key(m) != key(m, L.MRMF_DTYPE_C)
