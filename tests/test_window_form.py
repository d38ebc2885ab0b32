"""The window form of the generated matvec (csrc/window.cpp) where its code changes: merged and split channel pairs, tables
of the uniform digits, site orders of the second pass, blocks with a ragged last wave, plans with one pass, two passes or
no uniform site.  On the CPU through the emulator (every buffer access checked to lie inside its buffer), on the GPU
through the library; c128 to 1e-12, c64 to 2e-5 of the oracle."""
import re

import numpy as np
import pytest

import workloads as W
from oracle import mf
from paper_2606_02169_amd import _lib as L
from tests import kernel_emu as E
from tests.helpers import rel_err

TOL = {np.complex128: 1e-12, np.complex64: 2e-5}


def real_random(seed, n_sites=5, max_dim=2000, **kw):
    """Random mixed spin/boson lattice with real weights (the form's condition)."""
    m = W.random_model(np.random.default_rng(seed), n_sites=n_sites, max_dim=max_dim, n_params=3, n_terms=14, **kw)
    terms = [W.Term(t.site_a, t.op_a, t.site_b, t.op_b, t.param, complex(t.w).real) for t in m.terms]
    return W.Model(m.sites, terms, m.theta, name=f"real_random_{seed}")


def diagonal_only():
    sites = [W.spin_site(1), W.spin_site(2), W.boson_site(4)]
    return W.Model(sites, [W.Term(0, W.OP_Z, 2, W.OP_Z, 0, 0.7), W.Term(1, W.OP_Z2, -1, W.OP_Z, 1, -1.3)],
                   np.array([0.9, 1.1]))


MODELS = {
    "spin half ring": lambda: W.configs.staggered_xxz_ring([1] * 8),
    "spin 1 ring": lambda: W.configs.staggered_xxz_ring([2] * 6),          # both channels of a bond admitted at once
    "spins 1 and 3/2 above the tile": lambda: W.configs.open_xxz_chain([3, 3, 2, 2, 1, 2, 3, 2], np.ones(7), np.full(7, 0.7)),
    "spin 3/2 chain": lambda: W.configs.open_xxz_chain([3, 1, 3, 2, 3], np.ones(4), np.full(4, 0.7)),  # factor tables
    "ferrimagnet": lambda: W.ferrimagnetic_ring(8),
    "square": lambda: W.square_lattice_spin1(2, np.random.default_rng(3)),  # double bonds
    "bosons": lambda: W.tavis_cummings(4, 12, rng=np.random.default_rng(4)),
    "one site": lambda: W.zero_field_splitting(3, 0.8, 0.3),
    "diagonal": diagonal_only,
    "random 1": lambda: real_random(41),
    "random 2": lambda: real_random(42),
}
SHAPES = [(0, -1, {}), (1, 0, {}), (2, 1, {"schedule": 1, "load_group": 2}), (1, 2, {"addressing": 1}),
          (2, 0, {"far_pass": 10}), (1, 1, {"far_pass": 11, "addressing": 1}), (2, 0, {"unroll_top": 1, "schedule": 2})]


def shapes(m):
    return [s for s in SHAPES if s[0] + max(0, s[1]) + s[2].get("unroll_top", 0) <= len(m.sites)]


def state(m, dtype=np.complex128):
    return W.random_state(m.dim, np.random.default_rng(8)).astype(dtype)


@pytest.mark.parametrize("name", list(MODELS))
def test_emulated(name):
    m = MODELS[name]()
    ran = 0
    for inner, unrolled, tuning in shapes(m):
        for dtype in (np.complex128, np.complex64):
            x = state(m, dtype)
            try:
                passes, y = E.run_passes(m, x, inner=inner, unrolled=unrolled, tuning=tuning)
            except ValueError:  # the tile does not fit the plan
                continue
            ran += 1
            assert rel_err(y, mf.matvec(m, x.astype(np.complex128))) <= TOL[dtype], (inner, unrolled, tuning, dtype)
            assert np.all(np.isfinite(y))
    assert ran


@pytest.mark.parametrize("name", list(MODELS))
def test_every_shape_takes_the_form(name):
    """None of the shapes that the emulated and the GPU test run falls back to another form."""
    m = MODELS[name]()
    for inner, unrolled, tuning in shapes(m):
        for dtype in (L.MRMF_DTYPE_Z, L.MRMF_DTYPE_C):
            src = E.kernel_source(m, dtype, inner, unrolled, tuning={"variant": L.MRMF_VARIANT_WINDOW, **tuning})
            assert src is not None and "window form" in src, (inner, unrolled, tuning, dtype)


@pytest.mark.parametrize("far", [1, 10, 11])
def test_emulated_chebyshev_step(far):
    """One pass, and the two halves of a step."""
    m = W.ferrimagnetic_ring(8)
    x, rng = state(m), np.random.default_rng(9)
    prev, acc = W.random_state(m.dim, rng), W.random_state(m.dim, rng)
    c = 0.4 - 0.2j
    passes, (p, a) = E.run_passes(m, x, inner=3, unrolled=1, tuning={"far_pass": far}, cheb=(prev, acc, 0.7, -0.3, 0.9, c))
    want = 0.7 * mf.matvec(m, x) - 0.3 * x + 0.9 * prev
    assert passes == (1 if far == 1 else 2)
    assert rel_err(p, want) <= 1e-12 and rel_err(a, acc + c * want) <= 1e-12


def test_chosen_by_rule():
    """Real weights take the window form unless another form or one of its knobs is asked for; complex ones never do."""
    m = W.ferrimagnetic_ring(6)
    assert "window form" in E.kernel_source(m, L.MRMF_DTYPE_Z)
    for knob in ({"variant": 0}, {"variant": 1}, {"far_loads": 12}, {"outer_first": 1}, {"branch_skip": 1}):
        assert "window form" not in E.kernel_source(m, L.MRMF_DTYPE_Z, tuning=knob)
    cplx = W.Model(m.sites, m.terms + [W.Term(0, W.OP_RAISE, -1, W.OP_Z, 0, 0.3j),
                                       W.Term(0, W.OP_LOWER, -1, W.OP_Z, 0, -0.3j)], m.theta)
    assert "window form" not in E.kernel_source(cplx, L.MRMF_DTYPE_Z, tuning={"variant": 2})


def swapped_chain(n):
    """Open chain of spins 1/2 whose bonds list the lowering of their first site first."""
    terms = []
    for i in range(n - 1):
        terms += [W.Term(i, W.OP_LOWER, i + 1, W.OP_RAISE, 0, 0.5), W.Term(i, W.OP_RAISE, i + 1, W.OP_LOWER, 0, 0.5)]
    return W.Model([W.spin_site(1)] * n, terms, np.array([0.9]))


# Bonds whose two channels read 2^31 bytes or more apart: no 32-bit lane offset reaches both, so neither can share the
# other's gather.  At 27 spins of c128 (28 of c64) for a closing bond, one site more for the first bond of a chain.
FAR_PAIRS = {"ring 27 c128": (lambda: W.heisenberg_chain(27, periodic=True), L.MRMF_DTYPE_Z, (7, 3)),
             "ring 28 c64": (lambda: W.heisenberg_chain(28, periodic=True), L.MRMF_DTYPE_C, (0, -1)),
             "ferrimagnet 22 c64": (lambda: W.ferrimagnetic_ring(22), L.MRMF_DTYPE_C, (0, -1)),
             "lower first 28 c128": (lambda: swapped_chain(28), L.MRMF_DTYPE_Z, (0, -1))}


@pytest.mark.parametrize("name", list(FAR_PAIRS))
def test_far_pairs_read_each_channel_once(name):
    """No two gathers of a copy read the same rows (the channels of these lattices have offsets of their own)."""
    model, dtype, shape = FAR_PAIRS[name]
    src = E.kernel_source(model(), dtype, *shape, tuning={"variant": L.MRMF_VARIANT_WINDOW})
    assert "window form" in src
    at = {}
    for copy, base in re.findall(r"const C s(\d+)_\d+ = LD\(xs, \w+, F0 \+ \(unsigned long long\)\((-?\d+)ll\)\)", src):
        at.setdefault(copy, []).append(int(base))
    assert at
    for copy, bases in at.items():
        assert len(set(bases)) == len(bases), (copy, sorted(bases))


def test_far_pairs_emulated():
    """Rows of the ring of 27 spins 1/2 (2 GiB) whose closing bond is gathered, against the oracle: super-tiles all over
    the vector, site 0 up and down."""
    model, _, (inner, unrolled) = FAR_PAIRS["ring 27 c128"]
    m = model()
    x = np.resize(W.random_state(1000003, np.random.default_rng(12)), m.dim)
    tiles = m.dim >> (inner + unrolled)
    y = E.run(m, x, inner=inner, unrolled=unrolled, grid=tiles, tuning={"variant": L.MRMF_VARIANT_WINDOW}, blocks=(0, 8))
    rows = np.flatnonzero(~np.isnan(y.real))
    assert rows.size == 8 << (inner + unrolled) and rows[-1] >= m.dim // 2
    assert rel_err(y[rows], mf.matvec(m, x, rows=rows)) <= 1e-12


def lds_bytes(src):
    """LDS of each pass: the staged rows and the tables of the uniform digits."""
    f32 = "typedef float R" in src
    one = {"C": 8 if f32 else 16, "R": 4 if f32 else 8}
    return [sum(one[t] * int(n) for t, n in re.findall(r"__shared__ (C|R) \w+\[(\d+)\]", body))
            for body in src.split("extern \"C\" __global__")[1:]]


# lattices whose large sites leave tiles of many rows only: (lattice, default tile beyond the 160 KB of LDS in c128)
LARGE_SITES = {
    "16 and 250 levels": lambda: chain_of([W.spin_site(1)] * 10 + [W.boson_site(15), W.boson_site(249), W.spin_site(2)]),
    "12 and 256 levels": lambda: chain_of([W.spin_site(1)] * 10 + [W.boson_site(11), W.boson_site(255), W.spin_site(3)]),
    "15 and 200 levels": lambda: chain_of([W.spin_site(1)] * 10 + [W.boson_site(14), W.boson_site(199), W.spin_site(3)]),
}


def chain_of(sites):
    """Open chain with one exchange coupling per bond."""
    terms = []
    for i in range(len(sites) - 1):
        terms += [W.Term(i, W.OP_RAISE, i + 1, W.OP_LOWER, i, 0.5), W.Term(i, W.OP_LOWER, i + 1, W.OP_RAISE, i, 0.5),
                  W.Term(i, W.OP_Z, i + 1, W.OP_Z, i, 1.0)]
    return W.Model(sites, terms, np.linspace(0.6, 1.2, len(sites) - 1))


@pytest.mark.parametrize("name", list(LARGE_SITES))
@pytest.mark.parametrize("dtype", [L.MRMF_DTYPE_Z, L.MRMF_DTYPE_C, L.MRMF_SOURCE_CHEB])
def test_tile_by_rule_fits_in_lds(name, dtype):
    src = E.kernel_source(LARGE_SITES[name](), dtype)
    assert "window form" in src
    assert max(lds_bytes(src)) <= 163840


def test_tile_beyond_lds_takes_the_masked_form():
    """A shape asked for whose rows do not fit in LDS: the masked form, as for any plan that the window form does not take."""
    m = LARGE_SITES["16 and 250 levels"]()
    for tuning in ({}, {"variant": L.MRMF_VARIANT_WINDOW}):
        src = E.kernel_source(m, L.MRMF_DTYPE_Z, inner=2, unrolled=1, tuning=tuning)
        assert src is not None and "window form" not in src
    assert "window form" in E.kernel_source(m, L.MRMF_DTYPE_Z, inner=2, unrolled=0)


def pairs(sites, reach, per_bond=False, ring=False, by_site=False):
    """Couplings of sites up to `reach` apart: one pair (J_xy, J_z) for all bonds, or one a bond; bonds by distance, or
    site by site."""
    n, terms, theta = len(sites), [], [1.0, 0.8]
    bonds = [(i, (i + k) % n) for k in range(1, reach + 1) for i in range(n) if ring or i + k < n]
    for b, (i, j) in enumerate(sorted(bonds) if by_site else bonds):
        terms += W.xxz_bond_terms(i, j, 2 * b, 2 * b + 1) if per_bond else W.xxz_bond_terms(i, j, 0, 1)
    return W.Model(sites, terms, np.array(theta * (b + 1) if per_bond else theta))


# (lattice, window form by rule in c128, in c64): both sides of each line of the rule
RULE = {
    "16 spins 1/2, range 3": (lambda: pairs([W.spin_site(1)] * 16, 3, ring=True), True, True),
    "16 spins 1/2, range 4, a coupling a bond": (lambda: pairs([W.spin_site(1)] * 16, 4, True, True), False, False),
    "18 spins 1/2, range 4, a coupling a bond": (lambda: pairs([W.spin_site(1)] * 18, 4, True, True), True, True),
    "16 spins 1/2, all pairs": (lambda: pairs([W.spin_site(1)] * 16, 15), True, True),
    "18 spins 1/2, all pairs, a coupling a bond": (lambda: pairs([W.spin_site(1)] * 18, 17, True), True, True),
    "18 spins 1/2, all pairs site by site, a coupling a bond": (lambda: pairs([W.spin_site(1)] * 18, 17, True, by_site=True),
                                                                False, True),
    "18 spins 1/2, range 8, a coupling a bond": (lambda: pairs([W.spin_site(1)] * 18, 8, True, True), True, True),
    "20 spins 1/2, all pairs, a coupling a bond": (lambda: pairs([W.spin_site(1)] * 20, 19, True), True, True),
    "10 spins 1, all pairs, a coupling a bond": (lambda: pairs([W.spin_site(2)] * 10, 9, True), True, True),
    "10 spins 3/2": (lambda: pairs([W.spin_site(3)] * 10, 1, ring=True), True, True),
    "10 spins 3/2, range 2": (lambda: pairs([W.spin_site(3)] * 10, 2, ring=True), False, True),
    "12 spins 1/2 around a mode of 21 levels": (lambda: W.tavis_cummings(12, 20, rng=np.random.default_rng(5)), True, True),
    "12 spins 1/2 around a mode of 65 levels": (lambda: W.tavis_cummings(12, 64, rng=np.random.default_rng(5)), False, False),
    "14 spins 1/2 around a mode of 65 levels": (lambda: W.tavis_cummings(14, 64, rng=np.random.default_rng(5)), True, True),
    "8 spins 3/2, range 2": (lambda: pairs([W.spin_site(3)] * 8, 2, ring=True), False, False),
}


@pytest.mark.parametrize("name", list(RULE))
def test_form_of_plans_with_many_terms(name):
    model, z, c = RULE[name]
    m = model()
    for dtype, window in ((L.MRMF_DTYPE_Z, z), (L.MRMF_DTYPE_C, c)):
        assert ("window form" in E.kernel_source(m, dtype)) == window, dtype
        # asked for, it is taken all the same
        assert "window form" in E.kernel_source(m, dtype, tuning={"variant": L.MRMF_VARIANT_WINDOW})


@pytest.mark.parametrize("spins,copies", [("232222332322", 3), ("121221212121212", 6)])
def test_copies_of_varied_sites(spins, copies):
    """Tile by rule of two rings of about a million rows: above the tile a spin 3/2 is not unrolled, a spin 1/2 is."""
    m = pairs([W.spin_site(int(c)) for c in spins], 1, ring=True)
    src = E.kernel_source(m, L.MRMF_DTYPE_Z)
    assert int(re.search(r"(\d+) unrolled copies", src).group(1)) == copies


@pytest.mark.parametrize("spins,rows,copies", [("23223223322", 432, 3), ("312312312312", 144, 4), ("2222222222", 243, 1)])
def test_c64_tiles_of_one_copy(spins, rows, copies):
    """Tile by rule in c64: one copy of many rows is not taken where there is a tile of several."""
    m = pairs([W.spin_site(int(c)) for c in spins], 1)
    src = E.kernel_source(m, L.MRMF_DTYPE_C)
    assert re.search(r"(\d+) rows per block, (\d+) unrolled copies", src).groups() == (str(rows), str(copies))


@pytest.mark.parametrize("n,z,c", [(18, 1, 1), (19, 2, 1), (20, 2, 2)])
def test_passes_by_the_size_of_the_vector(n, z, c):
    """All pairs of spins 1/2: a second launch from vectors of 8 MB on (18 spins of c128 are 4 MB), unless asked for."""
    m = pairs([W.spin_site(1)] * n, n - 1)
    for dtype, passes in ((L.MRMF_DTYPE_Z, z), (L.MRMF_DTYPE_C, c)):
        assert len(E.launch_shapes(E.kernel_source(m, dtype))) == passes
        assert len(E.launch_shapes(E.kernel_source(m, dtype, tuning={"far_pass": 1}))) == 1
        assert len(E.launch_shapes(E.kernel_source(m, dtype, tuning={"far_pass": 18}))) == 2


@pytest.mark.parametrize("model,window", [
    (lambda: pairs([W.spin_site(1)] * 14, 13), True), (lambda: pairs([W.spin_site(1)] * 16, 2, True, True), False),
    (lambda: pairs([W.spin_site(1)] * 18, 17), False), (lambda: pairs([W.spin_site(1)] * 20, 19), True),
    (lambda: pairs([W.spin_site(1)] * 16, 15), True), (lambda: pairs([W.spin_site(3)] * 8, 1, ring=True), True),
    (lambda: W.ferrimagnetic_ring(8), True)])
def test_form_of_the_chebyshev_step(model, window):
    """Its own lines of the rule, on plans whose matvec takes the window form."""
    m = model()
    assert "window form" in E.kernel_source(m, L.MRMF_DTYPE_Z)
    assert ("window form" in E.kernel_source(m, L.MRMF_SOURCE_CHEB)) == window


@pytest.mark.parametrize("spin,bonds", [(1, 1), (3, 1), (3, 3), (1, 8), (3, 9), (2, 20)])
def test_tables_with_many_addends(spin, bonds):
    """Entries of the tables of the uniform digits that are a sum over `bonds` couplings: below, at and above the
    number that is read together, in one round of the block and in several."""
    terms, theta = [], []
    for k in range(5 * bonds):
        terms += W.xxz_bond_terms(k % 5, k % 5 + 1, 2 * k, 2 * k + 1)
        theta += [1.0 + 0.01 * k, 0.8 - 0.02 * k]
    m = W.Model([W.spin_site(spin)] * 6, terms, np.array(theta))
    for dtype in (np.complex128, np.complex64):
        x = state(m, dtype)
        for inner, unrolled in ((2, 0), (2, 1), (3, 0)):
            _, y = E.run_passes(m, x, inner=inner, unrolled=unrolled, tuning={"variant": L.MRMF_VARIANT_WINDOW})
            assert rel_err(y, mf.matvec(m, x.astype(np.complex128))) <= TOL[dtype] * bonds


@pytest.mark.parametrize("n", [20, 24, 26])
def test_gathers_of_all_copies_are_bounded(n):
    """Couplings of all pairs: the kernel by rule does not grow with copies times channels.  720 and 1440 by the rule's
    count, half of a copy's channels; a copy's own digits leave up to a third more of them."""
    m = pairs([W.spin_site(1)] * n, n - 1)
    for dtype, most in ((L.MRMF_DTYPE_Z, 720), (L.MRMF_DTYPE_C, 1440)):
        first = E.kernel_source(m, dtype).split('extern "C" __global__')[1]
        gathers = re.findall(r"const C s(\d+)_\d+ = LD", first)
        assert len(set(gathers)) > 1 and len(gathers) <= most * 4 / 3


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(LARGE_SITES))
def test_gpu_large_sites(name):
    """The default kernel of these plans is a specialized one, and its rows are the oracle's."""
    import torch

    from paper_2606_02169_amd.plan import Plan
    m = LARGE_SITES[name]()
    rows = np.unique(np.random.default_rng(2).integers(0, m.dim, 2000))
    for dtype, tdt in ((np.complex128, torch.float64), (np.complex64, torch.float32)):
        x = np.resize(W.random_state(1000003, np.random.default_rng(12)), m.dim).astype(dtype)
        p = Plan.from_model(m)
        p.set_kernel("specialized")
        y = p.matvec(torch.as_tensor(m.theta, dtype=tdt, device="cuda"), torch.from_numpy(x).cuda())
        assert p.kernel_info(y.dtype)["kind"] == "specialized"
        ref = mf.matvec(m, x.astype(np.complex128), rows=rows)
        assert rel_err(y[torch.from_numpy(rows).cuda()].cpu().numpy(), ref) <= TOL[dtype]


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(MODELS))
def test_gpu(name):
    import torch

    from paper_2606_02169_amd.plan import Plan
    m = MODELS[name]()
    for inner, unrolled, tuning in shapes(m):
        for dtype, tdt in ((np.complex128, torch.float64), (np.complex64, torch.float32)):
            p = Plan.from_model(m)
            p.set_kernel("auto", inner_sites=inner, unrolled_sites=unrolled)
            p.set_tuning(variant=2, **tuning)
            x = state(m, dtype)
            th = torch.as_tensor(m.theta, dtype=tdt, device="cuda")
            print(name, inner, unrolled, tuning, dtype.__name__, flush=True)
            y = p.matvec(th, torch.from_numpy(x).cuda()).cpu().numpy()
            assert rel_err(y, mf.matvec(m, x.astype(np.complex128))) <= TOL[dtype]


@pytest.mark.gpu
def test_gpu_two_passes_of_the_square_lattice():
    """The 4 x 4 lattice (43 million rows), which takes a second pass by rule, and one pass forced: the same vector."""
    import torch

    from paper_2606_02169_amd.plan import Plan
    m = W.square_lattice_spin1(4, np.random.default_rng(3))
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.view_as_complex(torch.randn((m.dim, 2), dtype=torch.float64, device="cuda", generator=g))
    th = torch.as_tensor(m.theta, dtype=torch.float64, device="cuda")
    two, one = Plan.from_model(m), Plan.from_model(m)
    one.set_tuning(far_pass=1)
    y2, y1 = two.matvec(th, x), one.matvec(th, x)
    assert "mrmf_spec_b" in two.kernel_source() and "mrmf_spec_b" not in one.kernel_source()
    assert float((y2 - y1).abs().max()) <= 1e-13 * float(y1.abs().max())
    rows = np.unique(np.random.default_rng(2).choice(m.dim, 2000, replace=False)).astype(np.int64)
    ref = mf.matvec(m, x.cpu().numpy(), rows=rows)
    assert rel_err(y2[torch.from_numpy(rows).cuda()].cpu().numpy(), ref) <= 1e-12


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(FAR_PAIRS))
def test_gpu_far_pairs(name):
    """The whole vector against the generic kernel's; a row sums at most 2 x 28 products, so 1e-14 (c128) and 1e-5 (c64)
    of the largest entry leave room for two orders of the roundings."""
    import torch

    from paper_2606_02169_amd.plan import Plan
    model, dtype, (inner, unrolled) = FAR_PAIRS[name]
    m = model()
    real = torch.float32 if dtype == L.MRMF_DTYPE_C else torch.float64
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.view_as_complex(torch.randn((m.dim, 2), dtype=real, device="cuda", generator=g))
    th = torch.as_tensor(m.theta, dtype=real, device="cuda")
    win, gen = Plan.from_model(m), Plan.from_model(m)
    win.set_kernel("specialized", inner_sites=inner, unrolled_sites=unrolled)
    gen.set_kernel("generic")
    assert "window form" in win.kernel_source(x.dtype)
    a, b = win.matvec(th, x), gen.matvec(th, x)
    scale = float(torch.view_as_real(b).abs().max())
    worst = max(float(torch.view_as_real(u - v).abs().max()) for u, v in zip(a.split(1 << 26), b.split(1 << 26)))
    assert worst <= (1e-5 if real == torch.float32 else 1e-14) * scale


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(MODELS))
def test_gpu_runs_the_form(name):
    """The kernel that the library builds for these shapes: specialized, of the window form, with the passes of its source."""
    import torch

    from paper_2606_02169_amd.plan import Plan
    m = MODELS[name]()
    for inner, unrolled, tuning in shapes(m):
        for dtype in (torch.complex128, torch.complex64):
            p = Plan.from_model(m)
            p.set_kernel("specialized", inner_sites=inner, unrolled_sites=unrolled)
            p.set_tuning(variant=2, **tuning)
            p.prepare(dtype)
            src, info = p.kernel_source(dtype), p.kernel_info(dtype)
            assert "window form" in src and info["kind"] == "specialized"
            assert (info["block"], info["super_tiles"]) == E.launch_shapes(src)[0]
