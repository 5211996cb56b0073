"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element,
on the same seeded inputs.  Bars: the q = inf aggregate is bit-exact; u and X are within
rtol 1e-5 / atol 1e-6 in fp32; the set of zeroed groups is identical."""
import numpy as np
import pytest

from oracle import mlproj_oracle as orc
from paper_2405_02086_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

RTOL, ATOL = 1e-5, 1e-6
QNAME = {"inf": "l1inf", 1: "l11", 2: "l12"}


@pytest.fixture(scope="module")
def mp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2405_02086_amd import binding
    binding.lib()            # raises if the HIP library is not built: no fallback
    return binding


@pytest.fixture
def l11_sweeps(mp):
    """Set the number of lock-step sweeps for one test; the default comes back afterwards."""
    def set_to(k):
        mp.set_l11_sweeps(k)
    yield set_to
    mp.set_l11_sweeps(0)


def run_gpu(mp, Y, eta, q, workspace=None, inplace=False):
    dev = torch.device("cuda:0")
    Yd = torch.from_numpy(Y).to(dev)
    n, m = Y.shape
    ws = workspace or mp.Workspace.for_call(QNAME[q], n, m, device=dev)
    v = torch.full((m,), -1.0, dtype=torch.float32, device=dev)
    u = torch.full((m,), -1.0, dtype=torch.float32, device=dev)
    fn = getattr(mp, "bilevel_proj_" + QNAME[q])
    X = fn(Yd, eta, X=Yd if inplace else None, workspace=ws, v_out=v, u_out=u)
    torch.cuda.synchronize()
    return {"X": X.cpu().numpy(), "v": v.cpu().numpy(), "u": u.cpu().numpy(), "res": ws.result()}


def split_call(mp, Y, eta, q):
    """bilevel_radii and bilevel_apply: the kernels of the general chain, whatever form a whole call would take."""
    Yd = torch.from_numpy(Y).to("cuda:0")
    m = Y.shape[1]
    ws = mp.Workspace.for_call(QNAME[q], *Y.shape, device=Yd.device)
    v, u = (torch.full((m,), -1.0, dtype=torch.float32, device=Yd.device) for _ in range(2))
    X = torch.empty_like(Yd)
    mp.bilevel_radii(QNAME[q], Yd, eta, ws, v_out=v)
    mp.bilevel_apply(QNAME[q], Yd, X, ws, u_out=u)
    torch.cuda.synchronize()
    return {"X": X.cpu().numpy(), "v": v.cpu().numpy(), "u": u.cpu().numpy(), "res": ws.result()}


def eta_for(Y, q, frac):
    """The radius both sides receive: a fraction of the oracle's fp64 norm, rounded to fp32."""
    return float(np.float32(frac * orc.norm_l1q(Y, q)))


def assert_close_in_row_chunks(X, R, chunk_elems=1 << 24):
    """Element by element to the fp32 bar, a block of rows at a time (the temporaries of a whole
    1 GiB comparison would be several times its size)."""
    assert X.shape == R.shape
    rows = max(1, chunk_elems // max(1, X.shape[1]))
    for r0 in range(0, X.shape[0], rows):
        np.testing.assert_allclose(X[r0:r0 + rows], R[r0:r0 + rows], rtol=RTOL, atol=ATOL)


def check_against_oracle(got, ref, q, columns=None):
    if q == "inf":
        assert np.array_equal(got["v"], ref["v"]), "column maxima must be bit-exact"
    else:
        np.testing.assert_allclose(got["v"], ref["v"].astype(np.float32), rtol=2e-7, atol=0)
    np.testing.assert_allclose(got["u"], np.asarray(ref["u"], dtype=np.float32), rtol=RTOL, atol=ATOL)
    assert np.array_equal(got["u"] == 0, np.asarray(ref["u"]) == 0), "support (zeroed columns) differs"
    assert got["res"]["tau"] == pytest.approx(ref["tau"], rel=1e-9, abs=1e-300)
    assert got["res"]["n_active"] == int((np.asarray(ref["u"], dtype=np.float64) > 0).sum())
    if columns is None:
        assert_close_in_row_chunks(got["X"], ref["X"])
        zero_cols = np.asarray(ref["u"]) == 0
        assert not got["X"][:, zero_cols].any()
    else:
        np.testing.assert_allclose(got["X"][:, columns], ref["X"][:, columns], rtol=RTOL, atol=ATOL)
    if q == 1:
        assert got["res"]["inner_pending"] == 0, "inner threshold searches did not converge"


SHAPES = [(1, 1), (1, 9), (9, 1), (7, 5), (33, 20), (256, 128), (300, 257), (131, 1028),
          (2065, 260), (33, 4100), (4100, 36), (1000, 1000)]


@pytest.mark.parametrize("q", ["inf", 1, 2])
@pytest.mark.parametrize("shape", SHAPES)
def test_bilevel_matches_oracle_on_ragged_shapes(mp, q, shape):
    rng = np.random.default_rng([shape[0], shape[1], {"inf": 0, 1: 1, 2: 2}[q]])
    Y = rng.standard_normal(shape).astype(np.float32)
    Y *= np.power(10.0, rng.uniform(-1.5, 0.0, shape[1])).astype(np.float32)[None, :]
    for frac in (0.03, 0.4, 0.97):
        eta = eta_for(Y, q, frac)
        check_against_oracle(run_gpu(mp, Y, eta, q), orc.bilevel(Y, eta, q), q)


@pytest.mark.parametrize("q", ["inf", 1, 2])
@pytest.mark.parametrize("shape", [(3, 40001), (8, 70000), (2, 16388), (40, 300000), (5, 65536), (5, 65540)])
def test_many_columns_use_the_grid_wide_search(mp, q, shape):
    """More columns than a map workgroup can search itself (m > 16384): the one-workgroup search
    with 64 values per thread up to 65536 columns, the grid-wide search beyond."""
    rng = np.random.default_rng([shape[0], shape[1], 99])
    Y = rng.laplace(size=shape).astype(np.float32)
    nrm = orc.norm_l1q(Y, q)
    for eta in (eta_for(Y, q, 0.01), eta_for(Y, q, 0.6), float(np.float32(1.01 * nrm)), 0.0):
        check_against_oracle(run_gpu(mp, Y, eta, q), orc.bilevel(Y, eta, q), q)


@pytest.mark.parametrize("m", [600, 4096, 4100, 10000, 16384])
@pytest.mark.parametrize("stride", [1, 256, 512])
def test_outer_search_with_few_groups_left(mp, m, stride):
    """The outer search starts from the root over its threads' largest values: the surviving groups lie in many threads, or
    share a few of them (stride = a workgroup's threads), close together, tied and far apart."""
    rng = np.random.default_rng([m, stride])
    base = rng.uniform(0.5, 1.0, m)
    at = (7 + stride * np.arange(min(40, (m - 8) // stride))) % m
    for lift in (1e-3, 0.5, 100.0):
        col = base.copy()
        col[at] = 1.0 + lift * np.linspace(0.0, 1.0, at.size) ** 2
        col[at[: at.size // 2]] = 1.0 + lift
        Y = np.stack([col, -0.5 * col, 0.25 * col]).astype(np.float32)
        for q in ("inf", 1, 2):
            for frac in (1e-4, 1e-3, 0.02):
                eta = eta_for(Y, q, frac)
                check_against_oracle(run_gpu(mp, Y, eta, q), orc.bilevel(Y, eta, q), q)


@pytest.mark.parametrize("limit", [0, 64])
def test_grid_wide_search_gives_up_and_the_kernel_behind_it_takes_over(mp, limit):
    """With a poll limit of 0 the several-workgroup search leaves at once and the one-workgroup
    kernel enqueued behind it does the work; with 64 some workgroups may give up half way.  Every
    kernel ends either way and the result is the same."""
    rng = np.random.default_rng(97)
    dev = torch.device("cuda:0")
    Y = rng.laplace(size=(3, 300001)).astype(np.float32)
    w = weights_for(300001, 9)
    before = mp.set_search_spin_limit(limit)
    try:
        for q in ("inf", 1):
            eta = eta_for(Y, q, 0.2)
            check_against_oracle(run_gpu(mp, Y, eta, q), orc.bilevel(Y, eta, q), q)
            eta = weighted_eta(Y, q, w, 0.2)
            check_stored(run_weighted(mp, Y, eta, q, "f32", w), orc.bilevel_stored(Y, eta, q, "f32", p=("w1", w)), q, "f32")
        T = rng.standard_normal((40000, 2, 4)).astype(np.float32)      # multi-level with a long top vector
        eta = float(np.float32(0.3 * nested_norm(T, [1, 1])))
        check_multi(run_multi(mp, T, [1, 1], eta), orc.multilevel(T, [1, 1], eta))
    finally:
        assert mp.set_search_spin_limit(before) == limit


def test_grid_wide_search_on_a_busy_gpu(mp):
    """The several-workgroup search with its default poll bound while another stream keeps the
    GPU full of the library's own long kernels (l1,1 projections of a 256 MiB matrix): whether
    its workgroups all become resident at once or some give up and the one-workgroup kernel
    takes over, every kernel ends and the result is the oracle's."""
    rng = np.random.default_rng(98)
    dev = torch.device("cuda:0")
    big = torch.from_numpy(rng.standard_normal((8192, 8192)).astype(np.float32)).to(dev)
    big_out = torch.empty_like(big)
    big_ws = mp.Workspace.for_call("l11", 8192, 8192, device=dev)
    Y = rng.laplace(size=(3, 300001)).astype(np.float32)
    eta = eta_for(Y, "inf", 0.2)
    ref = orc.bilevel_l1inf(Y, eta)
    Yd = torch.from_numpy(Y).to(dev)
    ws = mp.Workspace.for_call("l1inf", 3, 300001, device=dev)
    v = torch.empty(300001, dtype=torch.float32, device=dev)
    u = torch.empty(300001, dtype=torch.float32, device=dev)
    busy, mine = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for rep in range(3):
        for _ in range(6):
            mp.bilevel_proj_l11(big, 1000.0, X=big_out, workspace=big_ws, stream=busy)
        X = mp.bilevel_proj_l1inf(Yd, eta, workspace=ws, v_out=v, u_out=u, stream=mine)
        torch.cuda.synchronize()
        got = {"X": X.cpu().numpy(), "v": v.cpu().numpy(), "u": u.cpu().numpy(), "res": ws.result()}
        check_against_oracle(got, ref, "inf")


@pytest.mark.parametrize("q", ["inf", 1, 2])
@pytest.mark.parametrize("shape", [(50000, 3), (100000, 1), (1, 100000), (2, 20000), (70001, 65)])
def test_very_tall_and_single_row_shapes(mp, q, shape):
    """A handful of columns under many row groups (one tile, every workgroup on it), and the
    one-row matrix, where the aggregate is |Y| itself and the projection is the plain l1 one."""
    rng = np.random.default_rng([shape[0], shape[1], 5])
    Y = rng.standard_normal(shape).astype(np.float32)
    for frac in (0.02, 0.7):
        eta = eta_for(Y, q, frac)
        check_against_oracle(run_gpu(mp, Y, eta, q), orc.bilevel(Y, eta, q), q)


@pytest.mark.parametrize("q", ["inf", 1, 2])
def test_degenerate_radii_and_inputs(mp, q):
    rng = np.random.default_rng(7)
    Y = rng.standard_normal((65, 70)).astype(np.float32)
    nrm = orc.norm_l1q(Y, q)
    # inside the ball (and exactly on it when the fp32 radius rounds up): X = Y bit for bit
    for eta in (float(np.float32(2 * nrm)), float(np.nextafter(np.float32(nrm), np.float32(np.inf)))):
        got = run_gpu(mp, Y, eta, q)
        assert np.array_equal(got["X"], Y) and got["res"]["inside_ball"]
        assert got["res"]["tau"] == 0.0
    got = run_gpu(mp, Y, 0.0, q)                   # eta = 0: everything goes
    assert not got["X"].any() and not got["u"].any()
    Z = np.zeros((10, 12), dtype=np.float32)       # all-zero input
    got = run_gpu(mp, Z, 1.0, q)
    assert not got["X"].any() and not got["v"].any()
    # zero columns among live ones, negative zero kept as a zero
    Y2 = Y.copy()
    Y2[:, ::3] = 0.0
    Y2[0, 0] = -0.0
    eta = eta_for(Y2, q, 0.5)
    check_against_oracle(run_gpu(mp, Y2, eta, q), orc.bilevel(Y2, eta, q), q)
    # ties: many equal columns, threshold lands exactly on a value for q = inf
    T = np.tile(np.float32([[3, -1], [-2, 0.5]]), (8, 16))
    for eta in (16 * 2.0, 16 * 3.0, 5.0):
        check_against_oracle(run_gpu(mp, T, eta, q), orc.bilevel(T, eta, q), q)


@pytest.mark.parametrize("q", ["inf", 1, 2])
def test_inplace_repeatable_and_workspace_reuse(mp, q):
    rng = np.random.default_rng(11)
    dev = torch.device("cuda:0")
    big = mp.Workspace(max(mp.workspace_bytes(QNAME[q], 3000, 3000), mp.workspace_bytes(QNAME[q], 40, 5000)), device=dev)
    first = None
    for shape in [(3000, 1200), (40, 5000), (777, 333), (3000, 1200)]:
        Y = rng.standard_normal(shape).astype(np.float32) if shape != (3000, 1200) or first is None else first[0]
        eta = eta_for(Y, q, 0.2)
        ref = orc.bilevel(Y, eta, q)
        a = run_gpu(mp, Y, eta, q, workspace=big)
        b = run_gpu(mp, Y, eta, q, workspace=big, inplace=True)
        check_against_oracle(a, ref, q)
        assert np.array_equal(a["X"], b["X"]) and np.array_equal(a["u"], b["u"])   # bit-repeatable, aliasing ok
        if first is None:
            first = (Y, a)
        elif shape == (3000, 1200):
            assert np.array_equal(a["X"], first[1]["X"])


def test_norm_entry_point(mp):
    rng = np.random.default_rng(5)
    dev = torch.device("cuda:0")
    for shape in [(1, 1), (50, 70), (1025, 513)]:
        Y = rng.standard_normal(shape).astype(np.float32)
        Yd = torch.from_numpy(Y).to(dev)
        for q in ("inf", 1, 2):
            v = torch.empty(shape[1], dtype=torch.float32, device=dev)
            got = mp.norm_l1q(Yd, QNAME[q], v_out=v)
            assert got == pytest.approx(orc.norm_l1q(Y, q), rel=1e-12)
            np.testing.assert_allclose(v.cpu().numpy(), orc.column_norms(Y, q).astype(np.float32), rtol=2e-7)


# ------------------------------------------------------------------ tri-level
def run_tri(mp, Y, eta):
    dev = torch.device("cuda:0")
    Yd = torch.from_numpy(Y).to(dev)
    d0 = Y.shape[0]
    ws = mp.Workspace.for_call("tri", *Y.shape, device=dev)
    v = torch.full((d0,), -1.0, dtype=torch.float32, device=dev)
    u = torch.full((d0,), -1.0, dtype=torch.float32, device=dev)
    X = mp.trilevel_proj_l1infinf(Yd, eta, workspace=ws, v_out=v, u_out=u)
    torch.cuda.synchronize()
    return {"X": X.cpu().numpy(), "v": v.cpu().numpy(), "u": u.cpu().numpy(), "res": ws.result()}


def check_tri(got, ref):
    assert np.array_equal(got["v"], ref["w"])
    np.testing.assert_allclose(got["u"], ref["u"], rtol=RTOL, atol=ATOL)
    assert np.array_equal(got["u"] == 0, ref["u"] == 0)
    np.testing.assert_allclose(got["X"], ref["X"], rtol=RTOL, atol=ATOL)
    assert got["res"]["tau"] == pytest.approx(ref["tau"], rel=1e-9)


@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 4, 5), (5, 1, 7), (17, 16, 16), (6, 50, 41), (300, 3, 2), (4, 64, 1024)])
def test_trilevel_matches_oracle(mp, shape):
    rng = np.random.default_rng(sum(shape))
    Y = rng.standard_normal(shape).astype(np.float32)
    w = np.abs(Y).reshape(shape[0], -1).max(axis=1).astype(np.float64)
    for frac in (0.05, 0.5, 1.5, 0.0):
        eta = float(np.float32(frac * w.sum()))
        check_tri(run_tri(mp, Y, eta), orc.trilevel_l1infinf(Y, eta))


# Tensors that the register files hold (16-byte aligned slabs, at most 256 of them) take the one-pass kernel: one piece of a
# slab per workgroup, up to 256 of them.  The shapes cover one piece per slab and several, a ragged
# last piece, pieces shorter than a workgroup's 512 chunks, 256 slabs, one slab, and a slab length
# that is not a multiple of 16 bytes (which takes the three-kernel chain).
HELD_SHAPES = [(256, 32, 40), (256, 256, 64), (7, 300, 1000), (1, 1000, 1000), (3, 1, 4000004), (100, 50, 1004),
               (33, 77, 129), (16, 1024, 1024), (64, 1000, 33)]


@pytest.mark.parametrize("shape", HELD_SHAPES)
def test_trilevel_one_pass_matches_oracle(mp, shape):
    rng = np.random.default_rng(list(shape))
    Y = rng.standard_normal(shape).astype(np.float32)
    Y *= np.power(10.0, rng.uniform(-1.0, 0.0, shape[0])).astype(np.float32)[:, None, None]
    w = np.abs(Y).reshape(shape[0], -1).max(axis=1).astype(np.float64)
    for frac in (0.05, 0.5, 1.5, 0.0):
        eta = float(np.float32(frac * w.sum()))
        check_tri(run_tri(mp, Y, eta), orc.trilevel_l1infinf(Y, eta))


@pytest.mark.parametrize("limit", [0, 1])
@pytest.mark.parametrize("shape", [(256, 32, 40), (7, 300, 1000), (16, 512, 1024)])
def test_trilevel_one_pass_when_workgroups_do_not_wait_for_one_another(mp, shape, limit):
    """With no patience (poll limit 0 or 1) every workgroup computes the maxima it does not find
    posted itself, as it would on a GPU too busy to run all of them at once: same result, out of
    place and in place, and every kernel ends."""
    rng = np.random.default_rng(list(shape) + [limit])
    dev = torch.device("cuda:0")
    Y = rng.standard_normal(shape).astype(np.float32)
    w = np.abs(Y).reshape(shape[0], -1).max(axis=1).astype(np.float64)
    eta = float(np.float32(0.3 * w.sum()))
    ref = orc.trilevel_l1infinf(Y, eta)
    before = mp.set_search_spin_limit(limit)
    try:
        check_tri(run_tri(mp, Y, eta), ref)
        Z = torch.from_numpy(Y).to(dev)
        ws = mp.Workspace.for_call("tri", *shape, device=dev)
        mp.trilevel_proj_l1infinf(Z, eta, X=Z, workspace=ws)
        torch.cuda.synchronize()
        np.testing.assert_allclose(Z.cpu().numpy(), ref["X"], rtol=RTOL, atol=ATOL)
        assert ws.result()["tau"] == pytest.approx(ref["tau"], rel=1e-9)
    finally:
        assert mp.set_search_spin_limit(before) == limit


def test_trilevel_one_pass_in_place_unaligned_output_and_repeats(mp):
    """X = Y, an X that starts 4 bytes into its allocation (element-wise stores), and 30 calls in a
    row on one workspace (the posted words are cleared by every call): always the same bits."""
    rng = np.random.default_rng(77)
    dev = torch.device("cuda:0")
    shape = (40, 100, 200)
    Y = rng.standard_normal(shape).astype(np.float32)
    w = np.abs(Y).reshape(shape[0], -1).max(axis=1).astype(np.float64)
    eta = float(np.float32(0.4 * w.sum()))
    ref = orc.trilevel_l1infinf(Y, eta)
    Yd = torch.from_numpy(Y).to(dev)
    ws = mp.Workspace.for_call("tri", *shape, device=dev)
    first = None
    for rep in range(30):
        X = mp.trilevel_proj_l1infinf(Yd, eta, workspace=ws)
        torch.cuda.synchronize()
        if first is None:
            first = X.clone()
            np.testing.assert_allclose(X.cpu().numpy(), ref["X"], rtol=RTOL, atol=ATOL)
        else:
            assert torch.equal(X, first)
    buf = torch.zeros(Y.size + 4, dtype=torch.float32, device=dev)
    Xo = buf[1:1 + Y.size].view(shape)
    mp.trilevel_proj_l1infinf(Yd, eta, X=Xo, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(Xo, first) and float(buf[0]) == 0.0 and float(buf[-1]) == 0.0
    Z = Yd.clone()
    mp.trilevel_proj_l1infinf(Z, eta, X=Z, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(Z, first)


# ------------------------------------------------------------------ the five full-size workloads
def test_workload_small_256x128(mp):
    w, Y = workloads.make("small_256x128")
    eta = eta_for(Y, "inf", w.eta_frac)
    check_against_oracle(run_gpu(mp, Y, eta, "inf"), orc.bilevel_l1inf(Y, eta), "inf")


def test_workload_square_4096(mp):
    w, Y = workloads.make("square_4096")
    eta = eta_for(Y, "inf", w.eta_frac)
    check_against_oracle(run_gpu(mp, Y, eta, "inf"), orc.bilevel_l1inf(Y, eta), "inf")


@pytest.mark.parametrize("name", ["tall_262144x256", "wide_256x262144"])
def test_workload_skewed(mp, name):
    w, Y = workloads.make(name)
    eta = eta_for(Y, "inf", w.eta_frac)
    got = run_gpu(mp, Y, eta, "inf")
    check_against_oracle(got, orc.bilevel_l1inf(Y, eta), "inf")      # every element of X
    # and what holds by construction: entries are copied or clipped to u_j
    X, u = got["X"], got["u"]
    assert np.array_equal(np.abs(X).max(axis=0), u)
    assert np.all((X == Y) | (np.abs(X) == u[None, :]))


def test_workload_tensor_256(mp):
    w, Y = workloads.make("tensor_256x256x256")
    nrm = float(np.abs(Y).reshape(256, -1).max(axis=1).astype(np.float64).sum())
    eta = float(np.float32(w.eta_frac * nrm))
    check_tri(run_tri(mp, Y, eta), orc.trilevel_l1infinf(Y, eta))


@pytest.fixture(scope="module")
def big_square():
    return workloads.make("square_16384")


@pytest.mark.parametrize("q", ["inf", 2, 1])
def test_workload_square_16384(mp, big_square, q):
    """1 GiB input: v, u and every element of X against the oracle (which takes the 16384 columns
    one by one), plus whole-matrix properties."""
    w, Y = big_square
    eta = eta_for(Y, q, w.eta_frac)
    got = run_gpu(mp, Y, eta, q)
    rng = np.random.default_rng(16384)
    ref = orc.bilevel(Y, eta, q)
    check_against_oracle(got, ref, q)
    del ref
    X = got["X"]
    if q == "inf":
        assert np.array_equal(np.abs(X).max(axis=0), got["u"])
    rows = np.sort(rng.choice(Y.shape[0], size=64, replace=False))
    assert np.all(np.abs(X[rows]) <= np.abs(Y[rows])) and np.all(X[rows] * Y[rows] >= 0)
    dev = torch.device("cuda:0")
    Xd = torch.from_numpy(X).to(dev)
    assert mp.norm_l1q(Xd, QNAME[q]) == pytest.approx(eta, rel=1e-5)


@pytest.fixture(scope="module")
def beyond_int32():
    """132000 x 16384 fp32: 2 162 688 000 elements, more than 2^31 (8.6 GB; the tail rows sit past
    element 2^31).  Uniform entries, generated in row chunks from one seeded stream."""
    n, m = 132000, 16384
    rng = np.random.default_rng(2405_02086)
    Y = np.empty((n, m), dtype=np.float32)
    for r0 in range(0, n, 8250):
        Y[r0:r0 + 8250] = rng.random((8250, m), dtype=np.float32) - np.float32(0.5)
    return Y


@pytest.mark.parametrize("q", ["inf", 1])
def test_more_than_2_to_the_31_elements(mp, beyond_int32, q):
    """Every index is 64-bit: the aggregate is compared in full, X on sampled columns over all
    rows (the oracle computes those one by one), and the tail rows on their own."""
    Y = beyond_int32
    n, m = Y.shape
    assert n * m > 2 ** 31
    v = orc.column_norms(Y, q).astype(np.float64)
    eta = float(np.float32(0.25 * v.sum()))
    got = run_gpu(mp, Y, eta, q)
    rng = np.random.default_rng(31)
    cols = np.sort(rng.choice(m, size=24, replace=False))
    ref = orc.bilevel(Y, eta, q, columns=cols)
    check_against_oracle(got, ref, q, columns=cols)
    X = got["X"]
    tail = slice(n - 700, n)        # rows whose elements all sit past 2^31
    assert (n - 700) * m > 2 ** 31
    assert np.all(np.abs(X[tail]) <= np.abs(Y[tail])) and np.all(X[tail] * Y[tail] >= 0)
    if q == "inf":
        u = got["u"]
        assert np.array_equal(X[tail], np.sign(Y[tail]) * np.minimum(np.abs(Y[tail]), u[None, :]))
        assert np.array_equal(np.abs(X).max(axis=0), u)


def test_trilevel_more_than_2_to_the_31_elements(mp, beyond_int32):
    """The same buffer seen as a 132 x 16384 x 1000 tensor: slabs of 16 384 000 elements, the last
    ones past element 2^31; compared with the oracle in full."""
    Y = beyond_int32.reshape(132, 16384, 1000)
    w = np.abs(Y.reshape(132, -1)).max(axis=1).astype(np.float64)
    eta = float(np.float32(0.3 * w.sum()))
    check_tri(run_tri(mp, Y, eta), orc.trilevel_l1infinf(Y, eta))


# ------------------------------------------------------------------ API corners
@pytest.mark.parametrize("q", ["inf", 1, 2])
def test_unaligned_pointers(mp, q):
    """Y or X starting 4 bytes into an allocation, on the kernels that read and write 16 bytes at any address; nothing
    outside X is written."""
    rng = np.random.default_rng(21)
    dev = torch.device("cuda:0")
    n, m = 130, 264
    Y = rng.standard_normal((n, m)).astype(np.float32)
    eta = eta_for(Y, q, 0.3)
    ref = orc.bilevel(Y, eta, q)
    fn = getattr(mp, "bilevel_proj_" + QNAME[q])
    ws = mp.Workspace.for_call(QNAME[q], n, m, device=dev)
    for y_off, x_off in ((1, 0), (0, 1), (1, 1), (0, 0)):
        ybuf = torch.zeros(n * m + 4, dtype=torch.float32, device=dev)
        xbuf = torch.full((n * m + 4,), 7.0, dtype=torch.float32, device=dev)
        Yd = ybuf[y_off:y_off + n * m].view(n, m)
        Xd = xbuf[x_off:x_off + n * m].view(n, m)
        Yd.copy_(torch.from_numpy(Y))
        assert (Yd.data_ptr() % 16 != 0) == bool(y_off) and (Xd.data_ptr() % 16 != 0) == bool(x_off)
        fn(Yd, eta, X=Xd, workspace=ws)
        torch.cuda.synchronize()
        np.testing.assert_allclose(Xd.cpu().numpy(), ref["X"], rtol=RTOL, atol=ATOL)
        rest = torch.cat([xbuf[:x_off], xbuf[x_off + n * m:]]).cpu().numpy()
        assert np.all(rest == 7.0), "wrote outside X"


@pytest.mark.parametrize("q", ["inf", 1, 2])
def test_split_call_equals_whole_call_and_other_stream(mp, q):
    rng = np.random.default_rng(22)
    dev = torch.device("cuda:0")
    Y = rng.standard_normal((700, 520)).astype(np.float32)
    eta = eta_for(Y, q, 0.25)
    Yd = torch.from_numpy(Y).to(dev)
    ws = mp.Workspace.for_call(QNAME[q], *Y.shape, device=dev)
    whole = getattr(mp, "bilevel_proj_" + QNAME[q])(Yd, eta, workspace=ws)      # no v_out / u_out
    torch.cuda.synchronize()
    tau_whole = ws.result()["tau"]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        v = torch.empty(Y.shape[1], dtype=torch.float32, device=dev)
        u = torch.empty(Y.shape[1], dtype=torch.float32, device=dev)
        mp.bilevel_radii(QNAME[q], Yd, eta, ws, v_out=v, stream=stream)
        X2 = torch.empty_like(Yd)
        mp.bilevel_apply(QNAME[q], Yd, X2, ws, u_out=u, stream=stream)
    stream.synchronize()
    assert ws.result()["tau"] == tau_whole
    assert torch.equal(whole, X2)
    ref = orc.bilevel(Y, eta, q)
    np.testing.assert_allclose(u.cpu().numpy(), np.asarray(ref["u"], dtype=np.float32), rtol=RTOL, atol=ATOL)


def test_kernel_trace_records_one_event_per_kernel(mp):
    dev = torch.device("cuda:0")
    Yd = torch.randn(512, 512, device=dev)
    ws = mp.Workspace.for_call("l1inf", 512, 512, device=dev)
    tr = mp.KernelTrace(16)
    with tr:
        mp.bilevel_proj_l1inf(Yd, 10.0, workspace=ws)
    d = tr.durations_ms()
    tr.close()
    assert tr.count == 4 and len(d) == 3 and all(x > 0 for x in d)     # aggregate, reduce, map(+search)
    mp.bilevel_proj_l1inf(Yd, 10.0, workspace=ws)                          # tracing is off again
    assert mp.lib().mlproj_trace_end() == 0


@pytest.mark.parametrize("q", ["inf", 1, 2])
def test_extreme_magnitudes_and_radii(mp, q):
    rng = np.random.default_rng(23)
    base = rng.standard_normal((96, 80)).astype(np.float32)
    for scale in (np.float32(1e-18), np.float32(1e15)):
        Y = base * scale
        eta = eta_for(Y, q, 0.2)
        got, ref = run_gpu(mp, Y, eta, q), orc.bilevel(Y, eta, q)
        np.testing.assert_allclose(got["X"], ref["X"], rtol=RTOL, atol=ATOL * float(scale))
        assert np.array_equal(got["u"] == 0, np.asarray(ref["u"]) == 0)
    # a radius far below the resolution of the norms: everything (or all but one column) goes
    got = run_gpu(mp, base, 1e-30, q)
    assert np.abs(got["X"]).sum() <= 1e-6
    # a radius that keeps exactly one column for q = inf
    Y = base.copy()
    Y[:, 5] *= 50
    eta = 0.5 * float(np.abs(Y[:, 5]).max())
    check_against_oracle(run_gpu(mp, Y, eta, "inf"), orc.bilevel_l1inf(Y, eta), "inf")


def test_paper_timing_shape_uniform_entries(mp):
    """The shape and distribution of the paper's own timing runs (Sec. 6.1): 1000 x 10000, U(0,1), eta = 1."""
    w, Y = workloads.make("paper_1000x10000")
    for eta in (0.25, 1.0, 4.0):
        check_against_oracle(run_gpu(mp, Y, eta, "inf"), orc.bilevel_l1inf(Y, eta), "inf")


# ------------------------------------------------------------------ multi-level (generic)
def run_multi(mp, Y, norms, eta):
    dev = torch.device("cuda:0")
    Yd = torch.from_numpy(Y).to(dev)
    d0 = Y.shape[0]
    ws = mp.Workspace(mp.multilevel_workspace_bytes(Y.shape), device=dev)
    v = torch.full((d0,), -1.0, dtype=torch.float32, device=dev)
    u = torch.full((d0,), -1.0, dtype=torch.float32, device=dev)
    X = mp.multilevel_proj(Yd, norms, eta, workspace=ws, v_out=v, u_out=u)
    torch.cuda.synchronize()
    return {"X": X.cpu().numpy(), "v": v.cpu().numpy(), "u": u.cpu().numpy(), "res": ws.result()}


def nested_norm(Y, norms):
    a = Y.astype(np.float64)
    for q in norms:
        a = {"inf": lambda z: np.abs(z).max(axis=-1), 1: lambda z: np.abs(z).sum(axis=-1),
             2: lambda z: np.sqrt((z * z).sum(axis=-1))}[q](a)
    return float(a.sum())


def check_multi(got, ref):
    np.testing.assert_allclose(got["v"], ref["w"].astype(np.float32), rtol=2e-7)
    np.testing.assert_allclose(got["u"], ref["u"].astype(np.float32), rtol=RTOL, atol=ATOL)
    assert np.array_equal(got["u"] == 0, ref["u"] == 0)
    assert got["res"]["tau"] == pytest.approx(ref["tau"], rel=1e-9, abs=1e-300)
    np.testing.assert_allclose(got["X"], ref["X"], rtol=RTOL, atol=ATOL)


ML_CASES = [
    ((5, 7), [1]), ((5, 7), ["inf"]), ((300, 33), [2]), ((6, 1030), [1]),
    ((4, 3, 5), [1, 1]), ((4, 3, 5), ["inf", "inf"]), ((4, 3, 5), [2, 2]), ((9, 16, 3), ["inf", 1]),
    ((9, 16, 3), [1, 2]), ((7, 5, 64), [1, "inf"]), ((3, 40, 260), [1, 1]), ((3, 40, 260), [2, 1]),
    ((5, 4, 3, 6), [1, 1, 1]), ((5, 4, 3, 6), ["inf", 2, 1]), ((2, 3, 2, 2, 8), [1, "inf", 2, 1]),
    ((20000, 2, 4), [1, 1]), ((1, 1, 1), [1, 1]), ((3, 1, 2000), [1, 1]),
    # neighbouring l_inf levels (merged into one by the driver)
    ((5, 4, 3, 6), ["inf", "inf", 1]), ((5, 4, 3, 6), [1, "inf", "inf"]), ((4, 3, 5, 2), ["inf", "inf", 2]),
    ((3, 4, 2, 5, 6), ["inf", "inf", "inf", "inf"]), ((6, 2, 3, 4, 5), ["inf", "inf", 1, "inf"]),
]


@pytest.mark.parametrize("shape,norms", ML_CASES)
def test_multilevel_matches_oracle(mp, shape, norms):
    rng = np.random.default_rng(list(shape) + [len(norms)])
    Y = rng.standard_normal(shape).astype(np.float32)
    nrm = nested_norm(Y, norms)
    for frac in (0.05, 0.5, 1.5, 0.0):
        eta = float(np.float32(frac * nrm))
        check_multi(run_multi(mp, Y, norms, eta), orc.multilevel(Y, norms, eta))


@pytest.mark.parametrize("shape,norms", [((40, 30, 64), [1, 1]), ((12, 8, 3000), [1, 1]), ((64, 9, 5, 32), [1, "inf", 1]),
                                         ((30, 2000), [1]), ((50, 20, 256), [2, 1])])
def test_multilevel_sparse_radius_zeroes_most_groups(mp, shape, norms):
    """Groups of very different sizes and a small radius: most groups (and, one level down, many
    fibres of the kept ones) get radius 0, which the l1 fibre searches skip."""
    rng = np.random.default_rng(list(shape) + [77])
    Y = rng.standard_normal(shape).astype(np.float32)
    Y *= np.power(10.0, rng.uniform(-2.5, 0.0, shape[0])).astype(np.float32).reshape((-1,) + (1,) * (len(shape) - 1))
    if len(shape) > 2:
        Y *= (rng.random(shape[:2]) < 0.5).astype(np.float32).reshape(shape[:2] + (1,) * (len(shape) - 2))
    nrm = nested_norm(Y, norms)
    for frac in (0.002, 0.03):
        eta = float(np.float32(frac * nrm))
        ref = orc.multilevel(Y, norms, eta)
        assert 0 < (ref["u"] > 0).sum() < shape[0] * 0.7
        check_multi(run_multi(mp, Y, norms, eta), ref)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("shape,norms", [((5, 7), [1]), ((300, 33), ["inf"]), ((4, 3, 5), [1, 1]), ((40, 30, 64), ["inf", "inf"]),
                                         ((9, 16, 3), [1, 2]), ((7, 5, 260), [2, 1]), ((5, 4, 3, 6), ["inf", 2, 1]),
                                         ((5000, 2, 4), [1, 1]), ((40000, 8), ["inf"]), ((33000, 2, 4), ["inf", "inf"]),
                                         ((1, 1, 1), [1, 1])])
def test_multilevel_weighted_outer_norm_matches_oracle(mp, storage, shape, norms):
    """The multi-level projection with the weighted l1 ball on top (Sec. 3, Sec. 5.2)."""
    rng = np.random.default_rng(list(shape) + [len(norms), 5])
    Y = orc.round_to_storage(rng.standard_normal(shape).astype(np.float32), storage)
    w = np.exp(rng.uniform(-1.5, 1.5, shape[0])).astype(np.float32)
    dev = torch.device("cuda:0")
    top = orc.multilevel(Y, norms, 3.0e38)["w"]
    total = float(np.dot(w.astype(np.float64), top))
    for frac in (0.03, 0.5, 1.2, 0.0):
        eta = float(np.float32(frac * total))
        ref = orc.multilevel_stored(Y, norms, eta, storage, p=("w1", w))
        Yd = torch.from_numpy(Y).to(dev).to(getattr(torch, STORE_DTYPES[storage]))
        ws = mp.Workspace(mp.multilevel_workspace_bytes(shape), device=dev)
        v = torch.full((shape[0],), -1.0, dtype=torch.float32, device=dev)
        u = torch.full((shape[0],), -1.0, dtype=torch.float32, device=dev)
        X = mp.multilevel_proj_weighted(Yd, norms, eta, torch.from_numpy(w).to(dev), workspace=ws, v_out=v, u_out=u)
        torch.cuda.synchronize()
        got = {"X": X.float().cpu().numpy(), "v": v.cpu().numpy(), "u": u.cpu().numpy(), "res": ws.result()}
        np.testing.assert_allclose(got["v"], ref["w"].astype(np.float32), rtol=2e-7)
        np.testing.assert_allclose(got["u"], ref["u"].astype(np.float32), rtol=RTOL, atol=ATOL)
        assert np.array_equal(got["u"] == 0, ref["u"] == 0)
        if frac > 0:
            assert got["res"]["tau"] == pytest.approx(ref["tau"], rel=1e-9, abs=1e-300)
        x = ref["X32"].astype(np.float64)
        tol = RTOL * np.abs(x) + ATOL
        lo = orc.round_to_storage((x - tol).astype(np.float32), storage)
        hi = orc.round_to_storage((x + tol).astype(np.float32), storage)
        assert np.all((got["X"] >= lo) & (got["X"] <= hi))


def test_multilevel_inf_inf_equals_the_trilevel_entry_point(mp):
    rng = np.random.default_rng(31)
    Y = rng.standard_normal((40, 24, 36)).astype(np.float32)
    eta = float(np.float32(0.3 * nested_norm(Y, ["inf", "inf"])))
    a = run_multi(mp, Y, ["inf", "inf"], eta)
    b = run_tri(mp, Y, eta)
    assert np.array_equal(a["X"], b["X"]) and np.array_equal(a["u"], b["u"])


@pytest.mark.parametrize("norms", [[1, 1], ["inf", "inf"], [2, 1]])
def test_workload_tensor_256_multilevel(mp, norms):
    w, Y = workloads.make("tensor_256x256x256")
    eta = float(np.float32(w.eta_frac * nested_norm(Y, norms)))
    check_multi(run_multi(mp, Y, norms, eta), orc.multilevel(Y, norms, eta))


# ------------------------------------------------------------------ repeatability, concurrency
def test_results_repeat_bit_for_bit(mp):
    """Fixed reduction orders everywhere: every repetition gives the same bits, including the
    grid-wide search (m > 32768) whose workgroups exchange their sums every round."""
    rng = np.random.default_rng(41)
    dev = torch.device("cuda:0")
    for q, shape in (("inf", (64, 50000)), (1, (512, 1536)), (2, (1500, 700)), ("inf", (1500, 700))):
        Y = rng.standard_normal(shape).astype(np.float32)
        eta = eta_for(Y, q, 0.15)
        Yd = torch.from_numpy(Y).to(dev)
        ws = mp.Workspace.for_call(QNAME[q], *shape, device=dev)
        fn = getattr(mp, "bilevel_proj_" + QNAME[q])
        first, tau0 = None, None
        for rep in range(40):
            X = fn(Yd, eta, workspace=ws)
            torch.cuda.synchronize()
            tau = ws.result()["tau"]
            if first is None:
                first, tau0 = X.clone(), tau
            else:
                assert tau == tau0 and torch.equal(X, first), (q, shape, rep)


def test_two_streams_two_workspaces(mp):
    rng = np.random.default_rng(42)
    dev = torch.device("cuda:0")
    jobs = []
    # (the last two run the several-workgroup search side by side, each on its own slots)
    for q, shape in (("inf", (2048, 1024)), (2, (1024, 2048)), (1, (600, 900)), ("inf", (16, 70000)), (2, (8, 150000))):
        Y = rng.standard_normal(shape).astype(np.float32)
        eta = eta_for(Y, q, 0.3)
        jobs.append((q, Y, eta, torch.from_numpy(Y).to(dev), mp.Workspace.for_call(QNAME[q], *shape, device=dev),
                     torch.cuda.Stream()))
    torch.cuda.synchronize()
    outs = []
    for rep in range(5):
        outs = []
        for q, Y, eta, Yd, ws, st in jobs:
            with torch.cuda.stream(st):
                outs.append(getattr(mp, "bilevel_proj_" + QNAME[q])(Yd, eta, workspace=ws, stream=st))
    torch.cuda.synchronize()
    for (q, Y, eta, Yd, ws, st), X in zip(jobs, outs):
        np.testing.assert_allclose(X.cpu().numpy(), orc.bilevel(Y, eta, q)["X"], rtol=RTOL, atol=ATOL)


# ------------------------------------------------------------------ other outer norms (BP^{p,q}, general p)
def lp(x, p):
    x = np.asarray(x, dtype=np.float64)
    return float({1: np.abs(x).sum(), 2: np.sqrt((x * x).sum()), "inf": np.abs(x).max()}[p])


@pytest.mark.parametrize("p", [2, "inf"])
@pytest.mark.parametrize("q", ["inf", 1, 2])
@pytest.mark.parametrize("shape", [(1, 1), (9, 7), (300, 257), (2065, 260), (40, 5000), (8, 40000)])
def test_bilevel_pq_matches_oracle(mp, p, q, shape):
    rng = np.random.default_rng([shape[0], shape[1], 7])
    dev = torch.device("cuda:0")
    Y = rng.standard_normal(shape).astype(np.float32)
    Y *= np.power(10.0, rng.uniform(-1.0, 0.0, shape[1])).astype(np.float32)[None, :]
    vnorm = lp(orc.column_norms(Y, q), p)
    Yd = torch.from_numpy(Y).to(dev)
    n, m = shape
    for frac in (0.05, 0.5, 1.3, 0.0):
        eta = float(np.float32(frac * vnorm))
        ref = orc.bilevel(Y, eta, q, p=p)
        ws = mp.Workspace.for_call(QNAME[q], n, m, device=dev)
        u = torch.empty(m, dtype=torch.float32, device=dev)
        X = mp.bilevel_proj_pq(p, q, Yd, eta, workspace=ws, u_out=u)
        torch.cuda.synchronize()
        np.testing.assert_allclose(u.cpu().numpy(), np.asarray(ref["u"], dtype=np.float32), rtol=RTOL, atol=ATOL)
        np.testing.assert_allclose(X.cpu().numpy(), ref["X"], rtol=RTOL, atol=ATOL)
        res = ws.result()
        assert res["norm"] == pytest.approx(vnorm, rel=1e-12)
        assert res["inside_ball"] == (vnorm <= eta)
        if q == 1:
            assert res["inner_pending"] == 0
        if frac > 1:
            assert np.array_equal(X.cpu().numpy(), Y)


@pytest.mark.parametrize("p", [2, "inf"])
def test_multilevel_outer_norm_matches_oracle(mp, p):
    rng = np.random.default_rng(77)
    dev = torch.device("cuda:0")
    for shape, norms in (((30, 12, 20), [1, "inf"]), ((300, 40), [2]), ((6, 5, 4, 8), ["inf", 1, 2])):
        Y = rng.standard_normal(shape).astype(np.float32)
        a = Y.astype(np.float64)
        for qq in norms:
            a = {"inf": lambda z: np.abs(z).max(axis=-1), 1: lambda z: np.abs(z).sum(axis=-1),
                 2: lambda z: np.sqrt((z * z).sum(axis=-1))}[qq](a)
        eta = float(np.float32(0.4 * lp(a, p)))
        ref = orc.multilevel(Y, norms, eta, p=p)
        X = mp.multilevel_proj(torch.from_numpy(Y).to(dev), norms, eta, p=p)
        torch.cuda.synchronize()
        np.testing.assert_allclose(X.cpu().numpy(), ref["X"], rtol=RTOL, atol=ATOL)


def test_calls_can_be_captured_in_a_hip_graph_and_replayed(mp):
    """The library only enqueues kernels (no allocation, no memset, no synchronisation), so a
    call can be recorded once and replayed; every replay must equal the eager result."""
    rng = np.random.default_rng(51)
    dev = torch.device("cuda:0")
    for q, shape in (("inf", (1024, 768)), (2, (640, 512)), (1, (300, 260))):
        Y = rng.standard_normal(shape).astype(np.float32)
        eta = eta_for(Y, q, 0.25)
        fn = getattr(mp, "bilevel_proj_" + QNAME[q])
        Yd = torch.from_numpy(Y).to(dev)
        Xg = torch.zeros_like(Yd)
        ws = mp.Workspace.for_call(QNAME[q], *shape, device=dev)
        eager = fn(Yd, eta, workspace=ws).clone()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            fn(Yd, eta, X=Xg, workspace=ws)
        for rep in range(4):
            Xg.zero_()
            if rep == 2:                       # new data in the same buffers
                Yd.mul_(0.5)
                eager = fn(Yd, eta, workspace=ws).clone()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(Xg, eager), (q, rep)


def test_graph_replay_of_the_other_launch_chains(mp):
    """The same for the chains with kernels of their own: the several-workgroup search (its
    slots are cleared by a kernel of the same call, so every replay starts clean), the weighted
    outer norm, the one-kernel form of a small matrix, a batch in place, and a multi-level call."""
    rng = np.random.default_rng(52)
    dev = torch.device("cuda:0")

    def check(make_call, out, refresh, reps=4):
        eager = make_call(None).clone()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            make_call(out)
        for rep in range(reps):
            out.zero_()
            if rep == 2:
                refresh()
                eager = make_call(None).clone()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, eager), rep

    # more than 32768 columns: the several-workgroup search
    Y = torch.from_numpy(rng.laplace(size=(4, 70000)).astype(np.float32)).to(dev)
    ws = mp.Workspace.for_call("l1inf", 4, 70000, device=dev)
    eta = eta_for(Y.cpu().numpy(), "inf", 0.1)
    check(lambda X: mp.bilevel_proj_l1inf(Y, eta, X=X, workspace=ws), torch.zeros_like(Y), lambda: Y.mul_(0.5))
    # weighted outer norm, with more than 32768 columns and with few
    for shape in ((4, 70000), (300, 520)):
        Y = torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).to(dev)
        w = torch.from_numpy(weights_for(shape[1], 4)).to(dev)
        ws = mp.Workspace.for_call("l1inf", *shape, device=dev)
        eta = weighted_eta(Y.cpu().numpy(), "inf", w.cpu().numpy(), 0.2)
        check(lambda X: mp.bilevel_proj_weighted(Y, eta, "inf", w, X=X, workspace=ws), torch.zeros_like(Y), lambda: Y.mul_(0.5))
    # the one-kernel form of a small matrix
    Y = torch.from_numpy(rng.standard_normal((256, 128)).astype(np.float32)).to(dev)
    ws = mp.Workspace.for_call("l12", 256, 128, device=dev)
    eta = eta_for(Y.cpu().numpy(), 2, 0.3)
    check(lambda X: mp.bilevel_proj_l12(Y, eta, X=X, workspace=ws), torch.zeros_like(Y), lambda: Y.mul_(0.5))
    # a multi-level call
    T = torch.from_numpy(rng.standard_normal((20, 30, 64)).astype(np.float32)).to(dev)
    ws = mp.Workspace(mp.multilevel_workspace_bytes(T.shape), device=dev)
    eta = float(np.float32(0.2 * nested_norm(T.cpu().numpy(), [1, 1])))
    check(lambda X: mp.multilevel_proj(T, [1, 1], eta, X=X, workspace=ws), torch.zeros_like(T), lambda: T.mul_(0.5))


def test_graph_replay_of_the_one_pass_and_grid_chains(mp):
    """The one-pass tri-level kernel (its posted words are cleared by the small kernel recorded in
    front of it, so every replay starts clean), the l1,1 chain whose aggregate pass carries the
    grid, and the entry point that allocates nothing: recorded once, replayed four times with the
    program's own eager calls in between, new data from the third replay on."""
    rng = np.random.default_rng(53)
    dev = torch.device("cuda:0")

    def check(make_call, out, refresh, reps=4):
        eager = make_call(None).clone()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            make_call(out)
        for rep in range(reps):
            out.zero_()
            if rep == 2:
                refresh()
            eager = make_call(None).clone()       # (an eager call between the replays, on the same workspace)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, eager), rep

    T = torch.from_numpy(rng.standard_normal((96, 64, 128)).astype(np.float32)).to(dev)        # 3 MiB: one pass
    ws = mp.Workspace.for_call("tri", *T.shape, device=dev)
    w = T.abs().reshape(96, -1).max(dim=1).values.double().sum().item()
    eta = float(np.float32(0.3 * w))
    check(lambda X: mp.trilevel_proj_l1infinf(T, eta, X=X, workspace=ws), torch.zeros_like(T), lambda: T.mul_(0.5))
    Y = torch.from_numpy(rng.standard_normal((8200, 4096)).astype(np.float32)).to(dev)        # 128 MiB: the grid
    ws1 = mp.Workspace.for_call("l11", *Y.shape, device=dev)
    eta1 = float(np.float32(0.2 * Y.abs().double().sum().item()))
    check(lambda X: mp.bilevel_proj_l11(Y, eta1, X=X, workspace=ws1), torch.zeros_like(Y), lambda: Y.mul_(0.5))
    # l1,1 with the columns in registers: the kernel that searches itself, the one behind a search
    # kernel (whose first heavy columns leave whole stripes dropped), and the narrow stripes
    for shape in ((1000, 512), (300, 5000), (5000, 64)):
        A = rng.standard_normal(shape).astype(np.float32)
        A[:, :3] *= 40.0
        Yh = torch.from_numpy(A).to(dev)
        wsh = mp.Workspace.for_call("l11", *shape, device=dev)
        etah = float(np.float32(0.05 * Yh.abs().double().sum().item()))
        check(lambda X: mp.bilevel_proj_l11(Yh, etah, X=X, workspace=wsh), torch.zeros_like(Yh), lambda: Yh.mul_(0.5))
        assert wsh.result()["inner_sweeps"] == 0 and wsh.result()["inner_finished"] == wsh.result()["n_active"]
    Z = torch.from_numpy(rng.standard_normal((700, 900)).astype(np.float32)).to(dev)
    eta2 = float(np.float32(0.2 * Z.abs().max(dim=0).values.double().sum().item()))
    scratch_out = torch.zeros_like(Z)
    check(lambda X: mp.bilevel_proj_l1inf_no_alloc(Z, eta2, scratch_out if X is None else X), torch.zeros_like(Z),
          lambda: Z.mul_(0.5))


def test_trilevel_one_pass_on_a_busy_gpu(mp):
    """The one-pass kernel with its default patience while another stream keeps the GPU full of
    the library's own long kernels: whether all of its workgroups run at once or some start late
    and the others compute their maxima for them, the result is the oracle's and every kernel ends."""
    rng = np.random.default_rng(54)
    dev = torch.device("cuda:0")
    big = torch.from_numpy(rng.standard_normal((8192, 8192)).astype(np.float32)).to(dev)
    big_out = torch.empty_like(big)
    big_ws = mp.Workspace.for_call("l11", 8192, 8192, device=dev)
    shape = (256, 64, 256)
    Y = rng.standard_normal(shape).astype(np.float32)
    w = np.abs(Y).reshape(shape[0], -1).max(axis=1).astype(np.float64)
    eta = float(np.float32(0.25 * w.sum()))
    ref = orc.trilevel_l1infinf(Y, eta)
    Yd = torch.from_numpy(Y).to(dev)
    ws = mp.Workspace.for_call("tri", *shape, device=dev)
    busy, mine = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for rep in range(3):
        for _ in range(6):
            mp.bilevel_proj_l11(big, 1000.0, X=big_out, workspace=big_ws, stream=busy)
        X = torch.empty_like(Yd)
        mp.trilevel_proj_l1infinf(Yd, eta, X=X, workspace=ws, stream=mine)
        torch.cuda.synchronize()
        np.testing.assert_allclose(X.cpu().numpy(), ref["X"], rtol=RTOL, atol=ATOL)
        assert ws.result()["tau"] == pytest.approx(ref["tau"], rel=1e-9)


# ------------------------------------------------------------------ 16-bit storage
STORE_DTYPES = {"bf16": "bfloat16", "f16": "float16", "f32": "float32"}


def stored_input(shape, storage, seed, scale=1.0):
    rng = np.random.default_rng([shape[0], shape[1], seed])
    Y = (rng.standard_normal(shape) * scale).astype(np.float32)
    Y *= np.power(10.0, rng.uniform(-1.0, 0.0, shape[1])).astype(np.float32)[None, :]
    return orc.round_to_storage(Y, storage)


def run_stored(mp, Y, eta, q, storage, p=1, inplace=False, offset=0, x_offset=0):
    """Y: fp32 array of storage-representable values; offset / x_offset shift the device
    pointers by that many elements to reach the element-wise paths."""
    dev = torch.device("cuda:0")
    dt = getattr(torch, STORE_DTYPES[storage])
    n, m = Y.shape
    ybuf = torch.zeros(n * m + 16, dtype=dt, device=dev)
    Yd = ybuf[offset:offset + n * m].view(n, m)
    Yd.copy_(torch.from_numpy(Y).to(dev))
    assert np.array_equal(Yd.float().cpu().numpy(), Y)
    xbuf = torch.zeros(n * m + 16, dtype=dt, device=dev)
    Xd = Yd if inplace else xbuf[x_offset:x_offset + n * m].view(n, m)
    v = torch.full((m,), -1.0, dtype=torch.float32, device=dev)
    u = torch.full((m,), -1.0, dtype=torch.float32, device=dev)
    mask = torch.full((m,), 7, dtype=torch.uint8, device=dev)
    ws = mp.Workspace.for_call(QNAME[q], n, m, device=dev)
    X = mp.bilevel_proj_stored(Yd, eta, q, p=p, X=Xd, workspace=ws, v_out=v, u_out=u, mask_out=mask)
    torch.cuda.synchronize()
    if not inplace:   # nothing outside X's n*m elements was written
        assert not xbuf[:x_offset].any() and not xbuf[x_offset + n * m:].any()
    return {"X": X.float().cpu().numpy(), "v": v.cpu().numpy(), "u": u.cpu().numpy(),
            "mask": mask.cpu().numpy(), "res": ws.result()}


def check_stored(got, ref, q, storage):
    """The fp32 bar (rtol 1e-5, atol 1e-6) applies before rounding; rounding is monotone, so the
    stored value must lie between the roundings of the two ends of that interval."""
    check_against_oracle({**got, "X": ref["X32"]}, {**ref, "X": ref["X32"]}, q)      # v, u, tau, support
    assert np.array_equal(got["mask"], ref["mask"].astype(np.uint8))
    x = ref["X32"].astype(np.float64)
    tol = RTOL * np.abs(x) + ATOL
    lo = orc.round_to_storage((x - tol).astype(np.float32), storage)
    hi = orc.round_to_storage((x + tol).astype(np.float32), storage)
    assert np.all((got["X"] >= lo) & (got["X"] <= hi))
    if storage != "f32":   # 16-bit units are 2^8 .. 2^16 coarser than the fp32 differences
        assert np.mean(got["X"] != ref["X"]) < 0.02, "more than a few entries sit on a rounding boundary"
    assert not got["X"][:, ~ref["mask"]].any()


@pytest.mark.parametrize("storage", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("q", ["inf", 1, 2])
@pytest.mark.parametrize("shape", [(1, 1), (9, 7), (300, 257), (2065, 264), (131, 1032), (40, 5000),
                                   (8, 40000), (1000, 1024), (70, 4104)])
def test_stored_matches_oracle(mp, storage, q, shape):
    Y = stored_input(shape, storage, 31)
    for frac in (0.05, 0.6):
        eta = eta_for(Y, q, frac)
        check_stored(run_stored(mp, Y, eta, q, storage), orc.bilevel_stored(Y, eta, q, storage), q, storage)


@pytest.mark.parametrize("storage", ["bf16", "f16"])
@pytest.mark.parametrize("q", ["inf", 1, 2])
def test_stored_inplace_unaligned_outer_norms_and_degenerate(mp, storage, q):
    Y = stored_input((333, 520), storage, 32)
    eta = eta_for(Y, q, 0.3)
    ref = orc.bilevel_stored(Y, eta, q, storage)
    check_stored(run_stored(mp, Y, eta, q, storage, inplace=True), ref, q, storage)
    check_stored(run_stored(mp, Y, eta, q, storage, offset=1), ref, q, storage)        # Y 2-byte aligned
    check_stored(run_stored(mp, Y, eta, q, storage, x_offset=3), ref, q, storage)      # only X misaligned
    for p in (2, "inf"):
        v = orc.column_norms(Y, q).astype(np.float64)
        r = float(np.float32(0.4 * (np.sqrt((v * v).sum()) if p == 2 else v.max())))
        check_stored(run_stored(mp, Y, r, q, storage, p=p), orc.bilevel_stored(Y, r, q, storage, p=p), q, storage)
    big = float(np.float32(2 * orc.norm_l1q(Y, q)))                                       # inside the ball
    got = run_stored(mp, Y, big, q, storage)
    assert np.array_equal(got["X"], Y) and got["mask"].all() and got["res"]["inside_ball"]
    got = run_stored(mp, Y, 0.0, q, storage)
    assert not got["X"].any() and not got["mask"].any()


# ------------------------------------------------------------------ weighted l1 ball as outer norm
def run_weighted(mp, Y, eta, q, storage, w, inplace=False, offset=0):
    dev = torch.device("cuda:0")
    dt = getattr(torch, STORE_DTYPES[storage])
    n, m = Y.shape
    ybuf = torch.zeros(n * m + 16, dtype=dt, device=dev)
    Yd = ybuf[offset:offset + n * m].view(n, m)
    Yd.copy_(torch.from_numpy(Y).to(dev))
    v = torch.full((m,), -1.0, dtype=torch.float32, device=dev)
    u = torch.full((m,), -1.0, dtype=torch.float32, device=dev)
    mask = torch.full((m,), 7, dtype=torch.uint8, device=dev)
    ws = mp.Workspace.for_call(QNAME[q], n, m, device=dev)
    wd = torch.from_numpy(w).to(dev)
    X = mp.bilevel_proj_weighted(Yd, eta, q, wd, X=Yd if inplace else None, workspace=ws, v_out=v, u_out=u,
                                 mask_out=mask)
    torch.cuda.synchronize()
    assert np.array_equal(wd.cpu().numpy(), w), "the weights are read only"
    return {"X": X.float().cpu().numpy(), "v": v.cpu().numpy(), "u": u.cpu().numpy(),
            "mask": mask.cpu().numpy(), "res": ws.result()}


def weights_for(m, seed, spread=1.0):
    rng = np.random.default_rng([m, seed, 77])
    return np.exp(rng.uniform(-spread, spread, m)).astype(np.float32)


def weighted_eta(Y, q, w, frac):
    v = orc.column_norms(Y, q).astype(np.float64)
    return float(np.float32(frac * np.dot(w.astype(np.float64), v)))


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("q", ["inf", 1, 2])
@pytest.mark.parametrize("shape", [(1, 1), (9, 7), (256, 128), (300, 257), (2065, 264), (131, 1032), (40, 5000),
                                   (1000, 1024), (5, 16388), (3, 40001), (2500, 260), (2, 70000), (3, 300001)])
def test_weighted_outer_norm_matches_oracle(mp, storage, q, shape):
    """Alg. 1 with the weighted l1 ball as outer norm (Sec. 3), against the sort-based oracle."""
    Y = stored_input(shape, storage, 41)
    w = weights_for(shape[1], 1)
    for frac in (0.04, 0.5, 0.98):
        eta = weighted_eta(Y, q, w, frac)
        ref = orc.bilevel_stored(Y, eta, q, storage, p=("w1", w))
        got = run_weighted(mp, Y, eta, q, storage, w)
        check_stored(got, ref, q, storage)
        assert got["res"]["norm"] == pytest.approx(np.dot(w.astype(np.float64), ref["v"].astype(np.float64)), rel=1e-6)
        if q == 1 and shape[0] <= 4096 and shape[1] % (4 if storage == "f32" else 8) == 0:
            assert_columns_in_registers(got["res"])     # (the weighted search kernel ahead of the one-pass l1,1 kernel)


@pytest.mark.parametrize("q", ["inf", 1, 2])
def test_weighted_outer_norm_special_cases(mp, q):
    Y = stored_input((333, 520), "f32", 42)
    w = weights_for(520, 2, spread=3.0)         # weights over a range of 400 : 1
    v = orc.column_norms(Y, q).astype(np.float64)
    total = float(np.dot(w.astype(np.float64), v))
    eta = float(np.float32(0.3 * total))
    ref = orc.bilevel_stored(Y, eta, q, "f32", p=("w1", w))
    check_stored(run_weighted(mp, Y, eta, q, "f32", w), ref, q, "f32")
    check_stored(run_weighted(mp, Y, eta, q, "f32", w, inplace=True), ref, q, "f32")
    check_stored(run_weighted(mp, Y, eta, q, "f32", w, offset=1), ref, q, "f32")       # the element-wise path
    # inside the ball: nothing moves; radius 0: everything goes, tau = max v_j / w_j
    got = run_weighted(mp, Y, float(np.float32(1.5 * total)), q, "f32", w)
    assert np.array_equal(got["X"], Y) and got["mask"].all() and got["res"]["inside_ball"] and got["res"]["tau"] == 0.0
    got = run_weighted(mp, Y, 0.0, q, "f32", w)
    assert not got["X"].any() and not got["mask"].any()
    assert got["res"]["tau"] == pytest.approx(np.max(v / w.astype(np.float64)), rel=1e-12)
    # unit weights: the plain l1 outer norm (another summation order in the search: not bit for bit)
    one = np.ones(520, dtype=np.float32)
    eta = eta_for(Y, q, 0.3)
    check_stored(run_weighted(mp, Y, eta, q, "f32", one), orc.bilevel_stored(Y, eta, q, "f32"), q, "f32")
    # a tiny radius keeps the one column with the largest v_j / w_j
    j = int(np.argmax(v / w.astype(np.float64)))
    eta = float(np.float32(1e-4 * w[j] * v[j]))
    got = run_weighted(mp, Y, eta, q, "f32", w)
    check_stored(got, orc.bilevel_stored(Y, eta, q, "f32", p=("w1", w)), q, "f32")
    assert got["mask"].sum() == 1 and got["mask"][j] == 1


def test_weighted_outer_norm_special_cases_with_many_columns(mp):
    """The grid-wide form of the weighted search (more than 32768 columns): inside the ball, radius 0,
    a radius that keeps one column, unit weights."""
    Y = stored_input((4, 100003), "f32", 43)
    m = Y.shape[1]
    w = weights_for(m, 3, spread=2.0)
    for q in ("inf", 1):
        v = orc.column_norms(Y, q).astype(np.float64)
        total = float(np.dot(w.astype(np.float64), v))
        got = run_weighted(mp, Y, float(np.float32(1.1 * total)), q, "f32", w)
        assert np.array_equal(got["X"], Y) and got["mask"].all() and got["res"]["inside_ball"]
        got = run_weighted(mp, Y, 0.0, q, "f32", w)
        assert not got["X"].any() and not got["mask"].any()
        assert got["res"]["tau"] == pytest.approx(np.max(v / w.astype(np.float64)), rel=1e-12)
        j = int(np.argmax(v / w.astype(np.float64)))
        eta = float(np.float32(1e-3 * w[j] * v[j]))
        got = run_weighted(mp, Y, eta, q, "f32", w)
        check_stored(got, orc.bilevel_stored(Y, eta, q, "f32", p=("w1", w)), q, "f32")
        assert got["mask"].sum() == 1 and got["mask"][j] == 1
        eta = eta_for(Y, q, 0.2)
        one = np.ones(m, dtype=np.float32)
        check_stored(run_weighted(mp, Y, eta, q, "f32", one), orc.bilevel_stored(Y, eta, q, "f32"), q, "f32")


def test_weighted_outer_norm_on_the_headline_matrix(mp):
    """The 4096 x 4096 workload with the weights bench.py draws for it, q = inf in full and q = 1 on
    sampled columns."""
    w_, Y = workloads.make("square_4096")
    n, m = Y.shape
    w = np.exp(np.random.default_rng([n, m, 17]).uniform(-1, 1, m)).astype(np.float32)
    eta = weighted_eta(Y, "inf", w, w_.eta_frac)
    check_stored(run_weighted(mp, Y, eta, "inf", "f32", w), orc.bilevel_stored(Y, eta, "inf", "f32", p=("w1", w)), "inf", "f32")
    eta = weighted_eta(Y, 1, w, w_.eta_frac)
    cols = np.sort(np.random.default_rng(8).choice(m, size=96, replace=False))
    got = run_weighted(mp, Y, eta, 1, "f32", w)
    ref = orc.bilevel_l11(Y, eta, columns=cols, p=("w1", w))
    check_against_oracle(got, ref, 1, columns=cols)
    assert np.array_equal(got["mask"], (np.asarray(ref["u"]) > 0).astype(np.uint8))


def test_weighted_outer_norm_random_cases(mp):
    """Seeded random shapes, radii, value and weight distributions."""
    for seed in range(40):
        rng = np.random.default_rng([seed, 4242])
        n, m = int(rng.integers(1, 700)), int(rng.integers(1, 3000))
        q = ["inf", 1, 2][seed % 3]
        kind = seed % 4
        Y = (rng.standard_normal((n, m)) if kind < 2 else rng.laplace(size=(n, m)) ** 3).astype(np.float32)
        if kind == 1:
            Y *= (rng.random((1, m)) < 0.3)          # mostly empty columns
        w = np.exp(rng.uniform(-2, 2, m)).astype(np.float32)
        v = orc.column_norms(Y, q).astype(np.float64)
        total = float(np.dot(w.astype(np.float64), v))
        if total == 0.0:
            continue
        eta = float(np.float32(total * 10.0 ** rng.uniform(-4, 0)))
        check_stored(run_weighted(mp, Y, eta, q, "f32", w), orc.bilevel_stored(Y, eta, q, "f32", p=("w1", w)), q, "f32")


def test_stored_f32_is_the_fp32_entry_point_bit_for_bit(mp):
    dev = torch.device("cuda:0")
    for q in ("inf", 1, 2):
        Y = stored_input((700, 1028), "f32", 33)
        eta = eta_for(Y, q, 0.2)
        Yd = torch.from_numpy(Y).to(dev)
        a = mp.bilevel_proj_pq(1, q, Yd, eta)
        b = mp.bilevel_proj_stored(Yd, eta, q)
        assert torch.equal(a, b)


def test_stored_extreme_values(mp):
    """fp16 at the ends of its range (largest finite, subnormals); bf16 across fp32's exponents."""
    rng = np.random.default_rng(34)
    Yh = rng.standard_normal((64, 96)).astype(np.float32)
    Yh[:, :32] *= 2.0 ** -20            # subnormal fp16 territory after rounding
    Yh[:, 32:64] *= 9000.0
    Yh = np.clip(Yh, -65504.0, 65504.0)
    Yh[0, 40] = 65504.0
    Yh = orc.round_to_storage(Yh, "f16")
    Yb = orc.round_to_storage((rng.standard_normal((64, 96)) * 10.0 ** rng.uniform(-12, 12, 96)).astype(np.float32), "bf16")
    for Y, storage in ((Yh, "f16"), (Yb, "bf16")):
        for q in ("inf", 1, 2):
            eta = eta_for(Y, q, 0.5)
            ref = orc.bilevel_stored(Y, eta, q, storage)
            got = run_stored(mp, Y, eta, q, storage)
            assert np.array_equal(got["mask"], ref["mask"].astype(np.uint8))
            x = ref["X32"].astype(np.float64)
            tol = RTOL * np.abs(x) + 1e-30
            lo = orc.round_to_storage((x - tol).astype(np.float32), storage)
            hi = orc.round_to_storage((x + tol).astype(np.float32), storage)
            assert np.all((got["X"] >= lo) & (got["X"] <= hi))


# ------------------------------------------------------------------ l1,1 inner searches on hard inputs
def _hard_family(name, rng, n, m):
    if name == "cauchy":
        return rng.standard_cauchy((n, m))
    if name == "lognormal3":
        return rng.lognormal(0.0, 3.0, (n, m)) * rng.choice([-1.0, 1.0], (n, m))
    if name == "sparse":
        return rng.standard_normal((n, m)) * (rng.uniform(size=(n, m)) < 0.01)
    if name == "clusters":
        return np.where(rng.uniform(size=(n, m)) < 0.5, 1 + 0.01 * rng.standard_normal((n, m)),
                        10 + 0.1 * rng.standard_normal((n, m)))
    if name == "constant":
        return np.full((n, m), -2.5)
    if name == "integers":
        return rng.integers(-7, 8, (n, m)).astype(np.float64)
    if name == "geometric":
        return np.tile((0.999 ** np.arange(n))[:, None], (1, m))
    if name == "uniform":
        return rng.uniform(size=(n, m))
    raise KeyError(name)


@pytest.mark.parametrize("family", ["cauchy", "lognormal3", "sparse", "clusters", "constant", "integers",
                                    "geometric", "uniform"])
def test_l11_inner_searches_converge_on_hard_distributions(mp, family):
    """Heavy tails, clusters, ties and constant columns: the windowed lock-step search must
    close every column (inner_pending == 0, checked by check_against_oracle) well inside its
    sweep limit, and match the oracle's sort-based thresholds."""
    rng = np.random.default_rng([len(family), 77])
    n, m = 4099, 300
    Y = _hard_family(family, rng, n, m).astype(np.float32)
    for frac in (0.001, 0.1, 0.5, 0.95):
        eta = eta_for(Y, 1, frac)
        got = run_gpu(mp, Y, eta, 1)
        check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)
        assert got["res"]["inner_sweeps"] <= 10, (family, frac, got["res"]["inner_sweeps"])


@pytest.mark.parametrize("shape", [(32770, 1028), (16400, 2054)])
@pytest.mark.parametrize("family", ["gaussian", "laplace", "cauchy", "lognormal3", "sparse", "clusters", "constant",
                                    "integers", "geometric", "uniform", "misleading_head", "empty_head"])
def test_l11_grid_start_on_hard_distributions(mp, family, shape):
    """From 32M fp32 elements on the aggregate pass also evaluates every column on a grid of
    thresholds anchored at the mean magnitude of its first 128 rows, and the inner searches start
    from that instead of a probing pass.  Whatever the grid says (heavy tails, ties, a head that
    is a thousand times the rest or all zero), every threshold is still closed exactly.  The
    second shape has rows that are not 16-byte aligned."""
    rng = np.random.default_rng([len(family), shape[1], 80])
    n, m = shape
    if family == "gaussian":
        Y = rng.standard_normal((n, m))
    elif family == "laplace":
        Y = rng.laplace(size=(n, m))
    elif family in ("misleading_head", "empty_head"):
        Y = rng.standard_normal((n, m))
        Y[:128] *= 1000.0 if family == "misleading_head" else 0.0
    else:
        Y = _hard_family(family, rng, n, m)
    Y = Y.astype(np.float32)
    for frac in (0.001, 0.1, 0.5, 0.95):
        eta = eta_for(Y, 1, frac)
        got = run_gpu(mp, Y, eta, 1)
        check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)
        assert got["res"]["inner_sweeps"] <= 10, (family, frac, got["res"]["inner_sweeps"])


# ------------------------------------------------------------------ batches
BATCH_SHAPES = [(256, 128), (1, 1), (33, 20), (300, 257), (131, 1028), (64, 4100), (9, 5000), (512, 8192),
                (7, 16388), (40, 17000), (256, 128), (100, 260), (2065, 264), (5, 3), (77, 1024), (16, 16),
                (300, 300), (64, 64), (1000, 10)]      # 19 problems: two launches of the batch kernels


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("q", ["inf", 2, 1])
def test_batch_matches_oracle_and_single_calls(mp, q, storage):
    dev = torch.device("cuda:0")
    dt = getattr(torch, STORE_DTYPES[storage])
    Ys = [stored_input(sh, storage, 40 + i) for i, sh in enumerate(BATCH_SHAPES)]
    etas = [eta_for(Y, q, 0.05 + 0.9 * (i % 5) / 5) for i, Y in enumerate(Ys)]
    etas[3] = float(np.float32(2 * orc.norm_l1q(Ys[3], q)))     # one problem inside its ball
    etas[5] = 0.0                                               # one with radius zero
    Yd = [torch.from_numpy(Y).to(dev).to(dt) for Y in Ys]
    wss = [mp.Workspace.for_call(QNAME[q], *Y.shape, device=dev) for Y in Ys]
    vs = [torch.full((Y.shape[1],), -1.0, device=dev) for Y in Ys]
    us = [torch.full((Y.shape[1],), -1.0, device=dev) for Y in Ys]
    masks = [torch.full((Y.shape[1],), 7, dtype=torch.uint8, device=dev) for Y in Ys]
    Xs = mp.bilevel_proj_batch(Yd, etas, q, workspaces=wss, v_outs=vs, u_outs=us, mask_outs=masks)
    torch.cuda.synchronize()
    refs = orc.bilevel_batch(Ys, etas, q, storage)
    for i, (Y, ref) in enumerate(zip(Ys, refs)):
        got = {"X": Xs[i].float().cpu().numpy(), "v": vs[i].cpu().numpy(), "u": us[i].cpu().numpy(),
               "mask": masks[i].cpu().numpy(), "res": wss[i].result()}
        check_stored(got, ref, q, storage)
        single = mp.bilevel_proj_stored(Yd[i], etas[i], q)
        assert torch.equal(single, Xs[i]), "problem %d differs from its single call" % i


def test_batch_l11_problems_keep_their_own_sweep_plans(mp, l11_sweeps):
    """Heights from 3 to 9000 rows plan 1 to 6 lock-step sweeps; heavy tails need the finishing
    pass for some problems and not for others; all in one batch, and again with a fixed count."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(91)
    shapes = [(3, 40), (600, 33), (2500, 100), (5000, 64), (9000, 48), (700, 2000), (4097, 17)]
    Ys = []
    for i, sh in enumerate(shapes):
        Y = rng.standard_cauchy(sh) if i % 2 else rng.standard_normal(sh)
        Ys.append(Y.astype(np.float32))
    etas = [eta_for(Y, 1, [0.001, 0.3, 0.9][i % 3]) for i, Y in enumerate(Ys)]
    refs = orc.bilevel_batch(Ys, etas, 1, "f32")
    for fixed in (0, 2):
        l11_sweeps(fixed)
        Yd = [torch.from_numpy(Y).to(dev) for Y in Ys]
        wss = [mp.Workspace.for_call("l11", *Y.shape, device=dev) for Y in Ys]
        Xs = mp.bilevel_proj_batch(Yd, etas, 1, workspaces=wss)
        torch.cuda.synchronize()
        for i, ref in enumerate(refs):
            res = wss[i].result()
            assert res["inner_pending"] == 0
            np.testing.assert_allclose(Xs[i].cpu().numpy(), ref["X32"], rtol=RTOL, atol=ATOL)
            assert np.array_equal(Xs[i].cpu().numpy().any(axis=0), ref["mask"])
            assert torch.equal(mp.bilevel_proj_l11(Yd[i], etas[i]), Xs[i])


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_batch_l11_columns_in_registers(mp, storage):
    """Problems a single call keeps in registers take the same kernel inside a batch (32, 64 and
    128 values per thread in one launch), next to one whose search runs ahead and one with
    unaligned rows; the bits of the single calls either way."""
    dev = torch.device("cuda:0")
    dt = getattr(torch, STORE_DTYPES[storage])
    shapes = [(256, 128), (1024, 1024), (2048, 64), (4096, 32), (700, 2000), (37, 48), (3000, 400), (100, 4096),
              (130, 8200), (600, 33), (1, 8), (4096, 528)]
    Ys = [stored_input(sh, storage, 90 + i) for i, sh in enumerate(shapes)]
    etas = [eta_for(Y, 1, [0.01, 0.3, 0.9, 1.5][i % 4]) for i, Y in enumerate(Ys)]
    Yd = [torch.from_numpy(Y).to(dev).to(dt) for Y in Ys]
    wss = [mp.Workspace.for_call("l11", *Y.shape, device=dev) for Y in Ys]
    vs = [torch.full((Y.shape[1],), -1.0, device=dev) for Y in Ys]
    us = [torch.full((Y.shape[1],), -1.0, device=dev) for Y in Ys]
    masks = [torch.full((Y.shape[1],), 7, dtype=torch.uint8, device=dev) for Y in Ys]
    Xs = mp.bilevel_proj_batch(Yd, etas, 1, workspaces=wss, v_outs=vs, u_outs=us, mask_outs=masks)
    torch.cuda.synchronize()
    refs = orc.bilevel_batch(Ys, etas, 1, storage)
    for i, (Y, ref) in enumerate(zip(Ys, refs)):
        got = {"X": Xs[i].float().cpu().numpy(), "v": vs[i].cpu().numpy(), "u": us[i].cpu().numpy(),
               "mask": masks[i].cpu().numpy(), "res": wss[i].result()}
        check_stored(got, ref, 1, storage)
        if shapes[i] != (600, 33):
            assert_columns_in_registers(got["res"])
        assert torch.equal(mp.bilevel_proj_stored(Yd[i], etas[i], 1), Xs[i]), "problem %d differs from its single call" % i


def test_prepared_batch_can_be_called_again_on_new_contents(mp):
    """The argument block is marshalled once; the buffers it points to may change between calls."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(17)
    shapes = [(256, 128), (40, 1000), (700, 300), (64, 64)]
    Ys = [rng.standard_normal(sh).astype(np.float32) for sh in shapes]
    Yd = [torch.from_numpy(Y).to(dev) for Y in Ys]
    etas = [eta_for(Y, "inf", 0.2) for Y in Ys]
    batch = mp.PreparedBatch(Yd, etas, "inf")
    for rep in range(3):
        Xs = batch()
        torch.cuda.synchronize()
        for Y, eta, X in zip(Ys, etas, Xs):
            np.testing.assert_allclose(X.cpu().numpy(), orc.bilevel(Y, eta, "inf")["X"], rtol=RTOL, atol=ATOL)
        Ys = [np.float32(0.5) * Y + np.float32(rep) for Y in Ys]     # new contents, same buffers
        for d, Y in zip(Yd, Ys):
            d.copy_(torch.from_numpy(Y))


def test_batch_in_place_and_kernel_count(mp):
    """In place; and the launches of a small batch, seen through the event trace: one for the matrices
    of at most 128 KiB (one workgroup each when in place), three for the others."""
    dev = torch.device("cuda:0")
    Ys = [stored_input(sh, "f32", 60 + i) for i, sh in enumerate(BATCH_SHAPES[:8])]
    etas = [eta_for(Y, "inf", 0.3) for Y in Ys]
    Yd = [torch.from_numpy(Y).to(dev) for Y in Ys]
    tr = mp.KernelTrace(16)
    with tr:
        mp.bilevel_proj_batch(Yd, etas, "inf", Xs=Yd)
    tr.durations_ms()
    tr.close()
    assert tr.count == 6          # the one-kernel form and its closing event; aggregate, fold, map and the closing event
    for Y, eta, X in zip(Ys, etas, Yd):
        np.testing.assert_allclose(X.cpu().numpy(), orc.bilevel(Y, eta, "inf")["X"], rtol=RTOL, atol=ATOL)
        assert torch.equal(X, mp.bilevel_proj_stored(torch.from_numpy(Y).to(dev), eta, "inf")), "differs from the single call"
    # sixteen small matrices in place, as a training loop would: one launch, one workgroup each
    Ys = [stored_input((256, 128), "f32", 80 + i) for i in range(16)]
    etas = [eta_for(Y, 2, 0.2) for Y in Ys]
    Yd = [torch.from_numpy(Y).to(dev) for Y in Ys]
    tr = mp.KernelTrace(16)
    with tr:
        mp.bilevel_proj_batch(Yd, etas, 2, Xs=Yd)
    tr.durations_ms()
    tr.close()
    assert tr.count == 2
    for Y, eta, X in zip(Ys, etas, Yd):
        np.testing.assert_allclose(X.cpu().numpy(), orc.bilevel(Y, eta, 2)["X"], rtol=RTOL, atol=ATOL)
        assert torch.equal(X, mp.bilevel_proj_stored(torch.from_numpy(Y).to(dev), eta, 2))


# ------------------------------------------------------------------ seeded random cases
@pytest.mark.parametrize("seed", range(40))
def test_random_shapes_and_options(mp, seed):
    """Shape, storage type, inner and outer norm, radius and pointer offsets drawn from a seed."""
    rng = np.random.default_rng([seed, 2405])
    n = int(np.exp(rng.uniform(0, np.log(3000))))
    m = int(np.exp(rng.uniform(0, np.log(6000))))
    q = ["inf", 1, 2][rng.integers(3)]
    p = [1, 1, 2, "inf"][rng.integers(4)]
    storage = ["f32", "bf16", "f16"][rng.integers(3)]
    dist = rng.integers(3)
    Y = (rng.standard_normal((n, m)) if dist == 0 else rng.laplace(size=(n, m)) if dist == 1
         else rng.uniform(-1, 1, (n, m))).astype(np.float32)
    if rng.integers(2):
        Y *= np.power(10.0, rng.uniform(-2, 0, m)).astype(np.float32)[None, :]
    Y = orc.round_to_storage(Y, storage)
    v = orc.column_norms(Y, q).astype(np.float64)
    norm_p = v.sum() if p == 1 else (np.sqrt((v * v).sum()) if p == 2 else v.max())
    eta = float(np.float32(rng.uniform(0.01, 1.1) * norm_p))
    offset, x_offset = int(rng.integers(0, 4)), int(rng.integers(0, 4))
    got = run_stored(mp, Y, eta, q, storage, p=p, offset=offset, x_offset=x_offset)
    check_stored(got, orc.bilevel_stored(Y, eta, q, storage, p=p), q, storage)


def _adversarial_l11_cases():
    rng = np.random.default_rng(5)
    n, m = 1037, 130
    cases = {}
    cases["binary"] = (rng.uniform(size=(n, m)) < 0.3).astype(np.float32)
    c = np.full((n, m), 1e-30, np.float32)
    c[rng.integers(0, n, m), np.arange(m)] = 1e30
    cases["outlier"] = c
    cases["pow2"] = np.tile((2.0 ** -(np.arange(n) % 40))[:, None], (1, m)).astype(np.float32)
    t = np.ones((n, m), np.float32)
    t[: n // 3] = 3.0
    cases["two_levels"] = t
    cases["two_rows"] = rng.standard_normal((2, 5000)).astype(np.float32)
    cases["denormal"] = (rng.standard_normal((n, m)) * 1e-41).astype(np.float32)
    cases["huge"] = (rng.standard_normal((n, m)) * 1e30).astype(np.float32)
    cases["ramp"] = np.tile(np.arange(1, n + 1, dtype=np.float32)[:, None], (1, m))
    cases["mixed_columns"] = np.concatenate([cases["binary"][:, :40], cases["pow2"][:, :40],
                                             rng.standard_cauchy((n, 50)).astype(np.float32)], axis=1)
    return cases


@pytest.mark.parametrize("name", ["binary", "outlier", "pow2", "two_levels", "two_rows", "denormal", "huge", "ramp",
                                  "mixed_columns"])
def test_l11_inner_searches_on_adversarial_columns(mp, name):
    """Ties everywhere, one giant entry, powers of two, subnormal and huge magnitudes, and
    columns of different kinds side by side (lock step must serve the slowest)."""
    Y = _adversarial_l11_cases()[name]
    for frac in (1e-4, 0.01, 0.3, 0.9, 0.999):
        eta = eta_for(Y, 1, frac)
        got = run_gpu(mp, Y, eta, 1)
        check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)
        assert got["res"]["inner_sweeps"] <= 10


@pytest.mark.parametrize("sweeps", [1, 2, 4])
@pytest.mark.parametrize("family", ["gaussian", "cauchy", "lognormal3", "sparse", "clusters", "constant",
                                    "integers", "geometric", "uniform"])
def test_l11_finishing_pass_closes_what_the_sweeps_leave(mp, l11_sweeps, family, sweeps):
    """With few lock-step sweeps the column-wise finishing pass does most of the work (all of
    it after one sweep): same thresholds as the oracle's sort, nothing left pending."""
    rng = np.random.default_rng([len(family), 78, sweeps])
    n, m = 1037, 301            # ragged in both directions: 1037 = 2*512 + 13 rows, 301 = 18*16 + 13 columns
    Y = (rng.standard_normal((n, m)) if family == "gaussian" else _hard_family(family, rng, n, m)).astype(np.float32)
    l11_sweeps(sweeps)
    finished = 0
    for frac in (0.001, 0.1, 0.5, 0.95):
        eta = eta_for(Y, 1, frac)
        got = run_gpu(mp, Y, eta, 1)
        check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)
        assert got["res"]["inner_sweeps"] <= sweeps
        finished += got["res"]["inner_finished"]
    if sweeps == 1 and family == "gaussian":
        assert finished > 0, "one sweep cannot close Gaussian columns: the finishing pass must have run"


@pytest.mark.parametrize("n", [37, 600, 1024, 1025, 2049])
@pytest.mark.parametrize("family", ["gaussian", "cauchy", "lognormal3", "sparse", "clusters", "constant",
                                    "integers", "geometric", "uniform"])
def test_l11_default_plan_on_short_matrices(mp, family, n):
    """Whole calls of at most 4096 rows hold the columns in registers: no lock-step sweep.  Split calls take the
    sweeps' kernels, up to 4M elements without a sweep: up to 1024 rows the finishing kernel that seeds itself and runs
    the outer search, the seeding and finishing kernels above."""
    rng = np.random.default_rng([len(family), 79, n])
    m = 150
    Y = (rng.standard_normal((n, m)) if family == "gaussian" else _hard_family(family, rng, n, m)).astype(np.float32)
    for frac in (0.001, 0.1, 0.5, 0.95):
        eta = eta_for(Y, 1, frac)
        got = run_gpu(mp, Y, eta, 1)
        check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)
        assert got["res"]["inner_sweeps"] == 0
        ref = orc.bilevel(Y, eta, 1)
        got = split_call(mp, Y, eta, 1)
        check_against_oracle(got, ref, 1)
        assert got["res"]["inner_sweeps"] == 0
        assert got["res"]["inner_finished"] == (0 if got["res"]["inside_ball"] else got["res"]["n_active"])


@pytest.mark.parametrize("name", ["binary", "outlier", "pow2", "two_levels", "two_rows", "denormal", "huge", "ramp",
                                  "mixed_columns"])
def test_l11_finishing_pass_on_adversarial_columns(mp, l11_sweeps, name):
    Y = _adversarial_l11_cases()[name]
    l11_sweeps(1)
    for frac in (1e-4, 0.3, 0.999):
        eta = eta_for(Y, 1, frac)
        got = run_gpu(mp, Y, eta, 1)
        check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)


@pytest.mark.parametrize("storage", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("shape", [(1, 1), (3, 17), (70, 4104), (2065, 264), (5000, 40)])
def test_l11_finishing_pass_on_stored_types_and_odd_shapes(mp, l11_sweeps, storage, shape):
    Y = stored_input(shape, storage, 35)
    l11_sweeps(1)
    for frac in (0.05, 0.6):
        eta = eta_for(Y, 1, frac)
        check_stored(run_stored(mp, Y, eta, 1, storage), orc.bilevel_stored(Y, eta, 1, storage), 1, storage)
    check_stored(run_stored(mp, Y, eta_for(Y, 1, 0.3), 1, storage, offset=1, x_offset=3),
                 orc.bilevel_stored(Y, eta_for(Y, 1, 0.3), 1, storage), 1, storage)


def test_l11_sweep_count_does_not_change_the_result(mp, l11_sweeps):
    """The thresholds are exact whichever pass closes a column, so X agrees to the last few bits."""
    Y = workloads.generate((777, 1024), seed=5)
    eta = eta_for(Y, 1, 0.2)
    outs = []
    for k in (1, 3, 16, 0):
        l11_sweeps(k)
        outs.append(run_gpu(mp, Y, eta, 1))
    for o in outs[1:]:
        np.testing.assert_allclose(o["X"], outs[0]["X"], rtol=0, atol=1e-6)
        assert np.array_equal(o["X"] != 0, outs[0]["X"] != 0)
    assert outs[0]["res"]["inner_finished"] > 0 and outs[2]["res"]["inner_finished"] == 0


def test_l11_root_exactly_on_repeated_entries(mp):
    """Columns (3,3,3,1,1) with u_j = 6: the inner threshold is exactly 1, the value of two entries."""
    Y = np.tile(np.float32([3, 3, 3, 1, 1])[:, None], (1, 64))
    got = run_gpu(mp, Y, 384.0, 1)          # v_j = 11, tau = 5, u_j = 6
    ref = orc.bilevel(Y, 384.0, 1)
    assert np.allclose(ref["tau_col"], 1.0) and ref["tau"] == 5.0
    check_against_oracle(got, ref, 1)


# ------------------------------------------------------------------ l1,1 with the columns in registers
# Up to 4096 rows and 64M elements one kernel holds 16 whole columns per
# workgroup, runs the inner searches there and maps from the same registers.  The result record
# shows it: no lock-step sweep, every kept column closed by the column-wise pass.
# (rows: 1..4096 around the 1024 / 2048 register-count steps; columns: ragged stripes, more than
# 32 stripes so that the stripe-to-workgroup permutation has full runs and a rest, and more than
# 4096 columns, where a search kernel runs ahead)
LH_SHAPES = [(1, 4), (5, 16), (37, 48), (1024, 64), (1025, 36), (2048, 20), (2049, 532), (4096, 16), (4096, 532),
             (300, 1100), (333, 4100), (130, 8200), (1000, 10000), (2100, 1024)]


def assert_columns_in_registers(res):
    assert res["inner_sweeps"] == 0 and res["inner_pending"] == 0
    assert res["inner_finished"] == (0 if res["inside_ball"] else res["n_active"])


@pytest.mark.parametrize("shape", LH_SHAPES)
def test_l11_columns_in_registers_matches_oracle(mp, shape):
    Y = workloads.generate(shape, seed=61)
    for frac in (0.001, 0.1, 0.5, 0.95, 1.5):
        eta = eta_for(Y, 1, frac)
        got = run_gpu(mp, Y, eta, 1)
        check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)
        assert_columns_in_registers(got["res"])
    got = run_gpu(mp, Y, 0.0, 1)
    assert not got["X"].any() and not got["u"].any() and got["res"]["n_active"] == 0


@pytest.mark.parametrize("n", [700, 1500, 2500])
@pytest.mark.parametrize("family", ["cauchy", "lognormal3", "sparse", "clusters", "constant", "integers",
                                    "geometric", "uniform"])
def test_l11_columns_in_registers_on_hard_distributions(mp, family, n):
    """32, 64 and 128 values per thread; heavy tails, ties, constant and sparse columns."""
    rng = np.random.default_rng([len(family), 81, n])
    Y = _hard_family(family, rng, n, 528).astype(np.float32)
    for frac in (0.001, 0.1, 0.5, 0.95):
        eta = eta_for(Y, 1, frac)
        got = run_gpu(mp, Y, eta, 1)
        check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)
        assert_columns_in_registers(got["res"])


@pytest.mark.parametrize("name", ["binary", "outlier", "pow2", "two_levels", "two_rows", "denormal", "huge", "ramp",
                                  "mixed_columns"])
def test_l11_columns_in_registers_on_adversarial_columns(mp, name):
    Y = _adversarial_l11_cases()[name]
    Y = np.ascontiguousarray(Y[:, : Y.shape[1] // 4 * 4])
    for frac in (1e-4, 0.01, 0.3, 0.9, 0.999):
        eta = eta_for(Y, 1, frac)
        got = run_gpu(mp, Y, eta, 1)
        check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)
        assert_columns_in_registers(got["res"])


@pytest.mark.parametrize("ties", [1, 2, 31, 32, 33, 127, 128, 129, 500])
def test_l11_columns_in_registers_entries_close_to_the_threshold(mp, ties):
    """The window the second evaluation lists (128 entries per column): as many entries as named lie next to the root of
    every column, equal in some columns and one float apart in the others, on wide, ragged and narrow stripes."""
    for n, m in ((1500, 48), (1499, 37), (4500, 24)):
        rng = np.random.default_rng([n, ties])
        Y = rng.standard_normal((n, m)).astype(np.float32)
        eta = eta_for(Y, 1, 0.2)
        ref = orc.bilevel(Y, eta, 1)
        kept = np.abs(ref["X"]) > 0
        for j in range(m):
            rows = np.flatnonzero(kept[:, j])
            if rows.size == 0:
                continue
            root = np.float32(np.abs(Y[rows[0], j].astype(np.float64)) - np.abs(ref["X"][rows[0], j]))
            near = np.full(ties, root)
            if j % 2:
                near = (root.view(np.int32) + np.arange(ties) - ties // 2).astype(np.int32).view(np.float32)
            where = rng.permutation(n)[:ties]
            Y[where, j] = np.where(Y[where, j] < 0, -near, near)
        got = run_gpu(mp, Y, eta, 1)
        check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)
        assert_columns_in_registers(got["res"])


@pytest.mark.parametrize("shape", [(4097, 8), (4100, 36), (5000, 264), (8192, 20), (8192, 516), (6000, 2048), (7000, 1000)])
def test_l11_columns_in_registers_narrow_stripes(mp, shape):
    """fp32 matrices of 4097 to 8192 rows and at most 2048 columns: stripes of 8 columns, 128
    values per thread (ragged stripes, more than 32 of them, the most the form takes)."""
    rng = np.random.default_rng([shape[0], shape[1], 83])
    for family in ("gaussian", "cauchy", "integers"):
        Y = (rng.standard_normal(shape) if family == "gaussian" else _hard_family(family, rng, *shape)).astype(np.float32)
        for frac in (0.001, 0.3, 0.95, 1.5):
            eta = eta_for(Y, 1, frac)
            got = run_gpu(mp, Y, eta, 1)
            check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)
            assert_columns_in_registers(got["res"])
    got = run_gpu(mp, Y, eta_for(Y, 1, 0.2), 1, inplace=True)
    check_against_oracle(got, orc.bilevel(Y, eta_for(Y, 1, 0.2), 1), 1)
    assert_columns_in_registers(got["res"])


@pytest.mark.parametrize("storage", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("shape", [(1, 8), (70, 4104), (2065, 264), (4096, 40), (1000, 72), (3000, 1032)])
def test_l11_columns_in_registers_on_stored_types(mp, storage, shape):
    Y = stored_input(shape, storage, 36)
    for frac in (0.05, 0.6, 1.2):
        eta = eta_for(Y, 1, frac)
        got = run_stored(mp, Y, eta, 1, storage)
        check_stored(got, orc.bilevel_stored(Y, eta, 1, storage), 1, storage)
        assert_columns_in_registers(got["res"])
    eta = eta_for(Y, 1, 0.3)
    got = run_stored(mp, Y, eta, 1, storage, inplace=True)
    check_stored(got, orc.bilevel_stored(Y, eta, 1, storage), 1, storage)
    assert_columns_in_registers(got["res"])


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_l11_columns_in_registers_skips_dropped_stripes(mp, storage):
    """More than 4096 columns (the search runs ahead): a few columns carry all the weight, so whole
    stripes are dropped and zeroed without being read; neighbours of kept columns inside a kept
    stripe, stripes at the ragged end, in place, and X pre-filled with other values."""
    rng = np.random.default_rng(85)
    n, m = 600, 4648
    Y = rng.standard_normal((n, m)).astype(np.float32)
    heavy = np.r_[3, 4, 1000, 2047, 2048, 4632, 4647]
    Y[:, heavy] *= 50.0
    Y = orc.round_to_storage(Y, storage)
    for frac in (0.01, 0.03):
        eta = eta_for(Y, 1, frac)
        ref = orc.bilevel_stored(Y, eta, 1, storage)
        assert 0 < int(ref["mask"].sum()) <= len(heavy), "only heavy columns survive this radius"
        for inplace in (False, True):
            got = run_stored(mp, Y, eta, 1, storage, inplace=inplace)
            check_stored(got, ref, 1, storage)
            assert_columns_in_registers(got["res"])


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_l11_sweeps_skip_tiles_without_open_columns(mp, storage):
    """Too tall for the columns-in-registers kernel: a few heavy columns in two of the five
    256-column tiles carry all the weight, so the sweeps and the map pass skip the other tiles
    (and zero them); next to a radius that keeps every column."""
    rng = np.random.default_rng(86)
    n, m = 8300, 1100
    Y = rng.standard_normal((n, m)).astype(np.float32)
    heavy = np.r_[5, 6, 255, 1030, 1099]
    Y[:, heavy] *= 50.0
    Y = orc.round_to_storage(Y, storage)
    for frac, sparse in ((0.01, True), (0.04, True), (0.6, False)):
        eta = eta_for(Y, 1, frac)
        ref = orc.bilevel_stored(Y, eta, 1, storage)
        assert (int(ref["mask"].sum()) <= len(heavy)) == sparse
        for inplace in (False, True):
            got = run_stored(mp, Y, eta, 1, storage, inplace=inplace)
            check_stored(got, ref, 1, storage)
            assert got["res"]["inner_sweeps"] >= 1


def test_l11_columns_in_registers_in_place_and_against_the_sweeps(mp, l11_sweeps):
    """In place, twice on the same workspace, and the same thresholds as the lock-step sweeps give
    (both are exact, so X agrees to the last few bits)."""
    Y = workloads.generate((3000, 2052), seed=62)
    eta = eta_for(Y, 1, 0.2)
    dev = torch.device("cuda:0")
    ws = mp.Workspace.for_call("l11", 3000, 2052, device=dev)
    a = run_gpu(mp, Y, eta, 1, workspace=ws)
    b = run_gpu(mp, Y, eta, 1, workspace=ws, inplace=True)
    assert np.array_equal(a["X"], b["X"]) and np.array_equal(a["u"], b["u"])
    assert_columns_in_registers(b["res"])
    l11_sweeps(3)
    c = run_gpu(mp, Y, eta, 1, workspace=ws)
    assert c["res"]["inner_sweeps"] >= 1
    np.testing.assert_allclose(c["X"], a["X"], rtol=0, atol=1e-6)
    assert np.array_equal(c["X"] != 0, a["X"] != 0)


# ------------------------------------------------------------------ tri-level on 16-bit storage
@pytest.mark.parametrize("storage", ["bf16", "f16", "f32"])
# (the last three shapes are 1 MiB and more in every storage type: several pieces per slab in the one-pass kernel)
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 4, 5), (17, 16, 16), (6, 50, 41), (300, 3, 2), (4, 64, 1024), (40, 33, 264),
                                   (16, 128, 1024), (200, 40, 1000), (3, 1, 1000008)])
def test_trilevel_stored_matches_oracle(mp, storage, shape):
    dev = torch.device("cuda:0")
    dt = getattr(torch, STORE_DTYPES[storage])
    rng = np.random.default_rng(list(shape) + [9])
    Y = orc.round_to_storage(rng.standard_normal(shape).astype(np.float32), storage)
    w = np.abs(Y).reshape(shape[0], -1).max(axis=1).astype(np.float64)
    Yd = torch.from_numpy(Y).to(dev).to(dt)
    for frac in (0.1, 0.7, 1.5, 0.0):
        eta = float(np.float32(frac * w.sum()))
        ws = mp.Workspace.for_call("tri", *shape, device=dev)
        v = torch.full((shape[0],), -1.0, device=dev)
        u = torch.full((shape[0],), -1.0, device=dev)
        mask = torch.full((shape[0],), 7, dtype=torch.uint8, device=dev)
        X = mp.trilevel_proj_stored(Yd, eta, workspace=ws, v_out=v, u_out=u, mask_out=mask)
        torch.cuda.synchronize()
        ref = orc.trilevel_stored(Y, eta, storage)
        assert np.array_equal(v.cpu().numpy(), ref["w"])
        np.testing.assert_allclose(u.cpu().numpy(), np.asarray(ref["u"], dtype=np.float32), rtol=RTOL, atol=ATOL)
        assert np.array_equal(mask.cpu().numpy(), ref["mask"].astype(np.uint8))
        x = ref["X32"].astype(np.float64)
        tol = RTOL * np.abs(x) + ATOL
        lo = orc.round_to_storage((x - tol).astype(np.float32), storage)
        hi = orc.round_to_storage((x + tol).astype(np.float32), storage)
        got = X.float().cpu().numpy()
        assert np.all((got >= lo) & (got <= hi))
        if storage == "f32":
            assert torch.equal(X, mp.trilevel_proj_l1infinf(Yd, eta))


# ------------------------------------------------------------------ multi-level on 16-bit storage
ML_STORED_CASES = [
    ((5, 7), [1]), ((300, 33), [2]), ((6, 1032), [1]), ((4, 3, 5), [1, 1]), ((9, 16, 8), ["inf", 1]),
    ((7, 5, 64), [1, "inf"]), ((3, 40, 264), [1, 1]), ((3, 40, 264), [2, 1]), ((5, 4, 3, 16), [1, 1, 1]),
    ((5, 4, 3, 6), ["inf", 2, 1]), ((40, 24, 40), ["inf", "inf"]), ((3, 1, 2000), [2, 2]), ((2, 2, 5000), [1, 2]),
]


@pytest.mark.parametrize("storage", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("shape,norms", ML_STORED_CASES)
def test_multilevel_stored_matches_oracle(mp, storage, shape, norms):
    """Wide (last axis a multiple of 16 bytes) and element-wise paths, short and long fibres."""
    dev = torch.device("cuda:0")
    dt = getattr(torch, STORE_DTYPES[storage])
    rng = np.random.default_rng(list(shape) + [len(norms), 5])
    Y = orc.round_to_storage(rng.standard_normal(shape).astype(np.float32), storage)
    nrm = nested_norm(Y, norms)
    for frac, p in ((0.05, 1), (0.5, 1), (1.5, 1), (0.4, 2), (0.4, "inf")):
        w = orc.multilevel(Y, norms, 1e30)["w"]
        norm_p = nrm if p == 1 else (float(np.sqrt((w * w).sum())) if p == 2 else float(w.max()))
        eta = float(np.float32(frac * norm_p))
        Yd = torch.from_numpy(Y).to(dev).to(dt)
        assert np.array_equal(Yd.float().cpu().numpy(), Y)
        v = torch.full((shape[0],), -1.0, device=dev)
        u = torch.full((shape[0],), -1.0, device=dev)
        ws = mp.Workspace(mp.multilevel_workspace_bytes(shape), device=dev)
        X = mp.multilevel_proj_stored(Yd, norms, eta, p=p, workspace=ws, v_out=v, u_out=u)
        torch.cuda.synchronize()
        ref = orc.multilevel_stored(Y, norms, eta, storage, p=p)
        np.testing.assert_allclose(v.cpu().numpy(), ref["w"].astype(np.float32), rtol=2e-7)
        np.testing.assert_allclose(u.cpu().numpy(), ref["u"].astype(np.float32), rtol=RTOL, atol=ATOL)
        x = ref["X32"].astype(np.float64)
        tol = RTOL * np.abs(x) + ATOL
        lo = orc.round_to_storage((x - tol).astype(np.float32), storage)
        hi = orc.round_to_storage((x + tol).astype(np.float32), storage)
        got = X.float().cpu().numpy()
        assert np.all((got >= lo) & (got <= hi))
        if storage != "f32":
            assert np.mean(got != ref["X"]) < 0.02
        # in place gives the same bits
        Xi = mp.multilevel_proj_stored(Yd, norms, eta, p=p, X=Yd, workspace=ws)
        assert torch.equal(Xi, X)


def test_multilevel_stored_f32_is_the_fp32_entry_point_bit_for_bit(mp):
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(77)
    Y = torch.from_numpy(rng.standard_normal((12, 20, 36)).astype(np.float32)).to(dev)
    for norms in ([1, 1], [2, "inf"], ["inf", "inf"]):
        eta = float(np.float32(0.3 * nested_norm(Y.cpu().numpy(), norms)))
        assert torch.equal(mp.multilevel_proj(Y, norms, eta), mp.multilevel_proj_stored(Y, norms, eta))


# ------------------------------------------------------------------ matrices of at most 128 KiB (one kernel)
TINY_SHAPES = {"f32": [(256, 128), (16, 2048), (1, 2048), (8, 2048), (64, 512), (100, 64), (3, 8), (16, 4), (512, 4),
                       (255, 124), (17, 1000)],
               "bf16": [(128, 512), (256, 256), (16, 4096), (40, 1000), (2, 8)],
               "f16": [(128, 512), (100, 24)]}


def chain_result(mp, Y, eta, q, storage):
    """X of the general chain of kernels: a split call (fp32), or a weighted one with all weights 1 (16-bit storage: the
    search of a weighted ball is a kernel of its own).  Neither ever takes the one-kernel form, as the trace shows."""
    with mp.KernelTrace(24) as tr:
        if storage == "f32":
            X = split_call(mp, Y, eta, q)["X"]
        else:
            Yd = torch.from_numpy(Y).to("cuda:0").to(getattr(torch, STORE_DTYPES[storage]))
            X = mp.bilevel_proj_weighted(Yd, eta, q, torch.ones(Y.shape[1], device="cuda:0")).float().cpu().numpy()
    tr.close()
    assert tr.count > 3, "an aggregate, a search and a map at least"
    return X


@pytest.mark.parametrize("q", ["inf", 2, 1])   # (q = 1 has no one-kernel form: the general path)
@pytest.mark.parametrize("storage,shape", [(st, sh) for st, shapes in TINY_SHAPES.items() for sh in shapes])
def test_tiny_matrices_one_kernel_path(mp, storage, shape, q):
    """A matrix small enough for the single-kernel path: the oracle's result, one kernel in the
    trace, what the chain of kernels gives (its sums run in another order: tau to a few units of fp64, so a radius
    to one unit of fp32 and X to one unit of its storage type, with an absolute part where v_j - tau cancels), and the
    same bits again on rows that are not 16-byte aligned and when projected in place (one workgroup does the whole
    matrix)."""
    dev = torch.device("cuda:0")
    dt = getattr(torch, STORE_DTYPES[storage])
    Y = stored_input(shape, storage, 71)
    for frac, p in ((0.05, 1), (0.6, 1), (1.5, 1), (0.0, 1), (0.4, 2), (0.4, "inf")):
        v = orc.column_norms(Y, q).astype(np.float64)
        norm_p = v.sum() if p == 1 else (np.sqrt((v * v).sum()) if p == 2 else v.max())
        eta = float(np.float32(frac * norm_p))
        got = run_stored(mp, Y, eta, q, storage, p=p)
        check_stored(got, orc.bilevel_stored(Y, eta, q, storage, p=p), q, storage)
        assert np.array_equal(run_stored(mp, Y, eta, q, storage, p=p, offset=1)["X"], got["X"])
        if p == 1:
            np.testing.assert_allclose(chain_result(mp, Y, eta, q, storage), got["X"], rtol={"f32": 2.0 ** -22, "bf16": 2.0 ** -7, "f16": 2.0 ** -10}[storage],
                                       atol=2.0 ** -24 if storage == "f16" else 1e-12 * np.abs(Y).max() if q != 1 else ATOL)
        inplace = torch.from_numpy(Y).to(dev).to(dt)
        mp.bilevel_proj_stored(inplace, eta, q, p=p, X=inplace)
        assert np.array_equal(inplace.float().cpu().numpy(), got["X"]), "in place differs from out of place"
    for inplace in (False, True):
        Yd = torch.from_numpy(Y).to(dev).to(dt)
        ws = mp.Workspace.for_call(QNAME[q], *shape, device=dev)
        tr = mp.KernelTrace(8)
        with tr:
            mp.bilevel_proj_stored(Yd, eta, q, X=Yd if inplace else None, workspace=ws)
        tr.durations_ms()
        tr.close()
        if q != 1:
            assert tr.count == 2, "one kernel and the closing event"
