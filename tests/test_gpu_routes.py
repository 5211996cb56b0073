"""The routes a call can take by its sizes and alignment, each at the sizes where it can go wrong, against the oracle
(the bars of test_gpu_parity.py) or bit for bit against the route that computes the same sums in the same order."""
import numpy as np
import pytest

from oracle import mlproj_oracle as orc
from test_gpu_parity import (ATOL, QNAME, RTOL, STORE_DTYPES, check_against_oracle, check_multi, check_stored, eta_for, nested_norm,  # noqa: F401
                             run_gpu, run_multi, run_stored, run_weighted, stored_input, mp)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", ["inf", 2])
@pytest.mark.parametrize("shapes", [[(1024, 1024)] * 16, [(20000, 64)] + [(100, 16384)] * 12, [(4099, 4097)], [(17, 300), (16, 5000)], [(2000, 4096), (256, 256)], [(10000, 256)] * 8])
def test_batch_map_grid_is_planned_for_the_launch(mp, q, shapes):
    """Batches whose map workgroups take several row blocks each, a tall matrix beside wide ones (more column tiles
    than workgroups planned for), one matrix alone, ragged last blocks, the grids of the single calls kept, and narrow matrices:
    the bits of the single calls."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device="cuda").manual_seed(len(shapes))
    Yd = [torch.randn(sh, generator=gen, device=dev) for sh in shapes]
    etas = [0.1 * mp.norm_l1q(Y, QNAME[q]) for Y in Yd]
    Xs = mp.bilevel_proj_batch(Yd, etas, q)
    for Y, eta, X in zip(Yd, etas, Xs):
        assert torch.equal(mp.bilevel_proj_stored(Y, eta, q), X)
    ref = orc.bilevel(Yd[0].cpu().numpy(), float(np.float32(etas[0])), q)
    np.testing.assert_allclose(Xs[0].cpu().numpy(), ref["X"], rtol=RTOL, atol=ATOL)


# Row lengths around the 16-byte pieces, the tiles (256 fp32, 512 16-bit columns) and the 16- and 8-column stripes;
# and of the map pass's forms (an eighth of the second tile, three eighths of a single one); heights around the rows a
# workgroup holds.  At most 128 KiB takes the one-kernel form (q = inf, 2).
RAGGED = [("f32", (5, 5)), ("f32", (7, 4)), ("f32", (100, 77)), ("f32", (300, 257)), ("f32", (129, 259)), ("f32", (1025, 511)),
          ("f32", (4096, 9)), ("f32", (2049, 31)), ("f32", (1, 70001)), ("f32", (40, 5003)), ("f32", (4097, 15)),
          ("f32", (8192, 7)), ("f32", (6000, 1001)), ("f32", (9000, 301)), ("f32", (33, 17)),
          ("f32", (700, 288)), ("f32", (700, 287)), ("f32", (700, 289)), ("bf16", (8, 4001)), ("bf16", (16, 2049)), ("f16", (16, 2047)), ("bf16", (1100, 191)), ("bf16", (1100, 193)), ("bf16", (700, 575)), ("f16", (700, 577)), ("f32", (1100, 4101)), ("bf16", (1100, 4101)), ("bf16", (9, 9)), ("bf16", (200, 65)), ("bf16", (700, 513)), ("bf16", (2047, 135)), ("bf16", (65, 4103)),
          ("f16", (40, 1031)), ("f16", (5000, 71)), ("f16", (300, 15))]


@pytest.mark.parametrize("q", ["inf", 1, 2])
@pytest.mark.parametrize("storage,shape", RAGGED)
def test_rows_of_any_length_and_address(mp, q, storage, shape):
    """Rows that start anywhere, read and written in 16-byte pieces: out of place, in place, with Y and X off their
    16-byte boundaries by different amounts."""
    Y = stored_input(shape, storage, 7)
    eta = eta_for(Y, q, 0.2)
    ref = orc.bilevel_stored(Y, eta, q, storage)
    for kw in ({}, {"inplace": True}, {"offset": 1, "x_offset": 3}, {"offset": 2, "inplace": True}):
        check_stored(run_stored(mp, Y, eta, q, storage, **kw), ref, q, storage)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("q", ["inf", 1, 2])
def test_batch_of_ragged_rows_gives_the_bits_of_the_single_calls(mp, q, storage):
    dev = torch.device("cuda:0")
    dt = getattr(torch, STORE_DTYPES[storage])
    shapes = [(100, 77), (300, 257), (2049, 31), (33, 17), (700, 1001), (64, 64), (3, 3), (40, 5003)]
    Yd = [torch.from_numpy(stored_input(sh, storage, i)).to(dev).to(dt) for i, sh in enumerate(shapes)]
    etas = [eta_for(Y.float().cpu().numpy(), q, 0.2) for Y in Yd]
    for Y, eta, X in zip(Yd, etas, mp.bilevel_proj_batch(Yd, etas, q)):
        assert torch.equal(mp.bilevel_proj_stored(Y, eta, q), X)


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("p", [1, 2, "inf"])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("more", [[], [(16, 2048), (64, 512)]])
def test_small_matrices_beside_larger_ones(mp, more, storage, p, inplace):
    """q = inf: ragged matrices of the one-kernel form in a batch with larger ones go through the launches of those, with the
    bits of their single calls in every output: up to 512 columns (a wavefront's search there), more, and rows shorter than a
    16-byte access; beside matrices of whole chunks they share the launch of those."""
    dev = torch.device("cuda:0")
    shapes = [(1200, 60), (272, 544), (47, 291), (16, 2047), (5, 5), (60, 517), (33, 17), (100, 3), (64, 511)] + more
    Yd = [torch.from_numpy(stored_input(sh, storage, i)).to(dev).to(getattr(torch, STORE_DTYPES[storage])) for i, sh in enumerate(shapes)]
    for frac in (0.05, 0.7, 1.5, 0.0):
        etas = [frac * float(Y.float().abs().amax(0).sum() if p == 1 else Y.float().abs().amax(0).norm() if p == 2 else Y.float().abs().max()) for Y in Yd]
        def outputs():
            return [torch.full((Y.shape[1],), -1.0, device=dev) for Y in Yd], [torch.full((Y.shape[1],), -1.0, device=dev) for Y in Yd], \
                   [torch.full((Y.shape[1],), 7, dtype=torch.uint8, device=dev) for Y in Yd], [mp.Workspace.for_call("l1inf", *Y.shape, device=dev) for Y in Yd]
        v, u, mask, ws = outputs()
        Xs = [Y.clone() if inplace else torch.empty_like(Y) for Y in Yd]
        mp.bilevel_proj_batch(Xs if inplace else Yd, etas, "inf", p=p, Xs=Xs, v_outs=v, u_outs=u, mask_outs=mask, workspaces=ws)
        v1, u1, mask1, ws1 = outputs()
        for i, (Y, X) in enumerate(zip(Yd, Xs)):
            assert torch.equal(mp.bilevel_proj_stored(Y, etas[i], "inf", p=p, v_out=v1[i], u_out=u1[i], mask_out=mask1[i], workspace=ws1[i]), X)
            assert torch.equal(v1[i], v[i]) and torch.equal(u1[i], u[i]) and torch.equal(mask1[i], mask[i])
            assert ws1[i].result() == ws[i].result()


# Batches by the values per thread of their tallest matrix (32, 64, 128) and, at 64, by whether there are more stripes than
# compute units; rows on whole 64-byte sectors, ragged ones, and both in one batch.
L11_BATCHES = [[(1024, 64), (512, 128)], [(1000, 77), (500, 333)], [(2048, 256), (1500, 64)], [(2000, 333), (1500, 70)],
               [(2048, 1024)] * 5, [(2000, 1003)] * 5, [(2048, 1024)] * 3 + [(2000, 1003)] * 3, [(1024, 64), (1000, 77), (2048, 64), (3000, 333)],
               # ... of 4097 to 16384 columns (the search ahead), of 4097 to 8192 rows (fp32: narrow stripes), and of every kind
               [(200, 5001), (100, 4100), (33, 16384)], [(256, 5120)] * 2, [(1500, 4101), (2048, 4112)], [(2100, 4101)], [(5000, 101), (8192, 33), (4097, 15)],
               [(6000, 48), (4097, 16)], [(5000, 101), (200, 5001), (1000, 77), (64, 64), (3, 3), (9000, 40), (40, 20000)]]


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("shapes", L11_BATCHES)
def test_l11_batches_give_the_bits_of_the_single_calls(mp, shapes, storage):
    dev = torch.device("cuda:0")
    Yh = [stored_input(sh, storage, i) for i, sh in enumerate(shapes)]
    Yd = [torch.from_numpy(Y).to(dev).to(getattr(torch, STORE_DTYPES[storage])) for Y in Yh]
    etas = [eta_for(Y, 1, 0.2) for Y in Yh]
    Xs = mp.bilevel_proj_batch(Yd, etas, 1)
    for Y, eta, X in zip(Yd, etas, Xs):
        assert torch.equal(mp.bilevel_proj_stored(Y, eta, 1), X)
    check_stored(run_stored(mp, Yh[-1], etas[-1], 1, storage), orc.bilevel_stored(Yh[-1], etas[-1], 1, storage), 1, storage)
    for p in (2, "inf"):
        for Y, eta, X in zip(Yd, etas, mp.bilevel_proj_batch(Yd, etas, 1, p=p)):
            assert torch.equal(mp.bilevel_proj_stored(Y, eta, 1, p=p), X)
    Zs = [Y.clone() for Y in Yd]
    masks = [torch.empty(Y.shape[1], dtype=torch.uint8, device=dev) for Y in Yd]
    mp.bilevel_proj_batch(Zs, etas, 1, Xs=Zs, mask_outs=masks)
    for Z, X, mask in zip(Zs, Xs, masks):
        assert torch.equal(Z, X) and torch.equal(mask.bool() | (X != 0).any(0), mask.bool())


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("n", [9000, 20000])
def test_l11_columns_with_next_to_no_radius_cost_no_further_sweeps(mp, n, storage):
    """Every third column keeps a share of 1e-4 of its norm: its root lies beyond all but one or two of its Gaussian entries.  The guess stays
    left of the largest, so one sweep more than for ordinary columns closes them (a first step, then a window)."""
    rng = np.random.default_rng(n)
    Y = rng.standard_normal((n, 600)).astype(np.float32)
    Y[:, ::3] *= 0.5
    Y = orc.round_to_storage(Y, storage)
    v = np.abs(Y.astype(np.float64)).sum(0)
    tau = 0.6 * v.max()
    sweeps = []
    for share in (0.5, 1e-4):
        w = np.ones(600, np.float32)
        w[::3] = v[::3] * (1.0 - share) / tau
        eta = float(np.float32((w * np.maximum(v - w * tau, 0.0)).sum()))
        got = run_weighted(mp, Y, eta, 1, storage, w)
        sweeps.append(got["res"]["inner_sweeps"])
        check_stored(got, orc.bilevel_stored(Y, eta, 1, storage, p=("w1", w)), 1, storage)
    assert 0 < sweeps[0] and sweeps[1] <= sweeps[0] + 1, sweeps


@pytest.mark.parametrize("family", ["gaussian", "cauchy", "misleading_head"])
def test_l11_grid_start_on_short_ragged_rows(mp, family):
    """The aggregate pass with the grid of thresholds, one element per access: rows shorter than a tile, 32M elements."""
    rng = np.random.default_rng([len(family), 81])
    Y = (rng.standard_cauchy if family == "cauchy" else rng.standard_normal)((262147, 129)).astype(np.float32)
    if family == "misleading_head":
        Y[:128] *= 1000.0
    eta = eta_for(Y, 1, 0.1)
    got = run_gpu(mp, Y, eta, 1)
    check_against_oracle(got, orc.bilevel(Y, eta, 1), 1)
    assert got["res"]["inner_sweeps"] >= 1


# Where a matrix that the registers hold is left to the sweeps: ragged rows, one workgroup per CU, X apart from Y, 32M elements.
@pytest.mark.parametrize("held,shape,inplace", [(False, (4096, 8193), False), (False, (2049, 16380), False), (True, (4096, 8192), False), (True, (2048, 16385), False),
                                                (True, (4095, 8193), False), (True, (4096, 8193), True)])
def test_l11_leaves_large_ragged_matrices_to_the_grid(mp, held, shape, inplace):
    """(Held, no lock-step sweep runs: the result record shows it.)  Both forms give the same projection."""
    Y = torch.randn(shape, generator=torch.Generator(device="cuda").manual_seed(5), device="cuda")
    eta = 0.1 * mp.norm_l1q(Y, "l11")
    X = Y.clone()
    ws = mp.Workspace.for_call("l11", *shape)
    mp.bilevel_proj_l11(X if inplace else Y, eta, X=X, workspace=ws)
    assert (ws.result()["inner_sweeps"] == 0) == held
    before = mp.set_l11_sweeps(4)
    try:
        Z = mp.bilevel_proj_l11(Y, eta)
    finally:
        mp.set_l11_sweeps(before)
    torch.testing.assert_close(X, Z, rtol=RTOL, atol=ATOL)
    assert abs(float(X.abs().sum(dtype=torch.float64)) - eta) <= 1e-5 * eta
    Xb = mp.bilevel_proj_batch([Y[:, :64].contiguous(), Y], [1.0, eta], 1)[1]
    if not inplace:
        assert torch.equal(Xb, X)


@pytest.mark.parametrize("kind", ["normal", "heavy", "tied"])
@pytest.mark.parametrize("storage", ["bf16", "f16"])
def test_l11_batches_of_plain_steps_give_the_bits_of_calls_with_windows(mp, storage, kind):
    """16-bit matrices of 1025 to 2048 rows: together more stripes than CUs, stepped without windows; each for itself fewer, with
    windows.  Entries of one scale, over twelve decimal orders (f16: eight), and on a grid of a few values."""
    rng = np.random.default_rng(len(kind))
    Yd, etas = [], []
    for n, m in ((1100, 2048), (2048, 2040), (1025, 3001)):
        Y = rng.standard_normal((n, m))
        if kind == "heavy":
            Y = np.sign(Y) * 10.0 ** rng.uniform(*((-8, 4) if storage == "bf16" else (-4, 4)), (n, m))
        elif kind == "tied":
            Y = np.round(3 * Y) / 4
        Y = orc.round_to_storage(Y.astype(np.float32), storage)
        Yd.append(torch.from_numpy(Y).cuda().to(getattr(torch, STORE_DTYPES[storage])))
        etas.append(eta_for(Y, 1, {"normal": 0.2, "heavy": 0.9, "tied": 0.02}[kind]))
    for Y, eta, X in zip(Yd, etas, mp.bilevel_proj_batch(Yd, etas, 1)):
        assert torch.equal(mp.bilevel_proj_stored(Y, eta, 1), X)
        Yh = Y.float().cpu().numpy()
        check_stored(run_stored(mp, Yh, eta, 1, storage), orc.bilevel_stored(Yh, eta, 1, storage), 1, storage)


@pytest.mark.parametrize("shape", [(200, 5001), (256, 5120), (5000, 101), (6000, 48), (1000, 77), (2048, 64), (9000, 40)])
def test_l11_batches_share_their_launches(mp, shape):
    """Six matrices take the launches of two, whatever form of the l1,1 kernels they go to (16 x (5000 x 101): 84 us, 650 one
    after another)."""
    def intervals(count):
        Yd = [torch.randn(shape, device="cuda") for _ in range(count)]
        with mp.KernelTrace(256) as trace:
            mp.bilevel_proj_batch(Yd, [1.0] * count, 1)
        torch.cuda.synchronize()
        return len(trace.durations_ms())
    assert intervals(6) == intervals(2)


@pytest.mark.parametrize("q", ["inf", 2])
@pytest.mark.parametrize("m", [4097, 6144, 6145, 8192, 8200, 14337, 16384])
def test_search_over_part_of_its_register_slots(mp, q, m):
    """The threshold search of 4097 to 16384 columns works through its slots in chunks of 2048 columns; many rounds
    (a radius that keeps a handful of columns) and few."""
    rng = np.random.default_rng(m)
    Y = rng.random((37, m), dtype=np.float32)
    for frac in (1e-5, 0.3):
        eta = eta_for(Y, q, frac)
        check_stored(run_stored(mp, Y, eta, q, "f32"), orc.bilevel_stored(Y, eta, q, "f32"), q, "f32")


def one_pass(mp, storage, shape, norms):
    """Whether a call on this GPU takes the one-pass kernel (the rule the library's dispatch asks)."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return mp.lib().mlproj_multilevel_one_pass({"f32": 0, "bf16": 1, "f16": 2}[storage], {"inf": 0, 1: 1, 2: 2}[norms[0]], *shape, cus) == 1


# Tensors of two inner levels that take the one-pass kernel: fibres of one chunk, of a ragged last chunk, of the most chunks
# (256); one fibre per slab and the most fibres; one slab, one slab per workgroup, several, a last workgroup with fewer; every
# layout of the kernel.
HM_CASES = [((1, 1, 4), [1, 1]), ((3, 5, 7), [2, 1]), ((256, 3, 9), [1, 1]), ((257, 2, 8), ["inf", 1]), ((1000, 20, 77), [1, 1]),
            ((2048, 2, 5), [1, 2]), ((200, 128, 130), [1, 1]), ((190, 60, 513), [1, "inf"]), ((40, 30, 64), [1, 1]), ((255, 256, 256), [1, 1]),
            ((255, 2048, 4), ["inf", 1]), ((128, 512, 30), [2, 2]), ((200, 128, 257), ["inf", 2]), ((200, 64, 1023), [1, 2]), ((256, 64, 1024), [2, 1])]
# ... and tensors that would fit it but where the chain is the faster.
HM_REFUSED = [((5, 2000, 30), [2, 2]), ((4, 64, 1024), [2, 1]), ((3, 33, 1001), ["inf", 2]), ((600, 300, 33), [2, 1]), ((9, 100, 500), ["inf", 1])]


@pytest.mark.parametrize("taken,shape,norms", [(True, *c) for c in HM_CASES] + [(False, *c) for c in HM_REFUSED])
def test_multilevel_in_one_pass(mp, taken, shape, norms):
    assert one_pass(mp, "f32", shape, norms) == taken
    rng = np.random.default_rng(list(shape) + [4])
    Y = rng.standard_normal(shape).astype(np.float32)
    Y *= np.power(10.0, rng.uniform(-1.0, 0.0, shape[0])).astype(np.float32)[:, None, None]
    nrm = nested_norm(Y, norms)
    for frac in (0.03, 0.4, 1.5, 0.0):
        eta = float(np.float32(frac * nrm))
        ref = orc.multilevel(Y, norms, eta)
        check_multi(run_multi(mp, Y, norms, eta), ref)
        Z = torch.from_numpy(Y).cuda()
        mp.multilevel_proj(Z, norms, eta, X=Z)
        np.testing.assert_allclose(Z.cpu().numpy(), ref["X"], rtol=RTOL, atol=ATOL)


@pytest.mark.parametrize("limit", [0, 1])
@pytest.mark.parametrize("shape,norms", [((256, 3, 40), [1, 1]), ((600, 7, 33), [2, 1]), ((130, 40, 500), ["inf", 1])])
def test_multilevel_in_one_pass_without_patience(mp, shape, norms, limit):
    """Every workgroup computes the slab norms it does not find posted itself, as on a GPU too busy to run all of
    them at once: the same result, in place too, and every kernel ends."""
    assert one_pass(mp, "f32", shape, norms)
    rng = np.random.default_rng(list(shape) + [limit])
    Y = rng.standard_normal(shape).astype(np.float32)
    eta = float(np.float32(0.2 * nested_norm(Y, norms)))
    ref = orc.multilevel(Y, norms, eta)
    before = mp.set_search_spin_limit(limit)
    try:
        check_multi(run_multi(mp, Y, norms, eta), ref)
        Z = torch.from_numpy(Y).cuda()
        mp.multilevel_proj(Z, norms, eta, X=Z)
        np.testing.assert_allclose(Z.cpu().numpy(), ref["X"], rtol=RTOL, atol=ATOL)
    finally:
        mp.set_search_spin_limit(before)


@pytest.mark.parametrize("inplace", [False, True])
def test_multilevel_in_one_pass_on_several_streams(mp, inplace):
    """Four streams at once, each with a tensor whose workgroups would fill the chip alone: workgroups of one call wait for
    some that cannot start, and divide their shares among them.  The bits of a call that has the GPU to itself."""
    shape, norms = (256, 128, 512), [1, 1]
    assert one_pass(mp, "f32", shape, norms)
    gen = torch.Generator(device="cuda").manual_seed(11)
    Ys = [torch.randn(shape, generator=gen, device="cuda") for _ in range(4)]
    etas = [0.2 * float(Y.abs().sum()) for Y in Ys]
    alone = [mp.multilevel_proj(Y, norms, eta) for Y, eta in zip(Ys, etas)]
    Xs = [Y.clone() if inplace else torch.empty_like(Y) for Y in Ys]
    spaces = [mp.Workspace(mp.multilevel_workspace_bytes(shape)) for _ in Ys]
    streams = [torch.cuda.Stream() for _ in Ys]
    torch.cuda.synchronize()
    for _ in range(3):
        for Y, X, eta, ws, stream in zip(Ys, Xs, etas, spaces, streams):
            if inplace:
                with torch.cuda.stream(stream):
                    X.copy_(Y)
            mp.multilevel_proj(X if inplace else Y, norms, eta, X=X, workspace=ws, stream=stream)
    torch.cuda.synchronize()
    for X, A in zip(Xs, alone):
        assert torch.equal(X, A)


@pytest.mark.parametrize("storage", ["bf16", "f16"])
@pytest.mark.parametrize("taken,shape,norms", [(True, (100, 16, 65), [1, 1]), (True, (30, 40, 128), [2, 2]), (False, (300, 5, 520), ["inf", 1]), (True, (64, 64, 64), [1, 1]),
                                               (True, (256, 70, 256), [2, 1]), (True, (200, 30, 1001), ["inf", 1]), (True, (200, 100, 255), [1, 1]), (True, (200, 500, 30), [2, 2])])
def test_multilevel_in_one_pass_on_16_bit_storage(mp, storage, taken, shape, norms):
    assert one_pass(mp, storage, shape, norms) == taken
    dt = getattr(torch, STORE_DTYPES[storage])
    Y = orc.round_to_storage(np.random.default_rng(list(shape)).standard_normal(shape).astype(np.float32), storage)
    eta = float(np.float32(0.3 * nested_norm(Y, norms)))
    Yd = torch.from_numpy(Y).cuda().to(dt)
    X = mp.multilevel_proj_stored(Yd, norms, eta)
    x = orc.multilevel_stored(Y, norms, eta, storage)["X32"].astype(np.float64)
    tol = RTOL * np.abs(x) + ATOL
    got = X.float().cpu().numpy()
    assert np.all(got >= orc.round_to_storage((x - tol).astype(np.float32), storage))
    assert np.all(got <= orc.round_to_storage((x + tol).astype(np.float32), storage))
    assert torch.equal(mp.multilevel_proj_stored(Yd, norms, eta, X=Yd), X)


# Fibres whose entries are equal or nearly so, at radii far below an fp32 unit of them: every layout of the one-pass kernel (4 lanes; 16 with 4, 8 and
# 16 chunks each), ragged last chunks, and the chain.
FLAT = [("f32", True, (20, 16, 100)), ("f32", True, (20, 16, 129)), ("f32", True, (20, 8, 256)), ("f32", True, (20, 8, 511)), ("f32", True, (200, 30, 1001)),
        ("f32", True, (256, 256, 256)), ("f32", True, (256, 64, 1024)), ("f32", False, (3, 4, 1500)), ("bf16", True, (20, 30, 512)), ("bf16", True, (200, 30, 1001)),
        ("f16", True, (20, 8, 512)), ("f16", True, (250, 32, 1024)), ("f16", False, (3, 4, 2000))]


def assert_near(X, want, tol, storage):
    """Every entry within tol of the wanted value, as the storage type rounds the ends of that range."""
    got = X.float().cpu().numpy()
    assert np.all(got >= orc.round_to_storage((want - tol).astype(np.float32), storage))
    assert np.all(got <= orc.round_to_storage((want + tol).astype(np.float32), storage))


@pytest.mark.parametrize("storage,taken,shape", FLAT)
def test_multilevel_l1_of_constant_fibres(mp, storage, taken, shape):
    """All magnitudes a: every entry keeps eta / (number of entries) and its sign, whatever the radius.  A threshold is a difference of
    64-bit sums (at most 128 additions to one, three levels): 512 units of 2^-53 relative to the norm, 512 x 2^-53 / share relative to the result."""
    assert one_pass(mp, storage, shape, [1, 1]) == taken
    gen = torch.Generator(device="cuda").manual_seed(shape[2])
    signs = torch.randint(0, 2, shape, generator=gen, device="cuda").mul_(2).sub_(1)
    for a in (1.0, 0.703125, 24576.0):
        Y = (signs if a != 1.0 else torch.ones_like(signs)).to(getattr(torch, STORE_DTYPES[storage])) * a
        for share in (0.25, 1e-3, 2e-8, 1e-10):
            eta = float(np.float32(share * a * Y.numel()))
            want = Y.sign().float().cpu().numpy().astype(np.float64) * (eta / Y.numel())
            tol = (2.0 ** -22 + 512 * 2.0 ** -53 / share) * (eta / Y.numel())
            assert_near(mp.multilevel_proj_stored(Y, [1, 1], eta), want, tol, storage)


@pytest.mark.parametrize("kind", ["tied", "close", "heavy"])
@pytest.mark.parametrize("storage,taken,shape", [c for c in FLAT if c[2][0] <= 20])
def test_multilevel_l1_of_fibres_hard_to_search(mp, storage, taken, shape, kind):
    """Two values a few storage units apart, values in steps of one unit, and a few entries of a Cauchy sample far above the rest, at small radii, against
    the oracle; the bound as for constant fibres, absolute: a fibre whose other entries are dropped has the norm's rounding in one of them."""
    assert one_pass(mp, storage, shape, [1, 1]) == taken
    rng = np.random.default_rng(list(shape) + [len(kind)])
    unit = {"f32": 2.0 ** -23, "bf16": 2.0 ** -7, "f16": 2.0 ** -10}[storage]
    if kind == "tied":
        Y = 1.0 + 4 * unit * rng.integers(0, 2, shape)
    elif kind == "close":
        Y = 1.0 + unit * rng.integers(0, 9, shape)
    else:
        Y = np.clip(np.abs(rng.standard_cauchy(shape)), 1e-3, 6e4)
    Y = orc.round_to_storage((Y * rng.choice([-1.0, 1.0], shape)).astype(np.float32), storage)
    Yd = torch.from_numpy(Y).cuda().to(getattr(torch, STORE_DTYPES[storage]))
    for share in (0.02, 1e-4, 1e-7):
        eta = float(np.float32(share * nested_norm(Y, [1, 1])))
        ref = orc.multilevel(Y, [1, 1], eta)
        want = ref["U"][0]
        assert_near(mp.multilevel_proj_stored(Yd, [1, 1], eta), want, 2.0 ** -22 * np.abs(want) + 512 * 2.0 ** -53 * ref["w"].max(), storage)


def test_multilevel_in_one_pass_in_a_graph(mp):
    """Replays of a captured call, eager calls on other contents between them."""
    assert one_pass(mp, "f32", (200, 40, 60), [1, 1])
    gen = torch.Generator(device="cuda").manual_seed(3)
    Y = torch.randn((200, 40, 60), generator=gen, device="cuda")
    X, E = torch.empty_like(Y), torch.empty_like(Y)
    ws = mp.Workspace(mp.multilevel_workspace_bytes(tuple(Y.shape)))
    eta = 0.2 * float(Y.abs().sum())
    mp.multilevel_proj(Y, [1, 1], eta, X=X, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mp.multilevel_proj(Y, [1, 1], eta, X=X, workspace=ws)
    for _ in range(3):
        Y.copy_(torch.randn(Y.shape, generator=gen, device="cuda"))
        mp.multilevel_proj(Y, [1, 1], eta, X=E)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(X, E)
