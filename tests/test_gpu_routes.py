"""The routes a call can take by its sizes and alignment, each at the sizes where it can go wrong, against the oracle
(the bars of test_gpu_parity.py) or bit for bit against the route that computes the same sums in the same order."""
import numpy as np
import pytest

from oracle import mlproj_oracle as orc
from test_gpu_parity import ATOL, QNAME, RTOL, STORE_DTYPES, check_stored, eta_for, stored_input, mp  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", ["inf", 2])
@pytest.mark.parametrize("shapes", [[(1024, 1024)] * 16, [(20000, 64)] + [(100, 16384)] * 12, [(4099, 4097)], [(17, 300), (16, 5000)]])
def test_batch_map_grid_is_planned_for_the_launch(mp, q, shapes):
    """Batches whose map workgroups take several row blocks each, a tall matrix beside wide ones (more column tiles
    than workgroups planned for), one matrix alone, and ragged last blocks: the bits of the single calls."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device="cuda").manual_seed(len(shapes))
    Yd = [torch.randn(sh, generator=gen, device=dev) for sh in shapes]
    etas = [0.1 * mp.norm_l1q(Y, QNAME[q]) for Y in Yd]
    Xs = mp.bilevel_proj_batch(Yd, etas, q)
    for Y, eta, X in zip(Yd, etas, Xs):
        assert torch.equal(mp.bilevel_proj_stored(Y, eta, q), X)
    ref = orc.bilevel(Yd[0].cpu().numpy(), float(np.float32(etas[0])), q)
    np.testing.assert_allclose(Xs[0].cpu().numpy(), ref["X"], rtol=RTOL, atol=ATOL)
