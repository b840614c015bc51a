"""H on sector vectors without room for the tables of the matrix products: from row lists, as in
small sectors, and the same to rounding."""
import numpy as np
import pytest
import torch

from paper_2506_07430_amd import elocal, synth
from tests.gpu_common import make_ham

pytestmark = pytest.mark.gpu


def test_row_lists_where_the_tables_do_not_fit(monkeypatch):
    p = synth.random_problem(10, 5, 5, (32,), seed=870, n_chol=4, samples=1)   # 63504 rows of 876
    ham = make_ham(p)
    dim = ham.sector_dim
    v = torch.randn(dim, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    want, want_d = ham.sector_apply(v, dots=True)
    mu = ham.kpm_moments(v / v.norm(), 12, 60.0, 0.0)
    L = elocal.lib()
    full = [int(L.elocal_sector_workspace_bytes(ham._h, k)) for k in (0, 1)]
    assert full[0] > 4 * 8 * dim
    empty, asked = torch.empty, []

    def small(*size, **kw):
        if kw.get("dtype") is torch.uint8:
            asked.append(size[0])
            if size[0] in full:
                raise torch.cuda.OutOfMemoryError("no room for the tables")
        return empty(*size, **kw)

    monkeypatch.setattr(torch, "empty", small)
    got, got_d = ham.sector_apply(v, dots=True)
    mu2 = ham.kpm_moments(v / v.norm(), 12, 60.0, 0.0)
    monkeypatch.undo()
    assert asked[0] == full[0] and asked[1] <= (128 << 10) + 256 and len(asked) == 4
    # sums of about 1e3 products of order |H| |v| in two orders
    scale = want.abs().max().item()
    assert (got - want).abs().max().item() <= 1e-12 * scale
    assert np.allclose(got_d.cpu().numpy(), want_d.cpu().numpy(), rtol=1e-11)
    assert (mu - mu2).abs().max().item() <= 1e-12

    def status(nbytes):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        y = torch.empty_like(v)
        return L.elocal_sector_apply(ham._h, elocal._stream(None), 1.0, v.data_ptr(), 0.0, None, 0.0, y.data_ptr(),
                                     ws.data_ptr(), nbytes, None)

    assert status(128 << 10) == 0 and status(1024) == 3


@pytest.mark.parametrize("n,na,nb", [(11, 9, 5), (11, 5, 2), (11, 2, 5)])
def test_products_of_nearly_full_and_nearly_empty_shells(n, na, nb):
    """The shapes of few strings of one spin at the sizes from which products are taken, against row
    lists (1e-12 of the largest entry: sums of about 1e3 products in two orders)."""
    ham = make_ham(synth.random_problem(n, na, nb, (32,), seed=880 + na, n_chol=4, samples=1))
    v = torch.randn(ham.sector_dim, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    L = elocal.lib()
    assert int(L.elocal_sector_workspace_bytes(ham._h, 0)) > 4 * 8 * ham.sector_dim
    want = ham.sector_apply(v)
    ws, y = torch.empty(128 << 10, dtype=torch.uint8, device="cuda"), torch.empty_like(v)
    assert L.elocal_sector_apply(ham._h, elocal._stream(None), 1.0, v.data_ptr(), 0.0, None, 0.0, y.data_ptr(),
                                 ws.data_ptr(), ws.numel(), None) == 0
    assert (y - want).abs().max().item() <= 1e-12 * want.abs().max().item()
