"""H on full-sector vectors by matrix products over strings, at the edges of its range.

Rows of H v against the oracle, within 1e-12 of the largest |(H v)_r| (FP64, another order of
the sum), for closed, open and nearly empty or full shells of either spin, string counts that
are no multiple of a tile, more than one string per thread, and several passes over the
excitations of a string; the combination ch H v + cv v + cz z and its dot products; and the
recursion's moments against repeated products.
"""
import numpy as np
import pytest
import torch

from oracle import kpm as okpm
from paper_2506_07430_amd import synth
from tests.gpu_common import make_ham

pytestmark = pytest.mark.gpu

# n, n_alpha, n_beta: near the fewest entries of this route; shells empty or full but one;
# odd counts; K = 56 excitations of 48 a pass; 1140 strings of the spin that is gathered
SHAPES = [(9, 4, 4), (10, 8, 5), (10, 5, 2), (11, 4, 7), (12, 1, 6), (12, 11, 6), (14, 7, 3), (20, 2, 3)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    torch.cuda.set_device(0)


@pytest.mark.parametrize("n,na,nb", SHAPES)
def test_rows_match_oracle(n, na, nb):
    p = synth.random_problem(n, na, nb, (32,), seed=170 + n + na, n_chol=4, decay=4.0, samples=1)
    ham = make_ham(p)
    dim = ham.sector_dim
    print(f"n={n} {na}a+{nb}b: {dim} rows", flush=True)
    rng = np.random.default_rng(n * 100 + na)
    v, z = rng.standard_normal(dim), rng.standard_normal(dim)
    dv, dz = torch.tensor(v).cuda(), torch.tensor(z).cuda()
    y, d = ham.sector_apply(dv, ch=0.7, cv=-0.3, z=dz, cz=-1.0, dots=True)
    again = ham.sector_apply(dv, ch=0.7, cv=-0.3, z=dz, cz=-1.0)
    assert torch.equal(y, again)
    hv = ham.sector_apply(dv).cpu().numpy()
    scale = np.max(np.abs(hv))
    for r in [0, dim - 1] + list(rng.integers(0, dim, 4)):
        assert abs(hv[r] - okpm.row_apply(p.h1e, p.eri, n, na, nb, int(r), v)) <= 1e-12 * scale, f"row {r}"
    y, d = y.cpu().numpy(), d.cpu().numpy()
    assert np.max(np.abs(y - (0.7 * hv - 0.3 * v - z))) <= 1e-12 * scale
    assert abs(d[0] - y @ y) <= 1e-12 * (y @ y)
    assert abs(d[1] - y @ v) <= 1e-12 * (np.abs(y) @ np.abs(v))


def test_moments_match_repeated_products():
    n, na, nb = 9, 4, 5
    p = synth.random_problem(n, na, nb, (32,), seed=179, n_chol=4, decay=4.0, samples=1)
    ham = make_ham(p)
    v = torch.tensor(np.random.default_rng(9).standard_normal(ham.sector_dim)).cuda()
    a, b = 400.0, -20.0
    mu = ham.kpm_moments(v, 9, a, b).cpu().numpy()
    t = [v, ham.sector_apply(v, ch=1 / a, cv=-b / a)]
    while len(t) < 9:
        t.append(ham.sector_apply(t[-1], ch=2 / a, cv=-2 * b / a, z=t[-2], cz=-1.0))
    ref = np.array([float(v @ x) for x in t])
    assert np.max(np.abs(mu - ref)) <= 1e-11 * ref[0]
