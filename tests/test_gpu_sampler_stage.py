"""The sampler's tree is the same whether a step's weights are staged in LDS (many prefixes possible)
or read from cache: the kernel follows the bound on distinct prefixes that the caller gives."""
import numpy as np
import pytest
import torch

from oracle import sampler as osamp
from oracle import slater_condon as osc
from paper_2506_07430_amd import elocal, synth
from tests.gpu_common import make_ham, theta_for, words_from_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,na,nb,widths", [(10, 5, 5, (32,)), (13, 6, 6, (96, 128)), (13, 7, 5, (128, 64)),
                                            (15, 7, 8, (128,)), (18, 9, 9, (256, 256)), (16, 8, 7, (64, 64, 64)),
                                            (33, 3, 2, (128, 128)), (40, 14, 14, (160, 160))])
def test_tree_of_many_draws(n, na, nb, widths):
    p = synth.random_problem(n, na, nb, widths, seed=880 + n, n_chol=2, decay=3.0, samples=1)
    theta = 8.0 * p.theta   # a peaked distribution: far fewer distinct samples than draws
    ham, (th_dev, th) = make_ham(p), theta_for(theta, elocal.FP64)
    ans = elocal.Ansatz(widths, th_dev, elocal.FP64)
    x, c = ham.sample(ans, 50000, 880 + na, max_unique=60000)   # staged from 32768 possible prefixes on
    print(f"n={n} {na}a+{nb}b {widths}: {x.shape[0]} distinct", flush=True)
    y, d = ham.sample(ans, 50000, 880 + na, max_unique=32000)
    assert torch.equal(x, y) and torch.equal(c, d)
    occ, cnt = osamp.bas(th, n, na, nb, widths, 50000, 880 + na)
    assert np.array_equal(words_from_dev(x), osc.pack(occ)) and np.array_equal(c.cpu().numpy(), cnt)
