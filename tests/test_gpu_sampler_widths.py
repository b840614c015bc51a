"""The sampler's conditionals over networks whose weights are staged in LDS, or are not.

Distinct samples, order and counts equal the oracle's tree: one to three hidden layers, widths
of one to sixteen 16-unit blocks (with 256 the wide steps do not fit), layers of different
widths (not updated in place), input counts that are no multiple of a chunk of four k-steps,
and one and two words per determinant.
"""
import numpy as np
import pytest
import torch

from oracle import sampler as osamp
from oracle import slater_condon as osc
from paper_2506_07430_amd import elocal, synth
from tests.gpu_common import make_ham, theta_for, words_from_dev

pytestmark = pytest.mark.gpu

SHAPES = [
    # n, n_alpha, n_beta, widths
    (5, 2, 3, (32,)),
    (10, 5, 4, (64, 64, 64)),
    (13, 6, 6, (96, 128)),
    (13, 7, 5, (128, 64)),
    (15, 7, 8, (128,)),
    (18, 9, 9, (256, 256)),
    (33, 3, 2, (128, 128)),
    (40, 2, 2, (160, 160)),
]


@pytest.mark.parametrize("n,na,nb,widths", SHAPES)
def test_tree_equals_oracle(n, na, nb, widths):
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    torch.cuda.set_device(0)
    p = synth.random_problem(n, na, nb, widths, seed=810 + n, n_chol=2, decay=3.0, samples=1)
    ham = make_ham(p)
    th_dev, th = theta_for(p.theta, elocal.FP64)
    x, c = ham.sample(elocal.Ansatz(widths, th_dev, elocal.FP64), 3000, 810 + na, max_unique=4000)
    occ, cnt = osamp.bas(th, n, na, nb, widths, 3000, 810 + na)
    print(f"n={n} {na}a+{nb}b {widths}: {x.shape[0]} distinct (oracle {occ.shape[0]})", flush=True)
    assert np.array_equal(words_from_dev(x), osc.pack(occ))
    assert np.array_equal(c.cpu().numpy(), cnt)
