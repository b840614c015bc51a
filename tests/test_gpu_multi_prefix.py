"""Several systems whose shared evaluation runs in one launch of a width class wider than their
own, beside systems that take the plain kernels: every system exactly as by itself, and one
against the oracle."""
import numpy as np
import pytest
import torch

from oracle import energy as oen
from paper_2506_07430_amd import elocal, synth
from tests.gpu_common import ansatz_samples, make_ham, theta_for, words_to_dev

pytestmark = pytest.mark.gpu

# n, n_alpha, n_beta, widths; the shared evaluation from the second entry of each list on
BF16 = [(8, 4, 4, (64, 64)), (21, 10, 11, (64, 64)), (20, 10, 9, (128,)), (19, 9, 10, (96, 96)), (16, 8, 8, (256,)),
        (17, 8, 8, (192, 192))]
FP64 = [(8, 4, 4, (64, 64)), (12, 6, 6, (64, 64)), (12, 6, 6, (128, 128)), (13, 6, 7, (96,)), (16, 8, 7, (256,)),
        (17, 8, 8, (224, 224))]


@pytest.mark.parametrize("pick", [(1,), (1, 1), (2, 3), (4, 5), (0, 1, 2), (5, 4, 3, 2, 1, 0), (1, 4)])
@pytest.mark.parametrize("precision", [elocal.BF16, elocal.FP64])
def test_systems_of_different_width_classes(precision, pick):
    shapes = BF16 if precision == elocal.BF16 else FP64
    probs, hams, ans, xs = [], [], [], []
    for i, k in enumerate(pick):
        n, na, nb, widths = shapes[k]
        p = synth.random_problem(n, na, nb, widths, seed=850 + k, n_chol=4, decay=5.0, samples=1)
        th_dev, th = theta_for(p.theta, precision)
        x = ansatz_samples(p, 2 + 3 * i, seed=860 + i, theta=th)
        probs.append((p, x, th))
        hams.append(make_ham(p))
        ans.append(elocal.Ansatz(widths, th_dev, precision))
        xs.append(words_to_dev(x))
    multi, lps = elocal.MultiEval()(hams, ans, xs, want_logpsi=True)
    for i, (h, a, x) in enumerate(zip(hams, ans, xs)):
        single, lp = h.eval(a, x)
        assert torch.equal(multi[i], single) and torch.equal(lps[i], lp), f"system {i} of {pick}"
    p, x, th = probs[0]
    s = p.system
    ref = oen.local_energies(p.h1e, p.eri, s.n, s.n_alpha, s.n_beta, s.widths, th, x)
    e = multi[0].cpu().numpy()
    err = np.max(np.abs(e[:, 0] + 1j * e[:, 1] - ref))
    assert err <= (1e-10 * np.max(np.abs(ref)) if precision == elocal.FP64 else 1e-5)
