"""Prefix-shared evaluation at the edges of the range that it is used in: the shortest lists of
each network width and precision, every number of 32-unit blocks, one to four hidden layers, one
and two words per determinant, and 64 orbitals. (That these systems take it, and those with
fewer entries per pair of spin-orbitals do not, is checked on the host in test_host_plan.py.)

Tolerances as everywhere: 1e-5 Ha in BF16 mode, 1e-10 relative in FP64.
"""
import numpy as np
import pytest
import torch

from oracle import energy as oen
from paper_2506_07430_amd import elocal, synth
from tests.gpu_common import ansatz_samples, make_ham, theta_for, words_to_dev

pytestmark = pytest.mark.gpu

SHAPES = [
    # precision, n, n_alpha, n_beta, widths, samples
    (elocal.BF16, 21, 10, 11, (64,), 3),
    (elocal.BF16, 22, 11, 11, (64, 64, 64, 64), 2),
    (elocal.BF16, 19, 9, 10, (96, 96), 3),
    (elocal.BF16, 20, 10, 9, (128, 128), 3),
    (elocal.BF16, 24, 8, 6, (128,), 2),
    (elocal.BF16, 16, 8, 8, (256,), 4),
    (elocal.BF16, 18, 9, 9, (160, 160), 3),
    (elocal.BF16, 17, 8, 8, (192, 192, 192), 2),
    (elocal.BF16, 18, 9, 9, (224, 224), 2),
    (elocal.BF16, 33, 16, 17, (128, 128), 1),
    (elocal.BF16, 33, 11, 9, (256, 256), 1),
    (elocal.FP64, 11, 5, 6, (64,), 9),
    (elocal.FP64, 12, 6, 6, (64, 64, 64, 64), 5),
    (elocal.FP64, 12, 5, 5, (96, 96), 5),
    (elocal.FP64, 13, 6, 7, (128, 128), 4),
    (elocal.FP64, 16, 8, 7, (160,), 3),
    (elocal.FP64, 17, 8, 8, (192, 192, 192), 2),
    (elocal.FP64, 18, 9, 9, (224, 224), 2),
    (elocal.FP64, 20, 10, 9, (256, 256), 1),
    (elocal.FP64, 33, 16, 17, (64, 64), 1),
    (elocal.FP64, 33, 11, 9, (128,), 1),
]


@pytest.mark.parametrize("precision,n,na,nb,widths,samples", SHAPES)
def test_local_energies_match_oracle(precision, n, na, nb, widths, samples):
    p = synth.random_problem(n, na, nb, widths, seed=760 + n + len(widths), n_chol=4, decay=5.0, samples=samples)
    th_dev, th = theta_for(p.theta, precision)
    x = ansatz_samples(p, samples, 761, th)
    e = make_ham(p).eval(elocal.Ansatz(widths, th_dev, precision), words_to_dev(x))[0].cpu().numpy()
    ref = oen.local_energies(p.h1e, p.eri, n, na, nb, widths, th, x)
    err = np.max(np.abs(e[:, 0] + 1j * e[:, 1] - ref))
    print(f"n={n} {na}a+{nb}b {widths} {len(x)} samples precision={precision}: max|dE_loc|={err:.2e}", flush=True)
    assert err <= (1e-10 * np.max(np.abs(ref)) if precision == elocal.FP64 else 1e-5)


@pytest.mark.parametrize("widths", [(64, 64), (256, 256, 256)])
def test_64_orbitals_agree_across_precisions(widths):
    """1.1 million entries: the shared BF16 and FP64 evaluations against the three-term BF16 mode,
    which runs every entry by itself."""
    n, na, nb = 64, 21, 19
    p = synth.random_problem(n, na, nb, widths, seed=790, n_chol=4, decay=5.0, samples=2)
    th_dev, th = theta_for(p.theta, elocal.BF16)
    x = words_to_dev(ansatz_samples(p, 2, 791, th))
    ham = make_ham(p)
    whole = ham.eval(elocal.Ansatz(widths, th_dev, elocal.BF16X3), x)[0]
    for precision, t in ((elocal.BF16, th_dev), (elocal.FP64, torch.from_numpy(th).cuda())):
        err = (ham.eval(elocal.Ansatz(widths, t, precision), x)[0] - whole).abs().max().item()
        print(f"{widths} precision={precision}: max|dE_loc|={err:.2e}", flush=True)
        assert err <= 1e-5


@pytest.mark.parametrize("precision", [elocal.BF16, elocal.BF16X3, elocal.FP64])
def test_64_orbitals_few_electrons_match_oracle(precision):
    """2 + 3 electrons, 64x2, on samples of the ansatz itself, where the bound of 1e-5 Ha holds."""
    n, na, nb, widths = 64, 2, 3, (64, 64)
    p = synth.random_problem(n, na, nb, widths, seed=766, n_chol=4, decay=5.0, samples=1)
    th_dev, th = theta_for(p.theta, precision)
    x = ansatz_samples(p, 4, 767, th)
    e = make_ham(p).eval(elocal.Ansatz(widths, th_dev, precision), words_to_dev(x))[0].cpu().numpy()
    ref = oen.local_energies(p.h1e, p.eri, n, na, nb, widths, th, x)
    err = np.max(np.abs(e[:, 0] + 1j * e[:, 1] - ref))
    print(f"precision={precision}: max|dE_loc|={err:.2e}", flush=True)
    assert err <= (1e-10 * np.max(np.abs(ref)) if precision == elocal.FP64 else 1e-5)


@pytest.mark.parametrize("n,na,nb,widths", [(22, 11, 11, (64,)), (24, 11, 12, (96, 96)), (34, 12, 11, (128,)),
                                            (40, 14, 13, (64, 64))])
def test_parts_of_segments_give_the_same_bits(n, na, nb, widths):
    """Segments are cut into parts by the batch and the network: whatever the cut, a sample's
    energy is the same bit for bit (1, 5 and 20 samples against all 48)."""
    p = synth.random_problem(n, na, nb, widths, seed=795 + n, n_chol=4, decay=5.0, samples=48)
    th_dev, th = theta_for(p.theta, elocal.BF16)
    x = words_to_dev(ansatz_samples(p, 48, 796, th))
    ham, ans = make_ham(p), elocal.Ansatz(widths, th_dev, elocal.BF16)
    whole = ham.eval(ans, x)[0].clone()
    for b in (1, 5, 20):
        assert torch.equal(ham.eval(ans, x[:b].contiguous())[0], whole[:b]), b
