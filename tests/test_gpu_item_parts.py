"""Local energies of small batches, whose work items are run in parts, equal bit for bit those of
whole items: every precision of the plain fused kernels (one narrow layer, layers of different
widths, one and two words per determinant), lists of less than one group, of a ragged last
group and of several items, in `eval` and side by side in a launch over several systems."""
import pytest
import torch

from paper_2506_07430_amd import elocal, synth
from tests.gpu_common import make_ham, theta_for, words_to_dev

pytestmark = pytest.mark.gpu

SHAPES = [
    # n, n_alpha, n_beta, widths, samples
    (6, 1, 2, (32,), 5),
    (8, 4, 4, (32,), 37),
    (12, 6, 5, (64, 128), 9),
    (14, 7, 7, (32, 32), 3),
    (33, 3, 2, (32,), 2),
]


@pytest.mark.parametrize("precision", [elocal.BF16, elocal.BF16X3, elocal.FP64])
@pytest.mark.parametrize("n,na,nb,widths,samples", SHAPES)
def test_parts_equal_whole_items(n, na, nb, widths, samples, precision):
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    torch.cuda.set_device(0)
    p = synth.random_problem(n, na, nb, widths, seed=910 + n, n_chol=3, decay=4.0, samples=samples)
    ham = make_ham(p)
    ans = elocal.Ansatz(widths, theta_for(p.theta, precision)[0], precision)
    x = words_to_dev(p.x)
    parts, _ = ham.eval(ans, x)
    several, _ = elocal.MultiEval()([ham, ham], [ans, ans], [x, x])
    ham.tune(groups=16 if precision == elocal.FP64 else 8)   # the whole items of large batches
    whole, _ = ham.eval(ans, x)
    ham.tune()
    print(f"n={n} {na}a+{nb}b {widths} {samples} samples precision={precision}", flush=True)
    assert torch.equal(parts, whole)
    for e in several:
        assert torch.equal(e, whole)
