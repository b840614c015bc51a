"""Evaluations with less workspace than a launch could use: fewer blocks, batches in parts, whole
items in place of parts of items. Local energies and log psi are the same bit for bit."""
import ctypes

import pytest
import torch

from paper_2506_07430_amd import elocal, synth
from tests.gpu_common import make_ham, theta_for, words_to_dev

pytestmark = pytest.mark.gpu


def problem(n, na, nb, widths, precision, samples, seed):
    p = synth.random_problem(n, na, nb, widths, seed=seed, n_chol=2, decay=5.0, samples=min(samples, 400))
    x = words_to_dev(p.x)
    x = x.repeat((samples + x.shape[0] - 1) // x.shape[0], 1)[:samples].contiguous()
    return p, make_ham(p), elocal.Ansatz(widths, theta_for(p.theta, precision)[0], precision), x


def abi_eval(ham, ans, x, ws_bytes):
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    e = torch.empty((x.shape[0], 2), dtype=torch.float64, device="cuda")
    lp = torch.empty_like(e)
    st = elocal.lib().elocal_eval(ham._h, elocal._stream(None), ans.ref(), x.data_ptr(), x.shape[0], ws.data_ptr(),
                                  ws_bytes, e.data_ptr(), lp.data_ptr())
    return st, e, lp


@pytest.mark.parametrize("n,na,nb,widths,precision,samples", [
    (60, 26, 26, (256, 256, 256), elocal.BF16, 700),   # two words per determinant
    (24, 12, 12, (128, 128), elocal.BF16, 0),          # 0: the largest batch that the scratch takes
    (12, 6, 6, (64, 64), elocal.FP64, 0),
    (24, 12, 12, (64, 64), elocal.FP64, 0),
])
def test_batches_in_parts_give_the_same_energies(n, na, nb, widths, precision, samples):
    p, ham, ans, _ = problem(n, na, nb, widths, precision, 1, 830 + n)
    scratch = elocal.NOALLOC_SCRATCH_MIB << 20
    if samples == 0:
        samples, hi = 1, 1 << 22
        while samples < hi:
            mid = (samples + hi + 1) // 2
            if ham.workspace_bytes(elocal.OP_EVAL, mid, ans) <= scratch:
                samples = mid
            else:
                hi = mid - 1
    p, ham, ans, x = problem(n, na, nb, widths, precision, samples, 830 + n)
    print(f"n={n} {widths} precision={precision}: {samples} samples", flush=True)
    want, want_lp = ham.eval(ans, x)
    ham.timing()
    lp = torch.empty_like(want_lp)
    got, _ = ham.eval_noalloc(ans, x, logpsi=lp)
    launches = ham.kernel_time()[1]
    assert launches > 1
    assert torch.equal(got, want) and torch.equal(lp, want_lp)
    need = ham.workspace_bytes(elocal.OP_EVAL, samples, ans)
    st, e, lp = abi_eval(ham, ans, x, need)
    assert st == 0 and torch.equal(e, want) and torch.equal(lp, want_lp)
    st, _, _ = abi_eval(ham, ans, x, need - 1)
    assert st == 3


def test_pauli_route_with_room_for_whole_items_only():
    p, ham, ans, x = problem(8, 4, 4, (64, 64), elocal.BF16, 60, 841)
    ham.pauli_build()
    L = elocal.lib()
    full = int(L.elocal_pauli_workspace_bytes(ham._h, ans.ref(), x.shape[0]))
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")

    def run(nbytes):
        e = torch.full((x.shape[0], 2), float("nan"), dtype=torch.float64, device="cuda")
        st = L.elocal_eval_pauli(ham._h, elocal._stream(None), ans.ref(), ctypes.c_void_p(x.data_ptr()), x.shape[0],
                                 ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(nbytes), ctypes.c_void_p(e.data_ptr()))
        return st, e

    st, want = run(full)
    assert st == 0
    lo, hi = 1, full   # the least that is taken
    while lo < hi:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if run(mid)[0] == 0 else (mid + 1, hi)
    st, got = run(lo)
    print(f"workspace {full} -> {lo} bytes", flush=True)
    assert st == 0 and lo < full and torch.equal(got, want)
