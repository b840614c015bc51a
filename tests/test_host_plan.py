"""Launch planning on the host, for sizes whose evaluation would take a GPU minutes and most of
its memory: tests/host_plan.hip wraps the library's planning functions (no device needed)."""
import ctypes
import os
import subprocess

import pytest

from paper_2506_07430_amd import build, elocal


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host_plan") / "host_plan")
    src = os.path.join(build.ROOT, "tests", "host_plan.hip")
    subprocess.run([build.HIPCC, *build.FLAGS, "-w", "-c", src, "-o", out + ".o"], check=True)
    # (the kernels' launchers, which the planning source refers to, come from the built library)
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-shared", "-Wl,-Bsymbolic", out + ".o", build.LIB,
                    "-Wl,-rpath," + build.PKG, "-o", out + ".so"], check=True)
    L = ctypes.CDLL(out + ".so")
    L.host_handle.restype = ctypes.c_void_p
    L.host_free.argtypes = [ctypes.c_void_p]
    for f in ("host_items", "host_part", "elocal_launch_info", "elocal_tune"):
        getattr(L, f).restype = ctypes.c_int64
    for f in ("elocal_workspace_bytes", "elocal_workspace_bytes_multi", "elocal_pauli_workspace_bytes", "host_plan_bytes",
              "host_plain_bytes"):
        getattr(L, f).restype = ctypes.c_size_t
    return L


def ansatz(widths, precision):
    w = (ctypes.c_int * len(widths))(*widths)
    return elocal._Ansatz(len(widths), w, precision, None)


@pytest.mark.parametrize("n,na,widths,samples,precision", [
    (60, 26, (256,) * 3, 128, elocal.BF16),
    (60, 26, (256,) * 3, 5_800_000, elocal.BF16),     # 4.3e9 items in 142 GiB of workspace
    (60, 26, (256,) * 3, 5_800_000, elocal.FP64),
    (64, 32, (256,) * 8, 2_400_000, elocal.BF16),
])
def test_work_item_counter_does_not_wrap(plan, n, na, widths, samples, precision):
    """Every wave takes tickets until one is past the last, so the 32-bit counter must hold the
    tickets and one more per wave: a counter that wraps hands out work for ever. The tickets
    (items of samples b, b + step, ...) cover every item once."""
    h = ctypes.c_void_p(plan.host_handle(n, na, na))
    out = (ctypes.c_int64 * 4)()
    a = ansatz(widths, precision)
    items = plan.host_items(h, ctypes.byref(a), ctypes.c_int64(samples), out)
    plan.host_free(h)
    tickets, step, per_sample, waves = out
    assert items == per_sample * samples and waves > 0
    assert tickets + waves < 2 ** 32
    assert tickets == per_sample * step and 1 <= step <= samples


@pytest.mark.parametrize("precision", [elocal.BF16, elocal.FP64])
@pytest.mark.parametrize("n,na,nb,widths", [(12, 1, 0, (128, 128)), (24, 1, 1, (128, 128)), (40, 2, 2, (256,) * 3),
                                            (60, 1, 0, (256,) * 3), (60, 5, 5, (256,) * 3), (64, 2, 3, (64, 64))])
def test_few_electrons_run_every_entry(plan, n, na, nb, widths, precision):
    """The shared evaluation runs all n (2 n - 1) parents of a sample, which cost 2 to 7 entries
    each: systems of few electrons were up to 200 times slower by it (60 orbitals, one electron)."""
    h = ctypes.c_void_p(plan.host_handle(n, na, nb))
    a = ansatz(widths, precision)
    assert plan.host_prefix(h, ctypes.byref(a)) == 0
    plan.host_free(h)


@pytest.mark.parametrize("n,na,nb,widths", [(19, 9, 9, (128,)), (19, 9, 10, (96,)), (18, 9, 9, (128,))])
def test_one_hidden_layer_runs_every_entry_up_to_19_orbitals(plan, n, na, nb, widths):
    """The parents of so few entries take longer than one layer's products: 16 samples 63 us by
    themselves and 118 shared, 1024 samples 1.08 ms either way."""
    h = ctypes.c_void_p(plan.host_handle(n, na, nb))
    a = ansatz(widths, elocal.BF16)
    assert plan.host_prefix(h, ctypes.byref(a)) == 0
    plan.host_free(h)


def test_systems_of_the_gpu_test_take_the_shared_evaluation(plan):
    from tests.test_gpu_multi_prefix import BF16, FP64
    from tests.test_gpu_prefix_rule import SHAPES
    more = [(p, n, k, k, w, 1) for p in (elocal.BF16, elocal.FP64)
            for n, k, w in ((24, 12, (128, 128)), (24, 8, (128, 128)), (40, 14, (256,) * 3), (60, 26, (256,) * 3),
                            (60, 20, (64, 64)), (64, 21, (256,) * 3))]
    more += [(p, *s, 1) for p, shapes in ((elocal.BF16, BF16[1:]), (elocal.FP64, FP64[1:])) for s in shapes]
    for precision, n, na, nb, widths, _ in SHAPES + more:
        h = ctypes.c_void_p(plan.host_handle(n, na, nb))
        a = ansatz(widths, precision)
        assert plan.host_prefix(h, ctypes.byref(a)) == 1, (precision, n, na, nb, widths)
        plan.host_free(h)


@pytest.mark.parametrize("n,na,nb,widths,samples,parts", [
    (8, 4, 4, (32,), 1, 8), (8, 4, 4, (32,), 2048, 8), (8, 4, 4, (32,), 4096, 0),   # 4096 waves of the chip
    (4, 2, 2, (32,), 1, 0), (4, 2, 2, (32,), 4097, 0), (4, 2, 2, (32,), 16384, 0),  # one group per sample
    (6, 3, 3, (64, 64), 2048, 8), (6, 3, 3, (64, 64), 8192, 0),
    (12, 6, 6, (64, 64), 512, 8), (12, 6, 6, (64, 64), 1024, 0),
    (8, 4, 4, (256, 256), 1024, 8), (8, 4, 4, (256, 256), 2048, 0), (9, 4, 5, (256, 256), 2048, 8),
])
def test_items_in_parts_only_where_waves_are_idle(plan, n, na, nb, widths, samples, parts):
    """Parts of items (whose lanes' sums go through memory) were taken by every batch of few items,
    also where whole items already kept every wave busy: up to 17% slower."""
    h = ctypes.c_void_p(plan.host_handle(n, na, nb))
    a = ansatz(widths, elocal.BF16)
    assert plan.host_parts(h, ctypes.byref(a), ctypes.c_int64(samples)) == parts
    plan.host_free(h)


@pytest.mark.parametrize("n,widths,samples", [(21, (64,), 32), (22, (64,), 48), (24, (64,), 24), (28, (64,) * 3, 32),
                                              (24, (128,), 48), (20, (128, 128), 48)])
def test_few_samples_of_narrow_networks_run_few_parts(plan, n, widths, samples):
    """Every part of a segment runs the segment's parents again, which narrow networks take longer
    for than for a part's entries: about one part per wave, not four or five."""
    h = ctypes.c_void_p(plan.host_handle(n, n // 2, n // 2))
    out = (ctypes.c_int64 * 4)()
    a = ansatz(widths, elocal.BF16)
    items = plan.host_items(h, ctypes.byref(a), ctypes.c_int64(samples), out)
    plan.host_free(h)
    assert 0 < items <= 2 * out[3]


def test_units_up_to_a_degree_in_closed_form(plan):
    for n in (2, 3, 10, 33, 64):
        for w in (32, 96, 256):
            for d in range(-1, n + 66):
                assert plan.host_units_le(n, w, d) == sum(j % (n - 1) + 1 <= d for j in range(w))


I64, SIZE = ctypes.c_int64, ctypes.c_size_t
BATCHES = sorted({int(round(1.19 ** k)) for k in range(90)}
                 | {b + d for b in (2048, 4096, 5461, 16384, 32768) for d in (-1, 0, 1)})
SIZED = [
    # n, n_alpha, n_beta, widths, precision
    (4, 2, 2, (32,), elocal.BF16), (8, 4, 4, (32,), elocal.BF16), (8, 4, 4, (32,), elocal.FP64),
    (9, 4, 5, (64, 64), elocal.BF16X3), (12, 6, 6, (128, 128), elocal.BF16), (12, 6, 6, (128, 128), elocal.FP64),
    (16, 8, 8, (256,), elocal.BF16), (24, 12, 12, (128, 128), elocal.BF16), (24, 12, 12, (64, 64), elocal.FP64),
    (60, 26, 26, (256,) * 3, elocal.BF16), (60, 26, 26, (256,) * 3, elocal.FP64), (60, 2, 2, (256,) * 3, elocal.BF16),
]


@pytest.mark.parametrize("tune", [0, 1, 4])
@pytest.mark.parametrize("n,na,nb,widths,precision", SIZED)
def test_workspace_of_a_batch_serves_every_smaller_one(plan, n, na, nb, widths, precision, tune):
    """Sizes grow with the batch (those of the plans do not: a batch with few items has parts of
    items, with sums of their own), a call runs with exactly what it asks for, and with the size
    for all its blocks it takes all its blocks."""
    h, a = ctypes.c_void_p(plan.host_handle(n, na, nb)), ansatz(widths, precision)
    ref, last, last_room, last_pauli, last_multi = ctypes.byref(a), 0, 0, 0, 0
    plan.elocal_tune(h, 1, I64(tune))
    plan.host_set_pauli(h, I64(5000))
    for b in BATCHES:
        need = plan.elocal_workspace_bytes(h, ref, I64(b), 1)
        room = plan.elocal_launch_info(h, ref, I64(b), 8)
        assert need >= last and room >= last_room and 0 < need <= room, b
        assert plan.host_part(h, ref, I64(b), SIZE(need), (I64 * 1)()) >= 1, b
        assert plan.host_plan_bytes(h, ref, I64(b), I64(0)) <= room, b
        last, last_room = need, room
        if precision == elocal.BF16:
            pauli = plan.elocal_pauli_workspace_bytes(h, ref, I64(b))
            assert pauli >= last_pauli and plan.host_plan_bytes(h, ref, I64(b), I64(5000)) <= pauli, b
            last_pauli = pauli
        both, refs, sizes = (ctypes.c_void_p * 2)(h, h), (ctypes.c_void_p * 2)(*[ctypes.addressof(a)] * 2), (I64 * 2)(b, 100)
        multi = plan.elocal_workspace_bytes_multi(2, both, refs, sizes)
        assert multi >= last_multi, b
        last_multi = multi
    plan.host_free(h)


@pytest.mark.parametrize("n,na,nb,widths,precision", SIZED + [
    (12, 6, 6, (256, 256), elocal.BF16), (10, 5, 5, (256,), elocal.BF16), (10, 5, 5, (64,), elocal.BF16),
    (12, 6, 6, (64, 64), elocal.FP64), (40, 14, 14, (256,) * 3, elocal.BF16)])
def test_allocation_free_calls_take_what_fits_without_checkpoints(plan, n, na, nb, widths, precision):
    """elocal_eval_noalloc takes every batch whose arrays and whole items fit its scratch: the
    checkpoints of the shared evaluation, or the sums of parts of items, do not shrink the limit."""
    h, a = ctypes.c_void_p(plan.host_handle(n, na, nb)), ansatz(widths, precision)
    ref, scratch = ctypes.byref(a), elocal.NOALLOC_SCRATCH_MIB << 20
    lo, hi = 1, 1 << 24   # the largest such batch
    while lo < hi:
        mid = (lo + hi + 1) // 2
        lo, hi = (mid, hi) if plan.host_plain_bytes(h, ref, I64(mid)) <= scratch else (lo, mid - 1)
    for b in (lo, lo - 1, lo - 7, lo * 9 // 10, lo // 2):
        grid = (I64 * 1)()
        assert plan.elocal_workspace_bytes(h, ref, I64(b), 1) <= scratch, b
        assert 1 <= plan.host_part(h, ref, I64(b), SIZE(scratch), grid) <= b and grid[0] >= 1
    assert plan.elocal_workspace_bytes(h, ref, I64(2 * lo), 1) > scratch
    plan.host_free(h)


@pytest.mark.parametrize("n,na,widths,waves", [(12, 6, (128, 128), 8), (60, 26, (256,) * 3, 8), (8, 4, (32,), 4)])
def test_fp64_kernels_report_the_waves_they_are_built_for(plan, n, na, widths, waves):
    h, a = ctypes.c_void_p(plan.host_handle(n, na, na)), ansatz(widths, elocal.FP64)
    assert [plan.elocal_launch_info(h, ctypes.byref(a), I64(16), what) for what in (2, 4)] == [waves, waves]
    plan.host_free(h)


@pytest.mark.parametrize("n,na,nb,product", [(10, 8, 5, 0), (10, 5, 2, 0), (8, 4, 4, 0), (12, 1, 6, 0), (9, 4, 4, 1),
                                             (12, 6, 6, 1), (14, 7, 3, 1), (20, 3, 2, 1), (40, 2, 1, 0)])
def test_sectors_of_few_entries_keep_row_lists(plan, n, na, nb, product):
    h = ctypes.c_void_p(plan.host_handle(n, na, nb))
    assert plan.host_sector_product(h) == product
    plan.host_free(h)
