"""GPU exponential maps by the direct sums (VALU tiles, the split form, the
matrix-core forms and their batch launch), which sliding windows leave to
atoms, grids and callers they do not suit: the parity tests of those forms
again, under an explicit tiling, which keeps every map from sliding."""
import dataclasses

import numpy as np
import pytest

import oracle
import test_gpu_batch as batch_tests
import test_gpu_parity as parity
import tfsynth
from checks import TOL, check_map, check_results

pytestmark = pytest.mark.gpu

T = tfsynth.T_SFT
DENSE = 1 << 30   # a runs threshold that no tile reaches: the dense and split forms


@pytest.fixture(scope="module")
def _open():
    import paper_1805_05652_amd as tf
    c = tf.Context(0, arena_bytes=4 << 30)
    yield c
    c.close()


@pytest.fixture
def direct(_open):
    """A context whose exponential maps are summed directly; at the test's end
    no sliding launch may have been recorded."""
    c = _open
    c.tiling_config(DENSE, -1)
    c.profile_reset()
    c.profile(True)
    yield c
    c.profile(False)
    c.tiling_config(-1, -1)
    assert c.profile_read()["recur"][0] == 0, "a map slid"


def like(test):
    """The parametrization of another test."""
    def apply(f):
        for m in getattr(test, "pytestmark", []):
            if m.name == "parametrize":
                f = pytest.mark.parametrize(*m.args, **m.kwargs)(f)
        return f
    return apply


@like(parity.test_matrix_any_grid)
def test_matrix_any_grid(direct, case, prec):
    parity.test_matrix_any_grid(direct, case, prec)
    prof = direct.profile_read()   # (of the test's first map)
    assert (prof["abc"][0] > 0) == (case != "bins1_valu"), prof


@like(parity.test_matrix_ragged)
def test_matrix_ragged(direct, case, prec):
    parity.test_matrix_ragged(direct, case, prec)
    prof = direct.profile_read()
    assert prof["mfma"][0] == prof["abc"][0] == 1, prof


@like(parity.test_abc_scan_rows)
def test_abc_scan_rows(direct, case):
    parity.test_abc_scan_rows(direct, case)
    prof = direct.profile_read()
    # (few_taus: its one block of taus starts with a band too short for the matrix cores)
    assert prof["mfma"][0] == prof["abc"][0] == (case != "few_taus"), prof


def test_f16x3_bin_scales(direct):
    parity.test_f16x3_bin_scales(direct)
    assert direct.profile_read()["mfma"][0] == 1


@like(parity.test_exp_bins_groups)
def test_exp_bins_groups(direct, n_bins):
    parity.test_exp_bins_groups(direct, n_bins)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_ragged_grid_with_edges(direct, prec):
    parity.test_ragged_grid_with_edges(direct, prec, "exp")


@pytest.mark.parametrize("prec", ["fp32", "f16x3", "bf16x3"])
def test_full_exp_256_bins(direct, prec):
    """The 256-bin workload, sampled cells and every bin's argmax."""
    print("case: full exp 256 bins direct " + prec, flush=True)
    from checks import check_sampled
    atoms, win = tfsynth.workload_exp_bins()
    aid = direct.upload_atoms(atoms)
    try:
        res, twoF = direct.fmap(aid, win, prec, want_map=True)
        check_sampled(twoF, res, atoms, win, TOL[prec], np.random.default_rng(3))
        prof = direct.profile_read()
        assert (prof["mfma"][0] > 0) == (prec != "fp32") and prof["abc"][0] > 0, prof
    finally:
        direct.free(aid)


@like(batch_tests.test_matrix_batch_against_oracle_and_fmap)
def test_matrix_batch(direct, prec):
    batch_tests.test_matrix_batch_against_oracle_and_fmap(direct, prec)
    assert direct.profile_read()["mfma"][0] > 0   # (the maps alone)


@like(batch_tests.test_batch_split_form)
def test_batch_split_form(direct, prec):
    batch_tests.test_batch_split_form(direct, prec)
    assert (direct.profile_read()["abc"][0] > 0) == (prec == "fp32")


@like(batch_tests.test_small_batch_against_oracle_and_fmap)
def test_small_batch(direct, prec):
    batch_tests.test_small_batch_against_oracle_and_fmap(direct, prec)


@like(batch_tests.test_sparse_row_batch)
def test_sparse_row_batch(direct, prec):
    batch_tests.test_sparse_row_batch(direct, prec)


def test_autotuned_batch(direct):
    batch_tests.test_autotuned_batch(direct)


@like(batch_tests.test_batch_composition_invariance)
def test_batch_composition_invariance(direct, prec):
    batch_tests.test_batch_composition_invariance(direct, prec)


@pytest.mark.parametrize("n_bins", [5, 21, 60])
@pytest.mark.parametrize("prec", ["f16x3", "bf16x3", "fp32", "fp64"])
def test_atoms_that_do_not_slide(_open, prec, n_bins):
    """One bin with a value that is not finite: the map takes the direct forms
    of its precision without any tiling, and every other bin is right."""
    print("case: one bin not finite %s %d bins" % (prec, n_bins), flush=True)
    c = _open
    base = tfsynth.make_atoms(9990 + n_bins, 900, 0.1, n_bins=n_bins)
    win = tfsynth.linspace_grid(base, "exp", 140, 90)
    fa = base.fa.copy()
    fa[3, 400, 0] = np.inf
    others = [b for b in range(n_bins) if b != 3]
    keep = dataclasses.replace(base, fa=base.fa[others], fb=base.fb[others])
    ref = oracle.fmap_atoms(keep, win)
    aid = c.upload_atoms(dataclasses.replace(base, fa=fa))
    c.profile_reset()
    c.profile(True)
    try:
        res, twoF = c.fmap(aid, win, prec, want_map=True)
        c.profile(False)
        prof = c.profile_read()
        assert prof["recur"][0] == 0 and (prof["mfma"][0] > 0) == (prec in ("f16x3", "bf16x3"))
        check_map(twoF.cpu().numpy()[others], ref, TOL[prec])
        check_results([res[b] for b in others], ref, win, TOL[prec])
        with c.batch([(aid, win)], prec) as b:
            got = b.run()[0]
        assert [got[i] for i in others] == [res[i] for i in others]
    finally:
        c.profile(False)
        c.free(aid)


@pytest.mark.parametrize("shift", [17, 22, 26, 30, 40])
@pytest.mark.parametrize("case", ["one_slot", "every_fiftieth", "stretch"])
@pytest.mark.parametrize("prec", ["f16x3", "bf16x3"])
def test_strong_data_by_direct_sums(_open, prec, case, shift):
    """Slots 2^17 to 2^40 above the others, under the default plans and under
    an explicit tiling, bands long enough for the matrix cores: every cell to the
    precision's bound relative to max(2F, 1), also where the windows hold none
    of the strong slots."""
    print("case: strong data %s %s 2^%d" % (prec, case, shift), flush=True)
    c = _open
    base = tfsynth.make_atoms(9995, 900, 0.1, n_bins=5)
    at = {"one_slot": slice(400, 401), "every_fiftieth": slice(3, None, 50), "stretch": slice(300, 364)}[case]
    fa, fb = base.fa.copy(), base.fb.copy()
    fa[:, at] *= 2.0 ** shift
    fb[:, at] *= 2.0 ** shift
    atoms = dataclasses.replace(base, fa=fa, fb=fb)
    # (every fiftieth: also windows that fit between two strong slots)
    tau = np.arange(T // 2, 30 * T, T // 2) if case == "every_fiftieth" else np.arange(9, 129, 2) * T
    win = tfsynth.list_window("exp", np.arange(880) * T, tau)
    ref = oracle.fmap_atoms(atoms, win)
    aid = c.upload_atoms(atoms)
    try:
        for tiling in ((-1, -1), (DENSE, -1)):
            c.tiling_config(*tiling)
            res, twoF = c.fmap(aid, win, prec, want_map=True)
            check_map(twoF.cpu().numpy(), ref, TOL[prec])
            with c.batch([(aid, win)], prec) as b:
                assert b.run() == [res]
    finally:
        c.tiling_config(-1, -1)
        c.free(aid)
