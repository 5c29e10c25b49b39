"""Batches that fill the chip, on the automatic schedule: the launches inside a pass run
mid_pass (wave-level columns of 2^4..2^6 points, columns of 2^7 and 2^8 through LDS, rows of
2^5 up to the longest, couplings from a table refilled every 128 step boundaries). Members against the FP64 oracle."""
import sys

import numpy as np
import pytest

import torch  # noqa: F401  (imported at collection: the first import can take minutes)

import oracle
from paper_2410_02532_amd import opo as B
from test_gpu_lone import TOL, _instance, phase_rounding, rel_l2

pytestmark = pytest.mark.gpu


def _batch(sizes, nf, dk, n2):
    return [_instance(1 << l, nf, 70 + b, dk=dk * (b % 3), n2=n2 * (b % 2)) for b, l in enumerate(sizes)]


CASES = [
    ("f32", 3, [16, 13, 14, 15] * 3, 0.0, 0.0, 2),
    ("f32", 3, [16, 16, 15, 14, 14, 13], 0.4, 1e-17, 2),
    ("f32", 2, [16, 15, 14, 13] * 5, 0.0, 0.0, 4),
    ("f32", 3, [18, 18, 18], 0.4, 0.0, 2),
    ("f32", 2, [19, 19], 0.4, 1e-17, 2),
    ("f32", 3, [20, 20], 0.0, 0.0, 4),
    ("f64", 3, [18, 18], 0.0, 0.0, 2),
    ("f64", 2, [19, 19], 0.4, 0.0, 2),
    ("f64", 3, [16, 13, 14, 15, 12] * 3, 0.4, 1e-17, 2),
    ("f64", 2, [17, 16, 15, 13] * 3, 0.0, 0.0, 4),
]


@pytest.mark.parametrize("precision, nf, sizes, dk, n2, order", CASES)
def test_batch_round_trips(precision, nf, sizes, dk, n2, order):
    """Two round trips of every member; the first and last sizes' members are checked."""
    print("batch %s nf %d %s order %d" % (precision, nf, sizes, order), file=sys.stderr, flush=True)
    insts = _batch(sizes, nf, dk, n2)
    nz, nrt = 5, 2
    with B.Opo(insts, nz, precision=precision, split_order=order) as h:
        h.cavity_roundtrip(nrt)
        got = [h.get_fields(i) for i in range(len(insts))]
    for i in sorted({sizes.index(l) for l in sizes} | {len(sizes) - 1}):
        ins = insts[i]
        ref, _ = oracle.roundtrips(dict(ins["crystal"], order=order), ins["cavity"], ins["fields"], ins["pump_in"],
                                   nz, nrt)
        tol = TOL[precision] + phase_rounding(ins["crystal"], nz * nrt * (3 if order == 4 else 1), 5.0 / nz)
        for x in range(nf):
            assert rel_l2(got[i][x], ref[x]) <= tol, (i, x, rel_l2(got[i][x], ref[x]), tol)


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_batch_pass_over_the_coupling_chunk(precision):
    """More steps than the coupling table holds, with mismatch; two calls equal one bit for
    bit (the second call's table starts elsewhere)."""
    print("batch chunk %s" % precision, file=sys.stderr, flush=True)
    insts = _batch([14] * 22 + [13], 3, 0.4, 0.0)
    nz, dz = 140, 2.0 ** -5      # z of every step is exact, so both splits form the same phases
    out = []
    for calls in ((nz,), (131, 9)):
        with B.Opo(insts, nz, precision=precision) as h:
            for n in calls:
                h.ssfm_propagate(n, dz)
            out.append([h.get_fields(i) for i in (0, 1, 22)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    for i, a in zip((1, 22), out[0][1:]):
        ref = oracle.ssfm_pass(insts[i]["crystal"], insts[i]["fields"], nz, dz)
        for x in range(3):
            assert rel_l2(a[x], ref[x]) <= TOL[precision], (i, x, rel_l2(a[x], ref[x]))


@pytest.mark.parametrize("precision, log2nt, count", [("f32", 15, 345), ("f32", 16, 174), ("f64", 13, 699)])
def test_batch_beyond_the_last_cache_level(precision, log2nt, count):
    """Fields of more than 256 MB, where the kernels and the order of a launch change: equal
    members of a half of the batch (every other one; the halves' first and last row
    transforms run in different kernels) stay equal bit for bit wherever they lie, and
    match the oracle."""
    print("batch %s %d of 2^%d" % (precision, count, log2nt), file=sys.stderr, flush=True)
    insts = _batch([log2nt] * 3, 3, 0.0, 0.0)
    nz, nrt = 5, 2
    with B.Opo(insts * (count // 3), nz, precision=precision) as h:
        h.cavity_roundtrip(nrt)
        first = [h.get_fields(i) for i in range(6)]
        for i in range(count // 2, count, 7):
            assert np.array_equal(h.get_fields(i), first[i % 6]), i
    for ins, *halves in zip(insts, first, first[3:]):
        ref, _ = oracle.roundtrips(ins["crystal"], ins["cavity"], ins["fields"], ins["pump_in"], nz, nrt)
        tol = TOL[precision] + phase_rounding(ins["crystal"], nz * nrt, 5.0 / nz)
        for got in halves:
            for x in range(3):
                assert rel_l2(got[x], ref[x]) <= tol, (x, rel_l2(got[x], ref[x]), tol)


@pytest.mark.parametrize("precision, nf, log2nt, count, nz", [
    ("f32", 3, 16, 6, 3), ("f32", 3, 17, 4, 2), ("f32", 2, 16, 8, 1), ("f32", 3, 15, 12, 3), ("f64", 3, 16, 6, 3)])
def test_equal_members_of_both_halves_agree(precision, nf, log2nt, count, nz):
    """Equal members agree bit for bit whichever half of the batch they were dealt to (the
    halves' first and last row transforms fall into different launches)."""
    print("batch members %s nf %d %d of 2^%d nz %d" % (precision, nf, count, log2nt, nz), file=sys.stderr, flush=True)
    insts = _batch([log2nt], nf, 0.0, 0.0) * count
    insts[0]["crystal"]["length_mm"] = float(nz)
    with B.Opo(insts, nz, precision=precision) as h:
        h.cavity_roundtrip(2)
        first, energies = h.get_fields(0), h.energy_history(0)
        for i in range(1, count):
            assert np.array_equal(h.get_fields(i), first), i
            assert np.array_equal(h.energy_history(i), energies), i


@pytest.mark.parametrize("precision, nf, log2nt, count, order", [("f64", 3, 9, 684, 2), ("f64", 2, 9, 1024, 4),
                                                                 ("f32", 3, 10, 342, 4)])
def test_batch_of_small_grids_refills_its_couplings(precision, nf, log2nt, count, order):
    """Small grids hold the couplings of a few steps only (an eighth of their fields): passes
    over many refills against the oracle, and two calls equal to one bit for bit."""
    print("batch refills %s nf %d 2^%d order %d" % (precision, nf, log2nt, order), file=sys.stderr, flush=True)
    members = _batch([log2nt] * 3, nf, 0.4, 0.0)
    insts = [members[b % 3] for b in range(count)]
    nz, dz = 40, 2.0 ** -5
    out = []
    for calls in ((nz,), (29, 11)):
        with B.Opo(insts, nz, precision=precision, split_order=order) as h:
            for n in calls:
                h.ssfm_propagate(n, dz)
            out.append([h.get_fields(i) for i in (0, 1, 2, count - 1)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    for ins, a in zip(members, out[0]):
        ref = oracle.ssfm_pass(dict(ins["crystal"], order=order), ins["fields"], nz, dz)
        for x in range(nf):
            assert rel_l2(a[x], ref[x]) <= TOL[precision], (x, rel_l2(a[x], ref[x]))


def test_batch_of_small_grids_holds_few_tables():
    """Device memory of a handle per instance beyond its fields, from two handles (what both
    hold cancels): a second copy of the fields, 1024 rows of energies, and tables that stay
    below a quarter of the fields, each of some 20 allocations rounded up to 2 MiB."""
    ins = _batch([9], 3, 0.4, 0.0)[0]
    fields, counts, used = 3 * 512 * 16, (1000, 6000), []
    print("batch memory %s of 2^9" % (counts,), file=sys.stderr, flush=True)
    hold = torch.empty(fields * counts[1], dtype=torch.uint8, device="cuda")   # torch keeps room for the state
    del hold
    for n in counts:
        before = torch.cuda.mem_get_info()[0]
        with B.Opo([ins] * n, 4, precision="f64"):
            used.append(before - torch.cuda.mem_get_info()[0])
    assert used[1] - used[0] <= (counts[1] - counts[0]) * (fields + 1024 * 24 + fields // 4) + 20 * (2 << 20), used


@pytest.mark.parametrize("sizes, l, mid", [([13, 13, 18, 18], 13, False), ([13] * 44, 13, True), ([13] * 40 + [19], 13, False),
                                           ([13, 16] * 6, 16, True), ([15, 19, 15, 19], 15, False)])
def test_fp64_batch_splits_follow_its_kernels(sizes, l, mid):
    """The splits timed with mid_pass are taken only by batches that run it (one column and
    one row size range); the others take the table's, as a forced split or kernel would."""
    print("fp64 batch splits %s" % sizes[:4], file=sys.stderr, flush=True)
    with B.Opo(_batch(sizes, 3, 0.0, 0.0), 5, precision="f64") as h:
        log2n1, log2n2, resident = h.plan(sizes.index(l))
    assert not resident
    assert log2n1 + log2n2 == l and log2n2 == (6 if mid else {13: 4, 15: 4, 16: 5}[l])


@pytest.mark.parametrize("nf, log2nt, count, order", [(3, 9, 684, 2), (2, 9, 1024, 4), (2, 10, 512, 4), (3, 19, 2, 2)])
def test_fp32_batches_that_keep_mixed_pass(nf, log2nt, count, order):
    """FP32 batches that mid_pass runs slower (short columns, or a launch that fits the chip
    at once with the smaller kernel only) stay with the kernels of the two-pass schedule
    (same splits, so the same results bit for bit)."""
    print("fp32 mixed nf %d 2^%d order %d" % (nf, log2nt, order), file=sys.stderr, flush=True)
    members = _batch([log2nt] * 3, nf, 0.4, 0.0)
    out = []
    for schedule in ("auto", "two_pass"):
        with B.Opo([members[b % 3] for b in range(count)], 6, precision="f32", split_order=order,
                   schedule=schedule) as h:
            h.cavity_roundtrip(2)
            out.append([h.get_fields(i) for i in sorted({0, 1, min(2, count - 1), count - 1})])
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("precision, nf, log2nt, count, col, order", [
    ("f32", 3, 10, 344, 0, 4), ("f32", 3, 11, 174, 0, 4), ("f32", 2, 11, 258, 0, 4), ("f32", 3, 12, 87, 4, 4),
    ("f32", 3, 13, 44, 4, 2), ("f32", 3, 14, 24, 5, 2), ("f64", 3, 9, 690, 0, 2), ("f64", 3, 10, 344, 0, 4),
    ("f64", 2, 11, 258, 0, 4), ("f64", 3, 12, 87, 6, 2)])
def test_batch_short_rows_and_columns(precision, nf, log2nt, count, col, order):
    """Rows of 2^5 and 2^6 points and columns of 2^4 and 2^5 (the shapes that batches of small
    grids, forced splits, fourth-order steps and several crystals reach): with and without
    mismatch and Kerr terms against the oracle; equal members agree bit for bit."""
    print("batch short %s nf %d 2^%d col %d order %d" % (precision, nf, log2nt, col, order), file=sys.stderr, flush=True)
    members = _batch([log2nt] * 3, nf, 0.4, 1e-17)
    nz, nrt = 5, 2
    with B.Opo([members[b % 3] for b in range(count)], nz, precision=precision, col_log2=col, split_order=order) as h:
        h.cavity_roundtrip(nrt)
        got = [h.get_fields(i) for i in range(6)]
        for i in range(count - 3, count):
            assert np.array_equal(h.get_fields(i), got[i % 3]), i
    for a, b in zip(got, got[3:]):
        assert np.array_equal(a, b)
    for ins, a in zip(members, got):
        ref, _ = oracle.roundtrips(dict(ins["crystal"], order=order), ins["cavity"], ins["fields"], ins["pump_in"],
                                   nz, nrt)
        tol = TOL[precision] + phase_rounding(ins["crystal"], nz * nrt * (3 if order == 4 else 1), 5.0 / nz)
        for x in range(nf):
            assert rel_l2(a[x], ref[x]) <= tol, (x, rel_l2(a[x], ref[x]), tol)


@pytest.mark.parametrize("precision, sizes, col", [
    ("f32", [14] * 20 + [13] * 6, 0), ("f64", [14] * 20 + [13] * 6, 0),      # a batch
    ("f32", [11, 11], 4), ("f64", [11, 11], 4),                               # a pair of launches a step
    ("f32", [11, 13, 12], 0), ("f64", [11, 13, 12], 0)])                      # one launch a pass
def test_crystals_with_their_own_tables(precision, sizes, col):
    """Two crystals of other mismatch, dispersion and step count, the first longer than the
    coupling table (128 steps): their descriptors, propagators and refilled couplings."""
    print("two crystals %s %s x%d" % (precision, sizes[:2], len(sizes)), file=sys.stderr, flush=True)
    insts, nzs, nrt = [], [131, 6], 2
    for b, l in enumerate(sizes):
        ins = _instance(1 << l, 3, 40 + b, dk=0.4 * (b % 2))
        second = dict(ins["crystal"], dk_per_mm=-0.3, length_mm=3.0, n2_m2_per_w=1e-17 * (b % 2))
        second["b2_fs2_per_mm"] = (-150.0, 100.0, 250.0)
        insts.append(dict(ins, crystals=[ins["crystal"], second]))
    with B.Opo(insts, nzs, precision=precision, col_log2=col) as h:
        h.cavity_roundtrip(nrt)
        got = [h.get_fields(i) for i in range(len(insts))]
    for i in sorted({0, 1, len(sizes) - 1}):
        ins = insts[i]
        ref, _, _ = oracle.roundtrips_multi(ins["crystals"], nzs, ins["cavity"], ins["fields"], ins["pump_in"], nrt)
        tol = TOL[precision] + sum(phase_rounding(c, n * nrt, c["length_mm"] / n) for c, n in zip(ins["crystals"], nzs))
        for x in range(3):
            assert rel_l2(got[i][x], ref[x]) <= tol, (i, x, rel_l2(got[i][x], ref[x]), tol)


@pytest.mark.parametrize("sizes, nf, col, order", [
    ([9] * 128 + [10] * 320, 3, 0, 4), ([9] * 1024 + [10, 10], 2, 0, 4), ([9, 10, 11] * 100, 3, 6, 2)])
def test_fp32_batches_of_short_columns_and_several_shapes(sizes, nf, col, order):
    """Short columns of more than one shape: against the oracle, equal members bit for bit."""
    print("batch short mix nf %d %s x%d order %d" % (nf, sorted(set(sizes)), len(sizes), order), file=sys.stderr, flush=True)
    member = {l: _instance(1 << l, nf, 20 + l, dk=0.4) for l in set(sizes)}
    nz, nrt = 5, 2
    with B.Opo([member[l] for l in sizes], nz, precision="f32", split_order=order, col_log2=col) as h:
        h.cavity_roundtrip(nrt)
        got = [h.get_fields(i) for i in range(len(sizes))]
    for l, ins in member.items():
        ref, _ = oracle.roundtrips(dict(ins["crystal"], order=order), ins["cavity"], ins["fields"], ins["pump_in"], nz, nrt)
        tol = TOL["f32"] + phase_rounding(ins["crystal"], nz * nrt * (3 if order == 4 else 1), 5.0 / nz)
        mine = [g for g, size in zip(got, sizes) if size == l]
        for x in range(nf):
            assert rel_l2(mine[0][x], ref[x]) <= tol, (l, x, rel_l2(mine[0][x], ref[x]), tol)
        for g in mine[1:]:
            assert np.array_equal(g, mine[0])
