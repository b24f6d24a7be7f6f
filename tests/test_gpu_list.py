"""The list kernels (the automatic choice for most calls, rows of any length) against the sort oracle,
position by position: sizes around the tiles, the samples and the list capacities, ties, specials, crowded rows,
ragged rows and rows whose sample misleads."""
import numpy as np
import pytest

import oracle
from paper_2501_14336_amd import workloads as W
from tests import verify
from tests.gpu_util import BF16, F16, F32, gpu_topk, to_device
from tests.test_gpu_ragged import _check_ragged, _run_ragged

pytestmark = pytest.mark.gpu
LIST = (5, 6)  # rtopk_row_trace: where


def _bits(x, dtype):
    with np.errstate(over="ignore"):
        return x.view(np.uint32) if dtype == F32 else x.astype(np.float16).view(np.uint16) if dtype == F16 else W.to_bf16_bits(x)


def _check(name, x, dtype, k, largest=True, sorted=True, batch=1, by_list=True, why=0):
    bits = _bits(np.asarray(x, np.float32), dtype).reshape(batch, -1)
    print("list:", name, bits.shape, "dtype", dtype, "k", k, "largest", largest, "sorted", sorted, flush=True)
    gv, gi, tr, _ = gpu_topk(to_device(bits, dtype), dtype, k, largest, sorted=sorted)
    wv, wi = oracle.topk(bits, dtype, k, largest)
    for r in range(batch):
        assert tr[r].error == 0 and tr[r].done, (r, tr[r].error)
        if sorted:  # (unsorted, the route depends on the list's length as well)
            assert tr[r].redo_why == why, (r, tr[r].redo_why)
            assert by_list is None or (tr[r].passes[0].where in LIST) == by_list
            assert np.array_equal(gi[r], wi[r]) and np.array_equal(gv[r], wv[r]), "row %d" % r
        else:
            verify.assert_same_selection(bits[r], gv[r], gi[r], wv[r], wi[r])
    return tr


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
def test_rows_held_in_registers(dtype):
    # around the capacities of every variant, any k the list has room for; whole and broken first and last vectors
    for n in (1, 2, 7, 8, 9, 63, 65, 1000, 2047, 2049, 4096, 4097, 8191, 8200, 16384, 16389, 32768, 32771):
        x = W.normal(3 * n, seed=n, sigma=3.0)
        for k in sorted({1, min(n, 50), min(n, 300), max(1, n // 3), n - n // 7, n}):
            if n <= 8192 or k <= 1900:
                _check("held", x, dtype, k, largest=k % 2 == 0, batch=3)
        y = np.where(W.uniform01(3 * n, 1) < 0.7, np.float32(2.5), x).astype(np.float32)     # crowded
        y[:: max(1, n // 3)] = np.nan
        for k in sorted({1, max(1, n // 5), max(1, n // 2), n}):
            if n <= 8192 or k <= 1900:
                _check("held, crowded", y, dtype, k, largest=k % 2 == 1, batch=3)
                _check("held, crowded", y, dtype, k, largest=k % 2 == 0, batch=3, sorted=False)
    z = np.full(5000, np.float32(-np.inf))
    z[::9] = np.nan
    for k in (1, 600, 4999):
        for largest in (True, False):
            _check("held, worst numbers only", z, dtype, k, largest)


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
def test_sizes_and_ks(dtype):
    least = 8192 if dtype == F32 else 16384
    for n in (least, least + 1, 30011, 65535, 65536, 65537, 131072 + 5, (1 << 18) + 3, (1 << 20) + 7):
        x = W.normal(n, seed=n, sigma=3.0)
        for k in sorted({1, 50, 1000, 2500, n // 10, n // 5}):
            _check("normal", x, dtype, k, largest=(k % 3 != 1), by_list=n >= least)
        _check("unsorted", x, dtype, n // 100, sorted=False)
    # k at the upper end (with larger margins than half a row allows, the call goes elsewhere)
    x = W.normal(300007, 5)
    for k, by_list in ((100000, True), (2 * 300007 // 5, False)):
        _check("large k", x, dtype, k, by_list=by_list)
        _check("large k", x, dtype, k, largest=False, sorted=False, by_list=by_list)


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("n", [40003, 300001])
def test_ties_specials_and_crowds(dtype, n):
    u = W.uniform01(n, 3)
    data = {
        "duplicates": W.duplicates(n, 1),                       # counted, not listed (long row)
        "constant": np.full(n, np.float32(-1.5)),
        "five values": np.floor(u * 5).astype(np.float32) - 2,
        "clipped": np.minimum(W.normal(n, 4), np.float32(1.5)),  # many equal elements above the bound
        "grid": np.floor(u * 300).astype(np.float32),
        "narrow": W.narrow(n, 6),
        "specials": W.specials_ramp(n, 7, with_nan=True),
        "outlier": np.where(np.arange(n) == n // 3, np.float32(1e30), W.normal(n, 8)).astype(np.float32),
        "mostly NaN": np.where(u < 0.9, np.float32(np.nan), W.normal(n, 9)).astype(np.float32),
        "zeros": np.where(u < 0.6, np.float32(0.0), np.where(u < 0.8, np.float32(-0.0), W.normal(n, 10))).astype(np.float32),
        "ascending": np.arange(n, dtype=np.float32) - n / 3,
        "descending": n / 3 - np.arange(n, dtype=np.float32),
    }
    for name, x in data.items():
        for k in (1, 100, 3000, n // 5):
            for largest in (True, False):
                _check(name, x, dtype, k, largest)


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("value", [1.5, -1.5, 0.0, -0.0, 2.0 ** -24, np.inf, -np.inf, np.nan])
def test_crowd_of_one_value(dtype, value):
    # the k-th best is one value that most of the row holds: compared as a number where equal numbers have one key (the smallest
    # fp16 denormal among them), by key for the zeros and NaNs; NaNs and the other zero beside it; short tiles at both ends
    n = 300007
    u, x = W.uniform01(n, 31), W.normal(n, 32)
    y = np.where(u < 0.9, np.float32(value), x).astype(np.float32)
    y[u > 0.9995] = np.nan
    y[(u > 0.9990) & (u <= 0.9995)] = -0.0 if value == 0.0 and not np.signbit(value) else 0.0
    for largest in (True, False):
        # (beyond what is better than the crowd on either side)
        for k in (20, 33000, 40000):
            _check("crowd of %r" % value, y, dtype, k, largest=largest)


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
def test_long_lists_with_infinities(dtype):
    # bins of their own for infinities: fewer and more of them than k, NaNs above them, beside numbers of a narrow range
    n = 400003
    u = W.uniform01(n, 41)
    for x in (W.normal(n, 42), np.linspace(6.0e4, -6.0e4, n, dtype=np.float32)):
        for share in (0.0005, 0.02, 0.4):
            y = x.astype(np.float32).copy()
            y[u < share] = np.inf
            y[u > 1.0 - share] = -np.inf
            y[(u > 0.5) & (u < 0.5 + share / 8)] = np.nan
            for k in (9000, 50000, 100000):
                for largest in (True, False):
                    _check("infinities %g" % share, y, dtype, k, largest=largest, sorted=k != 9000)


def test_rows_shared_out_in_held_stretches():
    # few rows above 128 KB, k up to 64: stretches of 32 KB; rows that end just before, at and after a stretch, crowds in some
    # stretches only; on both sides of the rule's lines
    for dtype, per in ((F32, 8192), (F16, 16384), (BF16, 16384)):
        for n in (2 * per + 1, 4 * per, 4 * per + 8, 5 * per - 7, 5 * per, 5 * per + 1, 8 * per + 8):
            for batch in (1, 5):
                x = W.normal(batch * n, seed=n, sigma=3.0)
                y = x.copy()
                y[n // 3: n // 3 + per + 100] = 7.0       # one value over more than a stretch
                z = np.where(W.uniform01(batch * n, 2) < 0.8, np.float32(np.nan), x).astype(np.float32)
                for k in (1, 48, 50, 64, 65, 400):
                    _check("stretches", x, dtype, k, largest=k != 50, batch=batch)
                    _check("stretches, flat", y, dtype, k, largest=k != 64, batch=batch, sorted=k != 1)
                    _check("stretches, NaN", z, dtype, k, largest=k != 65, batch=batch)


def test_batches_and_odd_rows():
    for dtype in (F32, F16, BF16):
        for batch, n in ((3, 20011), (7, 100003), (140, 16387), (600, 16384)):
            x = W.normal(batch * n, 11, sigma=3.0)
            for k in (1, 77, 1500):
                _check("batch", x, dtype, k, largest=k != 77, batch=batch)
    _check("logits", W.bf16_bits_to_f32(W.llm_logits(40, 131072, 12)).reshape(-1), BF16, 1024, batch=40)


def test_ragged_rows_short_and_long():
    lens = [1, 0, 63, 5000, 8193, 40000, 100003, 200001, 65536, 199999, 100001]
    for dtype in (F32, BF16):
        rows = [_bits(W.normal(n, 20 + r, sigma=3.0) if r % 4 else W.duplicates(n, 20 + r), dtype) for r, n in enumerate(lens)]
        for kk in (50, 4000):
            ks = [min(n, kk) for n in lens]
            for srt in (False, True):
                _check_ragged("list", rows, dtype, ks, True, None, srt)
                _check_ragged("list", rows, dtype, ks, False, None, srt)


def _sampled(n, vectors, elems, run=8):
    """Positions of a row (starting on a 16-byte boundary) that the sample covers: runs of 8 vectors of 16 bytes, or of 4."""
    def mix(z):
        z = z.astype(np.uint32)
        z ^= z >> np.uint32(16); z *= np.uint32(0x7feb352d)
        z ^= z >> np.uint32(15); z *= np.uint32(0x846ca68b)
        return z ^ (z >> np.uint32(16))
    runs, groups = vectors // run, (n // elems) // run
    c = np.arange(runs, dtype=np.uint64)
    with np.errstate(over="ignore"):
        h = (mix(c) >> np.uint32(16)).astype(np.uint64)
    g = (((c << np.uint64(16)) | h) * np.uint64(groups) // np.uint64(runs)) >> np.uint64(16)
    return (g[:, None] * np.uint64(run * elems) + np.arange(run * elems, dtype=np.uint64)[None, :]).reshape(-1).astype(np.int64)


@pytest.mark.parametrize("k", [300, 9000])
def test_rows_whose_sample_misleads_are_done_again(k):
    # the sampled positions hold the row's best elements, fewer than k of them count: the list comes out short
    n = 400000
    pos = _sampled(n, 4096, 4)
    for largest in (True, False):
        x = W.normal(n, 31)
        x[pos] = 100.0 + W.uniform01(len(pos), 32)
        for srt in (False, True):
            _check("misled", x if largest else -x, F32, k, largest, srt, why=8)


def test_misled_short_lists_of_two_launches():
    # the same where the sample is a launch of its own: one row too short for the sweep that takes it along (a sample of 2048 vectors; lists for 256
    # and for 1024 threads to put in order), and more rows than that takes
    for n, batch, vectors, k in ((200000, 1, 2048, 300), (200000, 1, 2048, 3500), (400000, 33, 4096, 300)):
        pos = _sampled(n, vectors, 4)
        hidden = np.setdiff1d(np.arange(n), pos)
        for largest in (True, False):
            x = W.normal(batch * n, 36).reshape(batch, n)
            y = x.copy()
            x[:, pos] = 100.0 + W.uniform01(len(pos), 37)
            y[:, hidden[W.uniform01(len(hidden), 64) < 0.65]] = 9.0
            _check("misled", x if largest else -x, F32, k, largest, batch=batch, why=8)
            tr = _check("hidden majority", y if largest else -y, F32, k, largest, batch=batch, why=5)
            assert all(t.redo & 1 for t in tr)


@pytest.mark.parametrize("k,n", [(50, 40000), (1000, 40000), (2500, 40000), (1000, 40003)])
def test_misled_rows_of_one_workgroup(k, n):
    # more rows than are held in registers: by 256, 512 and 1024 threads, each row selected anew by its own; whole vectors and broken ones
    batch = 258
    pos = _sampled(n, 1024, 4)
    x = W.normal(batch * n, 38).reshape(batch, n)
    x[::2, pos] = 100.0 + W.uniform01(len(pos), 39)
    for largest in (True, False):
        bits = (x if largest else -x).view(np.uint32)
        print("misled rows of one workgroup:", k, largest, flush=True)
        gv, gi, tr, _ = gpu_topk(to_device(bits, F32), F32, k, largest, sorted=True)
        wv, wi = oracle.topk(bits, F32, k, largest)
        assert np.array_equal(gi, wi) and np.array_equal(gv, wv)
        # (rows off the 16-byte grid have their sample elsewhere)
        assert all(t.error == 0 for t in tr) and (n % 4 != 0 or [t.redo & 1 for t in tr] == [1, 0] * (batch // 2))


@pytest.mark.parametrize("n,batch,vectors,k,crowd", [(40000, 258, 1024, 1000, 900), (40000, 258, 1024, 2500, 2048), (200000, 1, 2048, 300, 250),
                                                     (1 << 20, 1, 4096, 3000, 2500), (400000, 33, 4096, 300, 250), (400000, 1, 4096, 9000, 8000)])
def test_rows_of_fewer_ties_than_the_sample_promises(n, batch, vectors, k, crowd):
    # the sampled positions hold one value, more often than their share of k and less often than k, and the rest of the row is worse: the equal elements are counted, they
    # and what is better are fewer than k, and the row is selected anew; by one workgroup, two launches, one, several rows, and a long list
    pos = _sampled(n, vectors, 4)
    x = (-10.0 - np.abs(W.normal(batch * n, 131))).astype(np.float32).reshape(batch, n)
    x[:, np.unique(pos)[:: max(1, len(np.unique(pos)) // crowd)][:crowd]] = 5.0
    for largest in (True, False):
        tr = _check("crowd in the sample", x if largest else -x, F32, k, largest, batch=batch, why=8)
        assert all(t.redo & 1 for t in tr)


def test_misled_long_lists_of_the_halved_sample():
    # rows from 16 MB up: 8192 vectors in runs of 4; sorted, and unsorted, whose kernel hands a row over whose list is no use (fewer than k, more than half the row)
    for n, k, srt in (((1 << 22) + 4, 12000, True), (1 << 25, 70000, False)):
        pos = _sampled(n, 8192, 4, run=4)
        x = W.normal(n, 40)
        y = x.copy()
        x[pos] = 100.0 + W.uniform01(len(pos), 41)
        hidden = W.uniform01(n, 42) < 0.65
        hidden[pos] = False
        y[hidden] = 9.0
        for name, z, why in (("misled", x, 8), ("hidden majority", y, 5)):
            for largest in (True, False):
                v = z if largest else -z
                if srt:
                    tr = _check(name, v, F32, k, largest, why=why)
                else:
                    print("unsorted:", name, largest, flush=True)
                    gv, gi, tr, _ = gpu_topk(to_device(v.view(np.uint32).reshape(1, -1), F32), F32, k, largest, sorted=False)
                    assert tr[0].error == 0 and tr[0].done and tr[0].redo_why == why
                    _assert_best(v, v.view(np.uint32), k, largest, gv[0], gi[0])
                assert tr[0].redo == 1


def test_misled_rows_beside_others():
    # long lists, several workgroups per row, and every second row's list is no use: its buckets stay empty, its record says so,
    # and the rows beside it are not touched
    n, batch, k = 400000, 6, 9000
    pos = _sampled(n, 4096, 4)
    x = W.normal(batch * n, 33).reshape(batch, n)
    for r in range(0, batch, 2):
        x[r, pos] = 100.0 + W.uniform01(len(pos), 34 + r)
    for largest in (True, False):
        bits = (x if largest else -x).view(np.uint32)
        gv, gi, tr, _ = gpu_topk(to_device(bits, F32), F32, k, largest, sorted=True)
        wv, wi = oracle.topk(bits, F32, k, largest)
        assert np.array_equal(gi, wi) and np.array_equal(gv, wv)
        assert [t.redo & 1 for t in tr] == [1, 0] * (batch // 2) and all(t.error == 0 for t in tr)


def test_lists_and_buckets_that_do_not_fit_are_shared_out():
    # a trend along the row: more is listed than one workgroup orders in LDS, and it is cut down first (bit 2); crowds that the sample does not show: a bucket
    # that holds most of the list is shared out (bit 4), of one value and of neighbouring keys; one workgroup per row, and several
    n = 1 << 20
    for dtype, k in ((F32, 1000), (F16, 1000), (F32, 3000)):
        x = np.linspace(6.0e4, -6.0e4, n, dtype=np.float32)
        for largest in (True, False):
            for srt in (True, False):
                tr = _check("trend", x, dtype, k, largest, sorted=srt)
                assert all(t.redo & 2 for t in tr), [t.redo for t in tr]
    x = np.stack([np.linspace(1.0, -1.0, 131072, dtype=np.float32)] * 260)
    tr = _check("trend, many rows", x, BF16, 1000, batch=260)
    assert any(t.redo & 2 for t in tr)
    n, k = 400000, 9000
    hidden = np.setdiff1d(np.arange(n), _sampled(n, 4096, 4))
    u = W.uniform01(n, 61)
    for crowd in (np.float32(9.0), (9.0 + u * 1e-3).astype(np.float32)):
        for count in (5000, 8000, 30000):
            y = W.normal(n, 62)
            where = hidden[:: len(hidden) // count][:count]
            y[where] = crowd if np.ndim(crowd) == 0 else crowd[where]
            for largest in (True, False):
                tr = _check("hidden crowd", y if largest else -y, F32, k, largest)
                assert tr[0].redo == 4


@pytest.mark.parametrize("n,batch,k,count", [(400000, 1, 9000, 180000), (400000, 1, 30000, 150000), (300000, 6, 9000, 120000)])
def test_buckets_of_more_parts_than_the_row_has_workgroups(n, batch, k, count):
    # parts of 2048 entries, a workgroup for each bucket and each 32 KB of the row at most (several rows: fewer): one part to each workgroup then, and a part
    # may have several runs of bins, or none
    hidden = np.setdiff1d(np.arange(n), _sampled(n, 4096, 4))
    u = W.uniform01(n, 161)
    where = hidden[u[hidden] < count / len(hidden)]
    y = W.normal(batch * n, 162).reshape(batch, n)
    for crowd in (np.full(len(where), np.float32(9.0)), (9.0 + W.uniform01(len(where), 163) * 1e-3).astype(np.float32)):
        y[:, where] = crowd
        for largest in (True, False):
            tr = _check("hidden crowd of many", y if largest else -y, F32, k, largest, batch=batch)
            assert all(t.redo == 4 and t.pre_kept > len(where) for t in tr), [(t.redo, t.pre_kept) for t in tr]


@pytest.mark.parametrize("dtype,n,batch,k,vectors,counts,threads", [
    (F32, 200000, 1, 300, 2048, (6000, 9000, 90000), 512), (F32, 400000, 33, 300, 4096, (9000, 100000), 512), (F32, 200000, 1, 3500, 2048, (10000, 17000, 60000), 1024),
    (F32, 1 << 20, 1, 1000, 4096, (12000, 17000, 300000), 1024), (F32, 600000, 3, 3000, 4096, (17000, 200000), 1024), (F16, 1441792, 1, 4100, 4096, (20000, 695000), 1024)])
def test_lists_far_longer_than_lds_holds(dtype, n, batch, k, vectors, counts, threads):
    # what the sample does not show lengthens the list, which one workgroup puts in order: more than 8 entries per thread are cut down to that first, more than 16 are read where they
    # lie, in two launches (by 512 and by 1024 threads) and in one; segments of a few entries and of many thousands, some of them empty.  The last row's second list is the only kind whose wanted
    # part is too much for a bound from a sample of it
    elems = 4 if dtype == F32 else 8
    hidden = np.setdiff1d(np.arange(n), _sampled(n, vectors, elems))
    u = W.uniform01(n, 141)
    for count in counts:
        chosen = hidden[u[hidden] < count / len(hidden)]
        for name, where in (("spread", chosen), ("together", hidden[len(hidden) // 3:][:len(chosen)])):
            x = W.normal(batch * n, 142).reshape(batch, n)
            x[:, where] = 20.0 + W.uniform01(len(where), 143)
            for largest in (True, False):
                for srt in (True, False) if count == counts[0] else (True,):
                    tr = _check("far too long, " + name, x if largest else -x, dtype, k, largest, sorted=srt, batch=batch, by_list=None)
                    # (who is spread is in every row, the sample's positions apart; a stretch of its own may hold some of them)
                    assert all(t.pre_kept > len(where) and t.redo & 1 == 0 for t in tr)
                    if len(where) > 16 * threads:
                        assert all(t.redo == 2 for t in tr), [t.redo for t in tr]


def test_lists_longer_than_half_the_row_are_selected_anew():
    # six elements in ten are one value that the sample does not show: everything listed, reason 5; a short list and a long one
    n = 400000
    hidden = np.setdiff1d(np.arange(n), _sampled(n, 4096, 4))
    y = W.normal(n, 63)
    y[hidden[W.uniform01(len(hidden), 64) < 0.65]] = 9.0
    for k in (300, 9000):
        for largest in (True, False):
            tr = _check("hidden majority", y if largest else -y, F32, k, largest, why=5)
            assert tr[0].redo & 1


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
def test_crowds_in_order(dtype):
    # what LDS holds of a list, with few values in it, or one far above the rest: bins between splitters; every size of workgroup
    for n, ks in ((1000, (1, 100, 300, 1000)), (4096, (100, 409, 1556)), (16384, (100, 1000)), (60000, (300, 2000))):
        u = W.uniform01(2 * n, 65)
        for name, x in (("two", np.floor(u * 2)), ("ten", np.floor(u * 10)), ("hundred", np.floor(u * 100)),
                        ("far", np.where(u < 0.001, np.float32(6.0e4), np.floor(u * 30) / 1024)), ("half", np.maximum(W.normal(2 * n, 66), 0))):
            for k in ks:
                for largest in (True, False):
                    _check("crowd of " + name, x.astype(np.float32), dtype, k, largest, batch=2, sorted=True)
                    _check("crowd of " + name, x.astype(np.float32), dtype, k, largest, batch=2, sorted=False)


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_crowds_around_what_the_samples_gathering_holds(dtype):
    # the sampled positions hold one value, as many of them as the gathered list holds, one more, and so on up to all of them:
    # the gathering is thinned until it fits, and ends
    n, vectors = 400000, 4096 if dtype == F32 else 2048
    elems = 4 if dtype == F32 else 8
    pos = np.unique(_sampled(n, vectors, elems))
    for crowd in (4096, 4097, 4098, 8191, 8192, 8193, 8200, 16000):
        crowd = min(crowd, len(pos))
        x = -np.abs(W.normal(n, 35)) - 1.0
        x[pos[:crowd]] = 5.0
        for k in (3, 9000):
            for largest in (True, False):
                gv, gi, tr, _ = gpu_topk(to_device(_bits(x if largest else -x, dtype), dtype), dtype, k, largest, sorted=True)
                wv, wi = oracle.topk(_bits(x if largest else -x, dtype), dtype, k, largest)
                print("crowd", dtype, crowd, k, largest, tr[0].redo, flush=True)
                assert np.array_equal(gi, wi) and np.array_equal(gv, wv) and tr[0].error == 0


@pytest.mark.parametrize("dtype", [F32, F16])
@pytest.mark.parametrize("values", [2, 3, 4, 8])
def test_few_values_never_fill_the_list(dtype, values):
    # equally frequent values, k between them: better and equal elements together are more than half the row, though neither is
    for n in (40000, 300007, 1 << 20):
        x = np.floor(W.uniform01(n, 71) * values).astype(np.float32)
        for share in (0.26, 0.3, 0.34, 0.38):
            for largest in (True, False):
                tr = _check("%d values" % values, x, dtype, int(share * n), largest, by_list=None)
                assert tr[0].redo & 1 == 0


@pytest.mark.parametrize("far", [np.float32(3.4e38), np.float32(1.0e9), np.float32(np.inf), np.float32(np.nan)])
def test_bins_do_not_follow_the_distance_to_a_few_keys(far):
    # one key in 2048 (NaN: in 200) lies far above the rest: the others share the long list's bins, so no bucket is too large
    n = 1 << 22
    u = W.uniform01(n, 72)
    for x in (W.uniform01(n, 73), W.normal(n, 74)):
        y = np.where(u < (1 / 200 if far != far else 1 / 2048), far, x).astype(np.float32)
        for k in (1 << 16, 1 << 18):
            tr = _check("far %r" % far, y, F32, k, by_list=True)
            assert tr[0].redo == 0, tr[0].redo
            if far == far:
                tr = _check("far %r" % -far, -y, F32, k, largest=False)
                assert tr[0].redo == 0, tr[0].redo


def test_splitters_are_the_same_every_time():
    # one key in 200 is a NaN, far above the rest: the interval between the last number's splitter and the first NaN's has its entries at its two
    # ends.  The waves that gather the sample come in any order; the row is put in order the same way all the same, without a bucket too long
    n, k = 1 << 22, 1 << 18
    x = np.where(W.uniform01(n, 72) < 1 / 200, np.float32(np.nan), W.uniform01(n, 73)).astype(np.float32)
    _check("far NaNs", x, F32, k)
    d = to_device(_bits(x, F32), F32)
    first = gpu_topk(d, F32, k, True, sorted=True)
    for i in range(40):
        gv, gi, tr, _ = gpu_topk(d, F32, k, True, sorted=True)
        assert tr[0].redo == 0 and np.array_equal(gi, first[1]) and np.array_equal(gv, first[0]), (i, tr[0].redo)


def test_crowd_of_nans_at_the_top_is_counted():
    # more NaNs than k: T is the NaNs' key, the last there is (the last of an even division's bins reaches beyond 32 bits)
    n = 1 << 22
    x = np.where(W.uniform01(n, 75) < 0.05, np.float32(np.nan), W.normal(n, 76)).astype(np.float32)
    for k in (40000, 100000):
        tr = _check("NaNs", x, F32, k)
        assert tr[0].redo == 0 and tr[0].pre_kept == 0


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_blocks_of_one_value_are_few_draws(dtype):
    # 64 neighbours each have one value: the sample's lines are as many draws, not its elements; no row of these is done again
    n = 1 << 21
    for seed in range(6):
        x = np.repeat(W.normal(n // 64, 80 + seed), 64)
        for k in (3000, n // 100, n // 10, n // 3):
            tr = _check("blocks", x, dtype, k, largest=seed % 2 == 0)
            assert tr[0].redo & 1 == 0


def test_rows_far_shorter_than_the_longest_have_samples_of_their_own():
    # a ragged batch: the sample's size goes by the longest row, but a row that is short against it is not listed whole
    lens = [50000] * 20 + [1 << 22] + [300, 1537, 3000, 12000, 98304, 98303]
    for dtype in (F32, BF16):
        rows = [_bits(W.normal(n, 90 + r, sigma=3.0), dtype) for r, n in enumerate(lens)]
        for kk in (100, 2000):
            ks = [min(n, kk) for n in lens]
            for srt in (False, True):
                _check_ragged("short rows", rows, dtype, ks, True, None, srt)
                for tr, n in zip(_run_ragged(rows, dtype, ks, True, None, srt, False)[2], lens):
                    assert tr.redo == 0 and (n < 20000 or tr.pre_kept < n // 3), (n, tr.redo, tr.pre_kept)


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
def test_nans_are_no_part_of_the_smallest(dtype):
    # held rows: a NaN is not below the bound on either side, so it has to be left out by name; otherwise every NaN is listed and ordered
    for n in (4096, 16384, 30000):
        x = np.where(W.uniform01(n, 77) < 0.05, np.float32(np.nan), W.normal(n, 78)).astype(np.float32)
        tr = _check("NaNs", x, dtype, 30, largest=False)
        assert tr[0].pre_kept < 100, tr[0].pre_kept
        # fewer numbers than k: NaNs follow them, and held rows that crowd at their bound
        z = np.where(W.uniform01(n, 79) < 0.9, np.float32(np.nan), W.normal(n, 78)).astype(np.float32)
        for k in (50, n // 8):
            for largest in (True, False):
                _check("mostly NaNs", z, dtype, k, largest, sorted=True)
                _check("crowd at the top", np.minimum(x, 1.0), dtype, k, largest, sorted=True)


def test_unsorted_calls_of_a_large_part_of_a_row_take_digit_passes():
    # on both sides of the rule's lines: the selection is the same, and which kernels made it is in the record
    for dtype, n, inside, beyond in ((F32, 4096, 256, 257), (F32, 16384, 1024, 1025), (F32, 20000, 1250, 5001),
                                     (F16, 4096, 64, 65), (BF16, 16384, 256, 257), (F16, 30000, 468, 1876)):
        x = W.normal(2 * n, 101)
        for k in (inside, beyond):
            for largest in (True, False):
                tr = _check("unsorted", x, dtype, k, largest, batch=2, sorted=False)
                assert all((t.passes[0].where in LIST) == (k == inside) for t in tr), (n, k, [t.passes[0].where for t in tr])
                _check("sorted", x, dtype, k, largest, batch=2)


def test_a_trend_has_a_short_list():
    # the sample has one run from every stretch of the row, so a trend's k-th key is known to a stretch or two: no margin for
    # independent runs, and a lane's best element does not stand for sixteen neighbouring stretches
    n = 1 << 22  # 2048 stretches
    x = np.linspace(1.0e6, -1.0e6, n, dtype=np.float32)
    for k in (16, 1000, 5000, 30000):
        for largest in (True, False):
            tr = _check("trend", x, F32, k, largest)
            # 65536 sampled elements, one in 64; the rank is taken among vectors of four, and the runs at either end are whole: up to four
            # times k and its margin of six deviations and six, and two stretches beyond
            ks = k / 64
            bound = 4 * 64 * (ks + 6 * ks ** 0.5 + 6) + 2 * 4 * 2048
            assert k <= tr[0].pre_kept < bound and tr[0].redo & 1 == 0, (tr[0].pre_kept, bound)


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
def test_rows_swept_by_waves(dtype):
    # short lists of few rows: tiles of 4 KB, a wave each; rows that end just before, at and after a tile, rows that begin
    # between 16-byte boundaries, batches on both sides of the rule's line, ties counted by tile (as numbers; zeros and NaNs by key)
    tile = 1024 if dtype == F32 else 2048
    for n in (16 * tile * 16, 16 * tile * 16 + 1, 17 * tile * 16 - 1, 16 * tile * 16 + 5 * tile - 9) if dtype == F32 else (2048 * tile + 1,):
        for batch in (1, 3) if dtype == F32 else (1,):
            x = W.normal(batch * n, seed=n, sigma=3.0)
            u = W.uniform01(batch * n, 3)
            for k in (70, 1500):
                _check("by waves", x, dtype, k, largest=k != 70, batch=batch, sorted=k != 70)
            for value in (2.5, 0.0, np.nan) if batch == 1 else (2.5,):
                y = np.where(u < 0.8, np.float32(value), x).astype(np.float32)
                _check("by waves, %g" % value, y, dtype, n // 3, value != 2.5, batch=batch)
                _check("by waves, %g" % value, y, dtype, 100, value == 2.5, batch=batch)
    if dtype == F32:
        for batch in (32, 33):
            x = W.normal(batch * 256 * tile, seed=batch, sigma=3.0)
            _check("batch", x, dtype, 200, batch=batch)
            y = np.where(W.uniform01(len(x), 4) < 0.9, np.float32(1.0), x).astype(np.float32)
            _check("batch, duplicates", y, dtype, 64 * tile, batch=batch)


def test_lists_a_little_too_long_are_cut_down():
    # a list of more than one workgroup orders in LDS, but no more than twice as long as expected, needs no second kernel; nor does one
    # whose segments have more entries than the places that are read at once
    n, k = 1 << 20, 3000
    hidden = np.setdiff1d(np.arange(n), _sampled(n, 4096, 4))
    for where in (hidden[:: len(hidden) // 5000][:5000], hidden[100000:105000]):
        x = W.normal(n, 51)
        x[where] = 9.0 + W.uniform01(len(where), 52)
        for largest in (True, False):
            for srt in (True, False):
                tr = _check("a little too long", x if largest else -x, F32, k, largest, sorted=srt)
                assert tr[0].redo == 0 and 8192 < tr[0].pre_kept <= 16384, (tr[0].redo, tr[0].pre_kept)


@pytest.mark.parametrize("k,most", [(300, 2048 + 1), (300, 2048 + 150), (3500, 8192 + 1500)])
def test_lists_a_little_too_long_are_cut_down_after_two_launches(k, most):
    # the same where sample and sweep are two launches, and a list's entries look for their segment: 512 threads (2048 entries, up to 2424 cut down
    # without a record of it) and 1024 threads (8192, up to 12788).  The bound is the sample's alone: so many more elements above it lengthen the list by just as many
    n = 200000
    hidden = np.setdiff1d(np.arange(n), _sampled(n, 2048, 4))
    x = W.normal(n, 51)
    below = hidden[x[hidden] < 0]
    for largest in (True, False):
        base = _check("as expected", x if largest else -x, F32, k, largest)[0].pre_kept
        more = most - base
        assert 0 < more < len(below)
        y = x.copy()
        y[below[:: len(below) // more][:more]] = 9.0 + W.uniform01(more, 52)
        for srt in (True, False):
            tr = _check("a little too long", y if largest else -y, F32, k, largest, sorted=srt)
            assert tr[0].redo == 0 and tr[0].pre_kept == most, (tr[0].redo, tr[0].pre_kept, base)


@pytest.mark.parametrize("dtype,n,runs", [(F32, (1 << 22) - 4099, 512), (F32, 1 << 22, 2048), (F32, (1 << 22) + 4099, 2048),
                                          (F16, (1 << 23) - 4099, 512), (F16, (1 << 23) + 5, 1024), (BF16, (1 << 23) + 5, 1024)])
def test_the_halved_sample_sees_a_trend(dtype, n, runs):
    # rows from 16 MB up: runs of half a line, and as many as there were.  A ramp's list is a few stretches of the row, of which there are as many as runs; on
    # either side of the rule's line, with a ragged end.  k = 600 is rank 25 of the sample at most, which seven of its best runs of four vectors
    # hold, one vector to a lane; 16-bit keys that equal the bound are listed with it, or counted (bf16: a value is up to n / 384 of the row)
    x = np.linspace(3, -3, n).astype(np.float32)
    for largest in (True, False):
        for k in (16, 100, 600):
            tr = _check("ramp", x, dtype, k, largest)
            assert (k if dtype == F32 else 0) <= tr[0].pre_kept <= 8 * (n // runs) + (0 if dtype == F32 else n // 384), tr[0].pre_kept


def _assert_best(x, bits, k, largest, gv, gi):
    key = x if largest else -x
    edge = np.partition(key, len(key) - k)[len(key) - k]
    want = np.concatenate([np.flatnonzero(key > edge), np.flatnonzero(key == edge)[: k - int((key > edge).sum())]])
    assert np.array_equal(np.sort(gi), np.sort(want)) and np.array_equal(bits[gi], gv)


def test_unsorted_long_lists_of_several_rows():
    # positions are reserved row by row: a batch, and a ragged one whose rows are empty, shorter than k, listed whole, or have k near their end
    n, k = 1 << 25, 70000
    x = np.stack([W.normal(n, 58), W.duplicates(n, 59)])
    for largest in (True, False):
        print("unsorted, two rows:", largest, flush=True)
        gv, gi, tr, _ = gpu_topk(to_device(x.view(np.uint32), F32), F32, k, largest, sorted=False)
        for r in range(2):
            assert tr[r].error == 0 and tr[r].done and tr[r].redo & 1 == 0 and tr[r].passes[0].where == 5
            _assert_best(x[r], x[r].view(np.uint32), k, largest, gv[r], gi[r])
    lens, ks = [n + 5, 0, 70000, 100001, 200003, 3000001, 1 << 20], [70000, 0, 70000, 70000, 69999, 1, 9000]
    rows = [W.normal(m, 60 + r) if r != 6 else W.duplicates(m, 66) for r, m in enumerate(lens)]
    for largest in (True, False):
        print("unsorted, ragged:", largest, flush=True)
        gv, gi, tr = _run_ragged([r.view(np.uint32) for r in rows], F32, ks, largest)
        for r, (row, kk) in enumerate(zip(rows, ks)):
            assert np.all(gi[r, kk:] == -1) and tr[r].error == 0
            if kk:
                assert tr[r].done and tr[r].passes[0].where in LIST
                _assert_best(row, row.view(np.uint32), kk, largest, gv[r, :kk], gi[r, :kk])


@pytest.mark.parametrize("k", [70000, (1 << 25) // 100])
def test_unsorted_long_lists(k):
    # better bins go to the output as they come, and the bin of rank k is ordered: keys of many values, duplicates (ties counted), a crowd in that
    # bin, and a row that ends inside a tile
    n = (1 << 25) + 5
    x = W.normal(n, 55)
    crowd = np.sort(x)[n - k]
    for name, y in (("normal", x), ("duplicates", W.duplicates(n, 56)),
                    ("crowd", np.where(W.uniform01(n, 57) < 0.0003, crowd, x))):
        bits = _bits(y.astype(np.float32), F32).reshape(1, -1)
        for largest in (True, False):
            print("unsorted:", name, k, largest, flush=True)
            gv, gi, tr, _ = gpu_topk(to_device(bits, F32), F32, k, largest, sorted=False)
            assert tr[0].error == 0 and tr[0].done and tr[0].passes[0].where == 5
            _assert_best(y, bits[0], k, largest, gv[0], gi[0])


@pytest.mark.parametrize("dtype", [F16, BF16])
def test_short_lists_in_many_segments(dtype):
    # one 16-bit row above 24 MB: 512 segments, of which a few have a little more than the places that are read at once, or (a ramp) one has nearly all; and a
    # row of which most is one value, so that next to nothing is listed
    n = 13000001
    x = W.normal(n, 91, sigma=3.0)
    for k in (16, 300, 1000):
        tr = _check("many segments", x, dtype, k, largest=k != 300)
        assert tr[0].redo == 0 and tr[0].pre_kept < 8192
    y = np.where(W.uniform01(n, 92) < 0.9, np.float32(0.5), x / 16).astype(np.float32)
    _check("many segments, ties", y, dtype, 1000, largest=True)
    _check("many segments, ramp", np.linspace(-3, 3, n).astype(np.float32), dtype, 100)


@pytest.mark.parametrize("dtype,n", [(F32, 300000), (F32, 524288 + 3), (F16, (1 << 21) + 9), (F32, (1 << 22) + 1)])
def test_ranks_on_both_sides_of_what_one_value_per_lane_holds(dtype, n):
    # the sample's rank of the k-th key is found among one value per lane, among two, and among vectors: k around 128 and 256 of 512 and 1024 values, with
    # crowds and in blocks, where a second, lower rank is looked for
    elems = 16384 if dtype == F32 and n < (1 << 22) else 32768  # of the sample
    for rank in (120, 136, 250, 264):
        s = (-6 + (36 + 4 * (rank - 6)) ** 0.5) / 2
        k = int(s * s * n / elems)
        x = W.normal(n, rank, sigma=3.0)
        for name, y in (("normal", x), ("nine in ten", np.where(W.uniform01(n, 5) < 0.9, np.float32(1.5), x)), ("blocks", np.repeat(x[: n // 64 + 1], 64)[:n])):
            tr = _check("rank %d, %s" % (rank, name), y.astype(np.float32), dtype, k, largest=rank != 136, by_list=True)
            assert tr[0].redo & 1 == 0


@pytest.mark.parametrize("dtype,n", [(F32, 300001), (F16, 1600001)])
@pytest.mark.parametrize("width", [40, 150, 700, 1500, 2500])
def test_crowds_of_which_little_is_wanted(dtype, n, width):
    # the best values have `width` elements each, neighbours or all over the row, and a list has a few such values: one bin has more than is ordered in one
    # go, and the bins up to it have less than half the list (256, 512 and 1024 threads, up to 2048 entries kept), just as much, or nearly all of it
    steps = np.arange(n) // width
    few = np.floor(W.uniform01(n, width) * (n // width))
    few = np.minimum(few, 2000.0) if dtype == F16 else few
    for name, x in (("steps", np.maximum(steps - (n // width - 1500), 0)), ("spread", few), ("a crowd and others", np.where(W.uniform01(n, 5) < 0.002, steps, few % 7))):
        for k in (1, 16, width - 1, width, width + 1, 3 * width):
            for largest in (True, False):
                y = x.astype(np.float32) if largest else -x.astype(np.float32)
                _check("%s of %d" % (name, width), y, dtype, k, largest, by_list=None)
                _check("%s of %d" % (name, width), y, dtype, k, largest, by_list=None, sorted=False)


@pytest.mark.parametrize("n", [(1 << 22) - 5, (1 << 22) + 4, (1 << 24) + 3])
def test_long_lists_bounded_by_half_the_largest_sample(n):
    # around the first row that has the largest sample at all; from k near the shortest long list's up; crowds right below what is wanted, of
    # whose betters the sample sees none, one or a few (the bins then reach beyond the best of the sample)
    x = W.normal(n, 3 + n % 7)
    for k in (3000, 12000, n // 5):
        for largest in (True, False):
            _check("half the largest sample", x, F32, k, largest, why=0)
    y = np.where(W.uniform01(n, 5) < 0.999, np.float32(1.0), np.float32(2.0) + W.uniform01(n, 6)).astype(np.float32)
    for k in (9000, n // 1000 - 1500):  # (about n / 1000 are better than the crowd)
        for sorted in (True, False):
            _check("few above a crowd", y, F32, k, sorted=sorted, by_list=None)
    _check("few above a crowd", -y, F32, 9000, largest=False, by_list=None)
    z = np.linspace(1.0e6, -1.0e6, n, dtype=np.float32)
    z[W.uniform01(n, 8) < 2.0 ** -11] = np.inf
    _check("ramp", z, F32, 12000, by_list=None)


@pytest.mark.parametrize("n", [13600000, 1 << 24, (1 << 24) + 9])
def test_half_the_largest_sample_has_as_many_runs(n):
    # a ramp's list is a few dozen of the sample's runs long: with as many runs as all of the sample has, half as long, its bins hold what they should; with half
    # as many, some hold several times that, and their buckets are shared out
    for amp in (3.0, 1.0e6):
        x = np.linspace(amp, -amp, n, dtype=np.float32)
        for k in (3000, 12000, 100000):
            for largest in (True, False):
                tr = _check("ramp", x, F32, k, largest)
                assert tr[0].redo == 0, (k, tr[0].redo)


@pytest.mark.parametrize("dtype", [F32, F16])
def test_lists_of_which_half_or_less_is_wanted(dtype):
    # by 256, 512 and 1024 threads, in one round, a few and all eight, either side of half; alone in a bin, two and many to one
    for n, batch in ((1 << 21, 1), (1 << 20, 2), (300000, 58), (259335, 4)):
        x = W.normal(n * batch, n % 11, sigma=2.0)
        y = (np.round(x * 256.0) / 256.0).astype(np.float32)
        for k in (1, 40, 300, 1100, 2200, 3300):
            for sorted in (True, False):
                _check("normal", x, dtype, k, sorted=sorted, batch=batch, by_list=None)
        _check("many equal", y, dtype, 900, largest=False, batch=batch, by_list=None)


@pytest.mark.parametrize("n,k", [(1 << 18, 50000), ((1 << 20) + 1, 20000), ((1 << 22) + 7, 1 << 20)])
def test_buckets_are_filled_from_both_ends(n, k):
    # buckets of a few workgroups and of many; empty ones between crowds; and the last one, of which a part is wanted
    x = W.normal(n, k % 5)
    y = (np.round(x * 8.0) / 8.0).astype(np.float32)
    z = np.where(W.uniform01(n, 2) < 0.9, np.float32(0.999), x).astype(np.float32)
    for dtype in (F32, F16):
        for largest in (True, False):
            _check("normal", x, dtype, k, largest)
            _check("crowds", y, dtype, k, largest, by_list=None)
            _check("nine in ten equal", z, dtype, k, largest, by_list=None)


@pytest.mark.parametrize("dtype,n", [(F32, 40001), (F32, (1 << 19) + 3), (F32, (17 << 17) + 1), (F32, 17 << 17), (F16, (1 << 22) + 3), (BF16, 17 << 18)])
def test_long_lists_of_half_tiles(dtype, n):
    # up to 8.5 MB of a single row, whole and broken last tiles; odd and even numbers of halves for the ties
    x = W.normal(n, n % 13)
    y = np.where(W.uniform01(n, 3) < 0.9, np.float32(0.999), W.uniform01(n, 4)).astype(np.float32)
    z = np.linspace(5.0e4, -5.0e4, n, dtype=np.float32)
    z[W.uniform01(n, 5) < 2.0 ** -11] = np.inf
    for k in (8200, n // 5, n // 4 + 1):
        for largest in (True, False):
            _check("normal", x, dtype, k, largest, by_list=None)
            _check("nine in ten equal", y, dtype, k, largest, by_list=None)
            _check("ramp", z, dtype, k, largest, by_list=None)
    _check("two rows", np.concatenate([x, y]), dtype, n // 5, batch=2, by_list=None)
