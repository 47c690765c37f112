"""Graph construction from pairs, each way the entries are sorted in: that a case goes the way it is for is checked on the host (sort_plan),
the result bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
import sort_plan as sp
from util import dev, host

torch = pytest.importorskip("torch")


def G():
    import paper_2005_03300_amd as g
    return g


FORMS = [(symmetrise, loops) for symmetrise in (False, True) for loops in (False, True)]


def background(rs, n, m, keep_out=None, bucket_rows=0):
    """Random pairs, none of whose ends lies in bucket `keep_out`."""
    src, dst = rs.integers(0, n, m), rs.integers(0, n, m)
    if keep_out is not None:
        for x in (src, dst):
            x[x // bucket_rows == keep_out] = bucket_rows * (keep_out + 2)
    return src, dst


def case(kind, symmetrise, loops):
    """(n, src, dst, what of the plan the case is for)"""
    rs = np.random.default_rng(161)
    n = 1 << 20
    src, dst = background(rs, n, 300_000)
    if kind[3:].isdigit():                       # neighbouring columns of one row, in a bucket whose columns are spread
        k = int(kind[3:])
        src[:k], dst[:k] = 777, 5000 + np.arange(k)
        return n, src, dst, (lambda p: p["digits"] == 0 and 10 < p["ranked"] <= sp.MOST_RANKED) if k == 8000 else (lambda p: p["digits"] == 1)
    if kind == "run_in_piece":                   # the same in a bucket that is cut
        src[:60_000] = 778
        src[60_000:61_500], dst[60_000:61_500] = 779, 400_000 + np.arange(1500)
        return n, src, dst, lambda p: p["digit_pieces"] == 1 and p["pieces"] == 4
    if kind == "most_pieces":                    # nearly as many keys read again as are accepted
        src[:140_000], dst[:140_000] = 780, rs.permutation(n)[:140_000]
        return n, src, dst, lambda p: p["pieces"] >= 7 and (p["read_again"] > 3 or symmetrise or loops)
    if kind == "same":                           # one pair again and again, more often than keys are sorted together
        src[:60_000], dst[:60_000] = 5000, 9000
        return n, src, dst, lambda p: p["crowded"] >= 1
    if kind == "same_each_end":                  # two that fill two pieces each, the bucket's first and last keys
        src[:50_000], dst[:50_000] = 2048 * 9, 0
        src[50_000:100_000], dst[50_000:100_000] = 2048 * 9 + 2047, n - 1
        return n, src, dst, lambda p: p["crowded"] >= 2
    if kind == "same_all_ones":                  # the largest key there is
        n = 1 << 21
        src[:30_000], dst[:30_000] = 2047, n - 1
        return n, src, dst, lambda p: p["crowded"] >= 1
    if kind == "few_again":                      # all keys of one prefix and the first of the next, in no order, beside a run
        src[:60_000], dst[:60_000] = 4000, 8192 + rs.integers(0, 129, 60_000)
        src[60_000:62_000], dst[60_000:62_000] = 3999, 70_000 + np.arange(2000)
        return n, src, dst, lambda p: p["crowded"] >= 1 and p["digit_pieces"] >= 1
    # a bucket of exactly so many keys, all different or each of them two or three times
    size, again = int(kind.split("_")[1]), int(kind.split("_")[2])
    n = 1 << 19
    src, dst = background(rs, n, 300_000, 7, 2048)
    k = size - (2048 if loops else 0)
    distinct = rs.choice(2048 * 300_000, (k + again - 1) // again, replace=False)
    x = np.resize(distinct, k)
    src[:k], dst[:k] = 2048 * 7 + x % 2048, 2048 * 8 + x // 2048
    return n, src, dst, lambda p: (size in p["whole"]) == (size <= sp.CAP) and p["pieces"] == (0 if size <= sp.CAP else 2)


KINDS = ["run1500", "run8000", "run10000", "run_in_piece", "most_pieces", "same", "same_each_end", "same_all_ones", "few_again"]
KINDS += [f"bucket_{sp.CAP + d}_{again}" for d in (-1, 0, 1) for again in (1, 3)]


def the_same(g, n, src, dst, symmetrise, loops):
    for norm, flag in (("sym", g.NORM_SYM), ("none", 0)) if loops else (("row", g.NORM_ROW),):
        flags = flag | (g.SYMMETRISE if symmetrise else 0) | (g.ADD_SELF_LOOPS if loops else 0) | g.BUILD_TRANSPOSE
        a = g.gcn_csr_create(n, dev(src.astype(np.int32)), dev(dst.astype(np.int32)), flags)
        for trans in (False, True):
            ref = oracle.build_csr(n, src, dst, symmetrise=symmetrise, self_loops=loops, norm=norm)
            ref = oracle.transpose(ref) if trans else ref
            rowptr, colidx, val, _ = a.arrays(trans)
            assert np.array_equal(host(rowptr), ref.rowptr) and np.array_equal(host(colidx), ref.colidx), (norm, trans)
            assert np.array_equal(host(val).view(np.uint32), ref.val.view(np.uint32)), (norm, trans)
        a.close()


@pytest.mark.parametrize("symmetrise,loops", FORMS)
@pytest.mark.parametrize("kind", KINDS)
def test_pairs_go_the_way_they_are_for(kind, symmetrise, loops):
    n, src, dst, holds = case(kind, symmetrise, loops)
    p = sp.plan(n, src, dst, symmetrise, loops)
    assert isinstance(p, dict) and holds(p), p


@pytest.mark.gpu
@pytest.mark.parametrize("symmetrise,loops", FORMS)
@pytest.mark.parametrize("kind", KINDS)
def test_crowded_and_full_buckets(kind, symmetrise, loops):
    """Places put in order by ranks and tasks sorted by digits, whole buckets and pieces; prefixes with more keys than are sorted together, of
    which only the distinct ones are wanted; buckets of as many keys as are sorted together, one less and one more."""
    n, src, dst, _ = case(kind, symmetrise, loops)
    the_same(G(), n, src, dst, symmetrise, loops)


def held_per_key(g, n, src, dst):
    """Device memory that a construction without loops asked for, what it keeps for the next one included, in bytes per pair."""
    s, d = dev(src.astype(np.int32)), dev(dst.astype(np.int32))
    g.gcn_csr_create(n, s, d, 0).close()                        # (what loading the kernels takes)
    g.gcn_scratch_release()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    a = g.gcn_csr_create(n, s, d, 0)
    held = free - torch.cuda.mem_get_info()[0]
    a.close()
    g.gcn_scratch_release()
    return held / src.size


@pytest.mark.gpu
def test_a_pair_that_fills_a_piece_is_no_reason_to_sort_again():
    """Two arrays of 32-bit keys (8 bytes per pair), the matrix (8 bytes per entry) and its rows, here a quarter of the entries (4); a second sort, of 64-bit keys,
    would ask for 16 more."""
    rs = np.random.default_rng(162)
    n, m = 1 << 20, 1 << 22
    src, dst = rs.integers(0, n, m), rs.integers(0, n, m)
    src[:60_000], dst[:60_000] = 5000, 9000
    assert sp.plan(n, src, dst, False, False)["crowded"] == 1
    held = held_per_key(G(), n, src, dst)
    assert 16 < held < 27, held


@pytest.mark.gpu
def test_a_refused_construction_reuses_the_keys():
    """Pairs of one vertex, refused after the counting: the radix sort's two arrays of 64-bit keys (16 bytes per pair) and little else, with the
    first attempt's arrays among them."""
    rs = np.random.default_rng(163)
    n, m = 1 << 20, 1 << 23
    src, dst = np.full(m, 3), rs.integers(0, n, m)
    assert sp.plan(n, src, dst, False, False) == "refused"
    held = held_per_key(G(), n, src, dst)
    assert 16 < held < 23, held


def by_keys(kind, extra, symmetrise, loops):
    """Pairs whose entries the radix sort of 64-bit keys orders, `extra` more than whole tiles of it."""
    rs = np.random.default_rng(164)
    if kind == "few_rows":                       # too many keys for a bucket of one row
        n, m = 3, 8 * sp.RS_TILE + extra
        src, dst = rs.integers(0, n, m), rs.integers(0, n, m)
    elif kind == "all_dropped":
        n, m = 2, 8 * sp.RS_TILE + extra
        src = dst = rs.integers(0, n, m)
    else:                                        # "star": refused after the counting
        n, m = 3000, 21 * sp.RS_TILE + extra
        src, dst = np.full(m, n - 1), rs.integers(1000, n, m)
    return n, src, dst


@pytest.mark.parametrize("symmetrise,loops", FORMS)
@pytest.mark.parametrize("extra", [-1, 0, 1])
@pytest.mark.parametrize("kind", ["few_rows", "all_dropped", "star"])
def test_pairs_go_to_the_radix_sort(kind, extra, symmetrise, loops):
    n, src, dst = by_keys(kind, extra, symmetrise, loops)
    assert sp.plan(n, src, dst, symmetrise, loops) == ("refused" if kind == "star" else None)


@pytest.mark.gpu
@pytest.mark.parametrize("symmetrise,loops", FORMS)
@pytest.mark.parametrize("extra", [-1, 0, 1])
@pytest.mark.parametrize("kind", ["few_rows", "all_dropped", "star"])
def test_entries_by_the_radix_sort(kind, extra, symmetrise, loops):
    """The radix sort that reads the pairs, at the edges of its tiles: sizes that the buckets do not take and matrices that they refuse; pairs of
    equal ends, up to all of them; rows without entries at the front; an id outside the range is refused wherever it stands."""
    g = G()
    n, src, dst = by_keys(kind, extra, symmetrise, loops)
    the_same(g, n, src, dst, symmetrise, loops)
    src, dst = src.astype(np.int32), dst.astype(np.int32).copy()
    flags = (g.SYMMETRISE if symmetrise else 0) | (g.ADD_SELF_LOOPS if loops else 0)
    for where, bad in ((0, -1), (src.size - 1, n), (src.size // 2, 2**31 - 1)):
        for arr in (src, dst):
            kept, arr[where] = arr[where], bad
            with pytest.raises(g.GcnError) as e:
                g.gcn_csr_create(n, dev(src), dev(dst), flags)
            assert e.value.code == -2
            arr[where] = kept
