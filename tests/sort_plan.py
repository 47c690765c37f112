"""Which way graph construction sorts the entries of given pairs: a host copy of the rules of csrc/row_sort.h, for tests that must reach each
of them.  Sizes come from the source, so that a case which no longer reaches what it is for fails."""
import os
import re

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2005_03300_amd", "csrc")


def constant(text, name):
    return int(re.search(rf"\b{name} = (\d+)", text).group(1))


ROW_SORT, PRIMS = (open(os.path.join(CSRC, f)).read() for f in ("row_sort.h", "prims.h"))
THREADS, KEYS, MAX_BUCKETS, MAX_SHIFT, BIN_BITS, SHARES = (
    constant(ROW_SORT, c) for c in ("THREADS", "KEYS", "MAX_BUCKETS", "MAX_SHIFT", "BIN_BITS", "SHARES"))
MOST_IN_WINDOW, MOST_BY_RANK, MOST_RANKED, MOST_AGAIN = (
    constant(ROW_SORT, c) for c in ("MOST_IN_WINDOW", "MOST_BY_RANK", "MOST_RANKED", "MOST_AGAIN"))
CAP = KEYS * THREADS
PIECE = CAP // 6 * 5
ROOM = CAP // 100 * 83
RS_TILE = constant(PRIMS, "P_TPB") * constant(PRIMS, "RS_ROUNDS")
for rule in ("PIECE = CAP / 6 * 5;", "ROOM = CAP / 100 * 83;", "(uint64_t)cap * MOST_AGAIN,", "CAP = KEYS * THREADS;"):
    assert rule in ROW_SORT + open(os.path.join(CSRC, "csr_build.hip")).read(), rule


def keys_of(n, src, dst, symmetrise, loops):
    src, dst = np.asarray(src, np.int64), np.asarray(dst, np.int64)
    apart = src != dst
    rows, cols = src[apart], dst[apart]
    if symmetrise:
        rows, cols = np.concatenate([rows, cols]), np.concatenate([cols, rows])
    if loops:
        rows, cols = np.concatenate([rows, np.arange(n)]), np.concatenate([cols, np.arange(n)])
    return rows, cols


def large_places(keys, cbits):
    """Of the sorted keys of a task: (keys, distinct keys) of every place that no window puts in order."""
    row, col = keys >> cbits, keys & ((1 << cbits) - 1)
    low, high = int(col.min()), int(col.max())
    inverse = 0xffffffff // (high - low + 1) if high > low else 0
    _, first, count = np.unique(row, return_index=True, return_counts=True)
    r0, length = np.repeat(first, count), np.repeat(count, count)
    place = r0 + (((col - low) * inverse) * length >> 32)
    at, begin, many = np.unique(place, return_index=True, return_counts=True)
    return [(int(m), np.unique(keys[b:b + m]).size) for b, m in zip(begin, many) if m > MOST_IN_WINDOW]


def plan(n, src, dst, symmetrise, loops):
    """None where the bucket sort does not take the sizes, "refused" where it refuses the buckets, else what its tasks are: sizes of the buckets
    that are not cut, keys that pieces read (of all keys), pieces, pieces with a crowded prefix, tasks sorted by digits (and those of them that are pieces), places put in order
    by ranks."""
    cbits = max(1, int(n - 1).bit_length())
    cap = len(src) * (2 if symmetrise else 1) + (n if loops else 0)
    buckets = lambda s: (n + (1 << s) - 1) >> s
    shift = min(32 - cbits, MAX_SHIFT)
    while shift > 0 and (buckets(shift) < SHARES or cap // buckets(shift) > ROOM):
        shift -= 1
    if cap <= 0 or buckets(shift) > MAX_BUCKETS or cap // buckets(shift) > ROOM:
        return None
    rows, cols = keys_of(n, src, dst, symmetrise, loops)
    bucket = rows >> shift
    keys = (rows & ((1 << shift) - 1)) << cbits | cols
    order = np.lexsort((keys, bucket))
    bucket, keys = bucket[order], keys[order]
    ends = np.searchsorted(bucket, np.arange(buckets(shift) + 1))
    sizes = np.diff(ends)
    parts = np.where(sizes > CAP, (sizes + PIECE - 1) // PIECE, 1)
    again = int((parts * sizes)[parts > 1].sum())
    if again > MOST_AGAIN * cap:
        return "refused"
    d1 = min(shift + cbits, BIN_BITS)
    sh2 = shift + cbits - d1 - min(shift + cbits - d1, BIN_BITS)
    found = dict(whole=set(), read_again=again / cap, pieces=0, crowded=0, digits=0, digit_pieces=0, ranked=0)
    for b in range(buckets(shift)):
        mine = keys[ends[b]:ends[b + 1]]
        prefix = mine >> sh2
        for p in range(parts[b]):
            part = mine
            if parts[b] > 1:
                bound = [0 if w == 0 else int(prefix[w - 1]) + 1 for w in (mine.size * p // int(parts[b]), mine.size * (p + 1) // int(parts[b]))]
                part = mine[np.searchsorted(prefix, bound[0]):np.searchsorted(prefix, bound[1])]
                found["pieces"] += 1
                if part.size > CAP:
                    found["crowded"] += 1
                    last = np.searchsorted(part >> sh2, bound[1] - 1)
                    part = np.concatenate([part[:last], np.unique(part[last:])])
                    assert part.size <= CAP
            else:
                found["whole"].add(mine.size)
            large = large_places(part, cbits) if part.size else []
            by_rank = [m for m, d in large if m > 64 and d > 64]
            if len(by_rank) > MOST_RANKED or any(m > MOST_BY_RANK for m in by_rank):
                found["digits"] += 1
                found["digit_pieces"] += parts[b] > 1
            else:
                found["ranked"] += len(by_rank)
    return found
