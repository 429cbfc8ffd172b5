"""A model of how a merge orders its new paths (csrc/canon.hip: ranks by counting within a block,
ranks among blocks, places, LCPs kept from the previous order), on comparisons that mislead as
colliding prefix hashes make them.  The library may reject an order, never accept a wrong one,
and no search for a chain's parent may start before position 0."""
import random


UNKNOWN = None


def _merge(rng, new, d_old, less, gap, block, left_over, checked):
    """Places of the new paths among the old ones as the kernels leave them: order, LCPs ("kept", a
    kept one; UNKNOWN, to be compared; a number, left over in memory at a place that nobody claimed),
    and whether the order is known to be broken.  Writers of one place come in any order."""
    n, d = len(new), len(new) + d_old
    nb = -(-n // block)
    ids, bgap, gsorted, placed = list(new), [gap[x] for x in new], [UNKNOWN] * n, set()
    order, lcp = list(left_over), [rng.randrange(4) for _ in range(d)]

    def place(rank, x, g):
        gsorted[rank] = g
        order[g + rank], lcp[g + rank] = ("new", x), UNKNOWN
        placed.add(x)

    writes = []
    for j, x in enumerate(new):  # ranks by counting within the block
        b0 = j // block * block
        others = [y for y in new[b0:b0 + block] if y != x]
        rank = sum(gap[y] < gap[x] or (gap[y] == gap[x] and less(y, x)) for y in others)
        writes.append((b0 + rank, x, gap[x]))
    rng.shuffle(writes)
    for at, x, g in writes:
        if nb == 1:
            place(at, x, g)
        else:
            ids[at], bgap[at] = x, g
    if nb > 1:  # ranks among the blocks: by gap, within a gap by path
        writes = []
        for j in range(n):
            x, g, rank = ids[j], bgap[j], j % block
            for b0 in range(0, n, block):
                if b0 == j // block * block:
                    continue
                end = min(b0 + block, n)
                lo, hi = b0, end
                while lo < hi:
                    mid = (lo + hi) // 2
                    lo, hi = (mid + 1, hi) if bgap[mid] < g else (lo, mid)
                if lo < end and bgap[lo] == g:
                    top, hi = lo, end
                    while top < hi:
                        mid = (top + hi) // 2
                        top, hi = (mid + 1, hi) if bgap[mid] <= g else (top, mid)
                    hi = top
                    while lo < hi:
                        mid = (lo + hi) // 2
                        lo, hi = (mid + 1, hi) if less(ids[mid], x) else (lo, mid)
                rank += lo - b0
            writes.append((rank, x, g))
        rng.shuffle(writes)
        for w in writes:
            place(*w)
    broken = any(g is UNKNOWN for g in gsorted)
    if checked:
        broken |= len(placed) < n or any(a is UNKNOWN or b is UNKNOWN or a > b for a, b in zip(gsorted, gsorted[1:]))
    for i in range(d_old):
        lo, hi = 0, n
        while lo < hi:
            mid = (lo + hi) // 2
            lo, hi = (mid + 1, hi) if gsorted[mid] is not UNKNOWN and gsorted[mid] <= i else (lo, mid)
        order[i + lo] = ("old", i)
        lcp[i + lo] = "kept" if i > 0 and not (lo > 0 and gsorted[lo - 1] == i) else UNKNOWN
    return order, lcp, broken


def _trial(seed, checked=True):
    """(order the host would accept or None, the true order, a chain's parent searched before
    position 0); checked: what the kernels check, against looking for ranks that
    no path took and taking every LCP below kInf as kept."""
    rng = random.Random(seed)
    d_old, n, block = rng.randrange(1, 7), rng.randrange(1, 13), rng.choice([4, 8])
    cut = [rng.randrange(d_old + 1) for _ in range(n)]  # old paths before each new one
    cut.sort()
    truth = sorted([(i, "old", i) for i in range(d_old)] + [(g - 0.5, "new", x) for x, g in enumerate(cut)])
    truth = [p[1:] for p in truth]
    rank = {p: k for k, p in enumerate(truth)}
    lies = {}  # pairs that the hashes mislead: the wrong way round, or neither before the other
    for x in range(n):
        for y in range(x + 1, n):
            if rng.random() < 0.15:
                lies[x, y] = rng.choice([(False, True), (False, False)])

    def less(x, y):
        if x == y:
            return False
        v = lies.get((min(x, y), max(x, y)), (True, False))
        return v[0] if x < y else v[1]

    new = list(range(n))
    rng.shuffle(new)
    # the memory of the order holds another order of the paths (a buffer of an earlier merge), or nothing
    left_over = [p if rng.random() < 0.95 else rng.choice(truth + [None]) for p in truth]
    order, lcp, broken = _merge(rng, new, d_old, less, cut, block, left_over, checked)
    # the exact pass: entries that are no path raise the flag and read as path 0
    kept = [v is not UNKNOWN and not (checked and (broken or i == 0)) for i, v in enumerate(lcp)]
    before0 = kept[0] and lcp[0] != 0
    for i, p in enumerate(order):
        broken |= p not in rank
        if i > 0 and not kept[i]:
            broken |= rank.get(order[i - 1], 0) >= rank.get(p, 0)
    return (None if broken else order), truth, before0


def test_no_parent_is_searched_before_the_first_position():
    assert any(_trial(seed, checked=False)[2] for seed in range(3000))  # (the model gets there)
    assert not any(_trial(seed)[2] for seed in range(20000))


def test_no_wrong_order_is_accepted():
    wrong = [seed for seed in range(20000) for o, truth, _ in [_trial(seed, checked=False)] if o not in (None, truth)]
    assert len(wrong) > 5  # (lost paths go unnoticed without the checks)
    accepted = 0
    for seed in list(range(20000)) + wrong:
        o, truth, _ = _trial(seed)
        assert o in (None, truth), seed
        accepted += o is not None
    assert accepted > 5000
