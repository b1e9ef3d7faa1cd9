"""Which form a batch takes: the library's own rules, asked on the host (CPU only)."""
import ctypes
import random

UNITS = 256


def _items(lengths, hq, hkv, tiles):
    return sum(-(-(-(-n // 32) * (hq // hkv)) // tiles) for n in lengths) * hkv


def test_small_packed_batches_have_a_unit_for_every_item(batch_rules):
    """Halved items and loading waves, which leave a unit to one item, are never taken by a batch with more items than units (but loading
    waves by one causal sequence of up to half as many again), whatever its lengths; and they are taken."""
    rng = random.Random(5)
    taken = [0, 0]
    for _ in range(20000):
        hkv = rng.choice([1, 2, 4, 8, 16, 32])
        hq = hkv * rng.choice([1, 2, 4, 6, 7, 8])
        n = rng.choice([1, 1, 2, 3, 4, 6, 8, 10, 16, 33, 64])
        longest = rng.choice([40, 66, 100, 160, 300, 600, 1400])
        lengths = [rng.choice([longest, rng.randint(1, longest), 65]) for _ in range(n)]
        if rng.random() < 0.3:
            lengths = [longest] * n
        total, causal = sum(lengths), rng.random() < 0.5
        d = rng.choice([64, 80, 128])
        if batch_rules.halved_items(d, n, total, hq, hkv, UNITS):
            taken[0] += 1
            assert _items(lengths, hq, hkv, 2) <= UNITS, (lengths, hq, hkv)
        for bound in (max(lengths), 2 * longest):
            if batch_rules.loading_waves(causal, n, total, bound, hq, hkv, UNITS):
                taken[1] += 1
                assert _items(lengths, hq, hkv, 4) <= (UNITS * 3 // 2 if causal and n == 1 else UNITS), (lengths, hq, hkv, causal)
    assert min(taken) > 500, taken
    # one image of 577 tokens, a request of 558; ten sequences of 65 tokens do not fit
    assert batch_rules.halved_items(64, 1, 577, 16, 16, UNITS) and batch_rules.halved_items(128, 1, 558, 28, 4, UNITS)
    assert not batch_rules.halved_items(64, 10, 651, 16, 16, UNITS)
    # sequences of two key tiles that would fill the chip with halves: not at head_dim 128
    assert not batch_rules.halved_items(128, 5, 5 * 66 - 1, 28, 4, UNITS) and batch_rules.halved_items(128, 3, 3 * 66 - 1, 28, 4, UNITS)
    assert batch_rules.halved_items(80, 7, 7 * 66 - 1, 16, 16, UNITS)


def _places(new, group, hkv, splits):
    """Places of a hybrid batch in wide workgroups: chains, and the decode steps' shares."""
    chains = sum(-(-(-(-n // 32) * group) // 4) for n in new if n * group > 32) * hkv
    return chains, sum(1 for n in new if n * group <= 32) * hkv * splits


def test_wide_workgroups_are_bounded_by_what_can_be_there(batch_rules):
    """Eight-wave workgroups of hybrid batches, where requests have any number of new tokens: never with more chains than pay, and with a
    place for each, unless the tokens are to the token those of whole chunks beside decode steps of one."""
    rules = batch_rules.wide_workgroups
    rules.restype = ctypes.c_int64
    rules.argtypes = [ctypes.c_int] * 6 + [ctypes.c_int64]
    rng = random.Random(7)
    taken = 0
    for _ in range(30000):
        hkv, group = rng.choice([(4, 7), (4, 7), (32, 1), (1, 8), (2, 8), (8, 4), (2, 40)])
        n = rng.choice([0, 1, 4, 10, 20, 40, 63, 99])
        k = rng.choice([1, 1, 2, 4, 5, 6, 8, 16])
        longest = rng.choice([40, 100, 300, 512])
        new = [k] * n + [rng.randint(1, longest) for _ in range(rng.randint(0, 6))] + [longest]
        splits, keys = rng.choice([1, 1, 2, 3]), rng.choice([128, 256, 600, 1200])
        workgroups = rules(len(new), sum(new), max(new), group, hkv, splits, keys)
        if workgroups == 0 or (sum(new) - len(new)) % (max(new) - 1) == 0:
            continue
        taken += 1
        chains, steps = _places(new, group, hkv, splits)
        paired = (steps + 1) // 2
        assert chains + paired <= 350 + 1, (new, group, hkv, splits)
        # (numbers of places that are rounded up to multiples of 8, and chains at the end of the grid)
        assert chains + (steps if chains + steps <= UNITS else max(paired, UNITS - chains)) + 16 <= workgroups, (new, group, hkv, splits, workgroups)
    assert taken > 1000
    # drafts being verified beside a chunk, of more chains than their tokens make at first sight; 28 / 4 heads
    for n, k, chunk in ((99, 5, 300), (63, 6, 256), (40, 8, 300), (40, 6, 512)):
        assert rules(n + 1, n * k + chunk, chunk, 7, 4, 1, 1100) == 0
    # under a bound on the new tokens that no request comes near
    assert rules(99, 99 * 5, 512, 7, 4, 1, 700) == 0
    # decode steps and whole chunks; chunks of unequal lengths that fit
    assert rules(60, 56 + 4 * 308, 308, 7, 4, 1, 1712) > 0 and rules(27, 23 + 4 * 158, 158, 7, 4, 1, 916) > 0
    assert rules(6, 393, 200, 7, 4, 1, 864) > 0 and rules(4, 960, 512, 7, 4, 1, 832) > 0
