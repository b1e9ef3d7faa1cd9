"""Which form a batch takes: the library's own rules, asked on the host (CPU only)."""
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
