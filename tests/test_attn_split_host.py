"""The arithmetic of the one-launch attention's split, checked over its whole range on the CPU: what the kernel works
out from the context lengths never exceeds the workgroups launched, the parts and plan records a pool's scratch holds,
or the slots a unit's waves can list - whatever the lengths, heads, table widths and number of compute units."""
import random

UNITS, ROWS, ARRIVE, UNIT_BLOCKS, WAVES, SEQS = 4096, 16384, 4096, 256, 4, 256


def up(x, y):
    return -(-x // y)


def test_every_split_fits_the_launch_and_the_scratch():
    rng = random.Random(1)
    taken = 0
    for _ in range(60000):
        n_cu = rng.choice([32, 64, 128, 256, 304])
        heads, group = rng.choice([1, 2, 3, 4, 8, 12, 16, 32, 40, 64, 300]), rng.choice([1, 2, 3, 4, 7, 8, 16])
        max_batch, max_width = rng.randint(1, 400), int(2 ** rng.uniform(0, 13))
        batch, width = rng.randint(1, min(SEQS, max_batch)), rng.randint(1, max_width)
        # the host: units the call may make
        least, room = batch * up(16 * width, 16 * UNIT_BLOCKS) * heads, min(ROWS // group, UNITS)
        if least > room:
            continue
        units = next((c * n_cu for c in (1, 3, 6, 9, 15) if least <= c * n_cu <= room), room)
        grid = min(batch * up(width, WAVES) * heads, units)
        # the kernel: parts of k quanta (passes of the waves, 64 tokens) and per sequence as equal as quanta allow
        quanta = [max(1, up(rng.choice([0, rng.randint(0, 16 * width), 16 * width]), 16 * WAVES)) for _ in range(batch)]
        max_items, limit = units // heads, UNIT_BLOCKS // WAVES
        k = up(sum(quanta), max_items)
        while k < limit and sum(up(x, k) for x in quanta) > max_items:
            k += 1 + k // 8
        k = min(k, limit)
        items = 0
        for x in quanta:
            each = up(x, up(x, k))
            assert each <= limit                                        # a lane of the slot list per block and wave
            items += up(x, each)
        # the pool's scratch, sized for its largest batch and widest table
        pool_items = min(UNITS // heads + 1, max_batch * up(max_width, WAVES) + 1)
        assert items * heads <= grid                                    # a workgroup for every unit
        assert items * heads * group <= min(pool_items * heads * group, ROWS)   # a partial state for every row
        assert (grid - 1) // heads < pool_items                         # a record for every place, used or not
        assert batch * heads <= min(max_batch * heads, ARRIVE)          # an arrival word for every (sequence, head)
        taken += 1
    assert taken > 5000
