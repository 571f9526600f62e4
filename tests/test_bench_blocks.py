"""Host logic of bench.py for block steps (no GPU): the blocks of a process, the
vector passes the roofline divides by the launch time, and the reductions."""
import bench


def test_blocks_of_a_process():
    assert bench.block_starts(1) == [(0, 1)]
    assert bench.block_starts(3) == [(0, 3)]
    assert bench.block_starts(4) == [(0, 2), (2, 2)]
    assert bench.block_starts(7) == [(0, 2), (2, 3), (5, 2)]
    assert bench.block_starts(8) == [(0, 2), (2, 3), (5, 3)]
    for m in range(1, 65):
        b = bench.block_starts(m)
        assert sum(n for _, n in b) == m and len(b) == -(-m // 3)
        assert all(j + n == k for (j, n), (k, _) in zip(b, b[1:] + [(m, 0)]))


def test_block_vector_passes_by_hand():
    # p = 2, c = 1, one substep of m = 5 (blocks of 2 and 3).  Stage: 3 columns of
    # B read, u written (4).  Column 0 from the state (2).  Block of two from j = 0:
    # inner products and combination read column 0 each (2), B and the field (3),
    # two columns written (2) = 7.  Block of three from j = 2: three columns each
    # (6), 3, three written = 12.  Combine: 5 columns and u (6).  The result (1).
    base = 4 + 2 + 7 + 12 + 6 + 1
    # on chip: the first of three products is written and read twice (3)
    assert bench.block_vectors_per_call([(0.1, 5)], 2, 1, True) == base + 3
    # in memory: a block of two writes 2 products, the second reads the first (1),
    # the passes read 2 each (4), and B and the field once more (3); a block of
    # three 3 written, 2 read by the next product, 3 + 3 by the passes (11), and B
    # and the field twice more (6)
    assert bench.block_vectors_per_call([(0.1, 5)], 2, 1, False) == base + (7 + 3) + (11 + 6)
    # two substeps: stage and result once
    assert bench.block_vectors_per_call([(0.1, 5)] * 2, 2, 1, True) == 5 + 2 * (base + 3 - 5)


def test_reductions_of_a_process():
    assert bench.process_syncs(64) == 22 + 1
    assert bench.process_syncs(40) == 14 + 1
    assert bench.process_syncs(64, "h-gsmgs", "f32") == 65
    assert bench.process_syncs(40, "h-cwy") == 41
    assert bench.process_syncs(4, "mgs") == 2 + 3 + 4 + 5
    assert bench.process_syncs(40, "iocgs") == 80
