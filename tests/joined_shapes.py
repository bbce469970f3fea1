"""Backward calls whose dK/dV stages hold the rows of several heads one behind the other.  The GPU tests take them, and the host checks
assert that the rules still plan them so, with every form of the kernel among them."""

# (batch, query heads, KV heads, chunk rows, first row)
DENSE = [
    (1, 4, 2, 1, 64),          # one row of two heads; a column tile that starts at it
    (2, 8, 2, 5, 123),         # a stage of all four heads' rows, and 44 that do not exist
    (1, 8, 1, 16, 240),        # heads that end with the stages
    (2, 16, 4, 32, 96),
    (1, 16, 2, 21, 4100),      # a stage and its half end inside heads; the last stage 40 rows
    (1, 16, 2, 31, 4194),      # heads shorter than the 32 rows of a block of scores, on the diagonal
    (1, 16, 2, 40, 4300),      # a head's end in one block of a stage, in either or in the same one
    (2, 24, 8, 36, 1500),      # three heads
    (1, 32, 8, 66, 1100),      # a head's rows longer than a stage
    (1, 16, 2, 70, 4284),      # the last column tile sees the last six rows of each head
    (1, 32, 4, 86, 2621),
    (1, 16, 4, 70, 8195),      # column tiles shared out, a share's first stage behind a head's end
    (1, 32, 8, 19, 8300),      # several rounds of column tiles
    (1, 24, 8, 6, 3610),       # dK/dV by itself, 16x16x32 products
    (1, 32, 8, 150, 16000),    # likewise, 22 rows of each head in the last column tile
    (1, 32, 8, 199, 8127),     # likewise, column tiles of the last round shared out
    (1, 64, 8, 70, 2500),      # by itself, 32x32x16 products
    (2, 64, 8, 71, 1211),
]
# (batch, query heads, KV heads, chunk rows, first row, later rows): the transposed order, whose query rows are the chunk's and the later ones
GATHER = [
    (1, 8, 1, 16, 64, 0),
    (1, 16, 2, 9, 23, 7),
    (16, 32, 2, 130, 0, 0),    # the second column tile sees the last two rows of each head
]
# (batch, query heads, KV heads, chunk rows, chunks, selected chunks): dQ over the selected chunks, dK/dV over all
SELECTED = [
    (1, 8, 1, 16, 16, [3, 9]),           # whole row tiles
    (1, 8, 2, 32, 20, [3, 12]),
    (1, 32, 8, 19, 60, [0, 7, 8, 41, 58]),
    (2, 16, 2, 21, 100, [5, 6, 7, 80]),
    (1, 16, 2, 40, 104, [1, 100]),
]
# (batch, query heads, KV heads, chunk rows, chunks, {chunk: weight}): dK/dV over the chunks of the table, each with its weight
WEIGHTED = [
    (1, 8, 2, 32, 12, {1: 2.5, 2: 2.5, 7: -0.5, 11: 1.0}),
    (2, 16, 2, 5, 30, {0: 3.0, 17: 1.5, 29: 1.0}),
    (1, 16, 2, 40, 80, {**{i: 1.0 + i / 16 for i in range(2, 76, 2)}, 79: 1.0}),
]


def arguments():
    """The calls as the host checks take them: one word each, with its kind."""
    join = lambda kind, *v: kind + ":" + ",".join(map(str, v))
    return ([join("d", *s) for s in DENSE] + [join("g", *s) for s in GATHER] +
            [join(kind, *s[:5], *s[5]) for kind, calls in (("s", SELECTED), ("w", WEIGHTED)) for s in calls])
