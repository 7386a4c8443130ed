"""Shapes of the kernels for long groups, for the GPU tests; that calls on them reach the kernels meant is checked on the
CPU (test_plans.py).  A shape is (B, R, candidate row, reference row, vocabulary, orders)."""

# Dealt positions: shape -> the calls that they serve, of BLEU (b), BLEU with dictionary sizes (d), ROUGE-1 and ROUGE-2.
# (The others go to the sorted runs, the fused kernel or, with 20-bit tokens, the stages.)
DEALT = {
    (3, 1, 20000, 20481, 50257, 4): "bd12",          # 1024 positions a chunk
    (20, 1, 15360, 15361, 50257, 4): "bd12",         # 2048 a chunk; rows that end with one and one behind it
    (20, 2, 10000, 10100, 3000, 4): "bd1",           # counters of 16 bits, two words
    (9, 8, 4097, 4100, 900, 4): "b1",                # five words
    (4, 4, 12100, 9000, 900, 4): "bd12",             # three, also with dictionary sizes and for ROUGE
    (2, 2, 70000, 66000, 1000, 4): "bd12",           # of 32 bits, three words
    (2, 1, 70000, 66000, 2, 4): "bd12",              # sixteen 4-grams: counts beyond 16 bits
    (4, 1, 14000, 14000, (1 << 20) - 2, 4): "12",    # the largest vocabulary, ...
    (4, 1, 14000, 14000, (1 << 20) - 2, 3): "bd12",  # ... and of BLEU with three orders
    (2, 1, 140000, 140000, 1 << 19, 4): "bd12",      # ... and with four
    (5, 2, 9000, 9001, 300, 3): "bd1",
    (5, 3, 9000, 9001, 50257, 2): "bd1",
    (5, 1, 30000, 30000, 50257, 1): "bd12",
    (1, 1, 600, 120000, 500, 4): "bd1",              # candidate much shorter than the reference
    (1, 1, 120000, 600, 500, 4): "bd12",
}

# Sorted runs, BLEU with and without dictionary sizes: shape -> positions per thread of the sorting kernel, counter words
# and whether they have 32 bits.
RUNS = {
    (2, 1, 7000, 7000, 50257, 4): (1, 1, False),
    (8, 1, 9000, 8000, 5000, 5): (2, 1, False),
    (20, 1, 9000, 8000, 5000, 5): (4, 1, False),
    (25, 3, 6000, 6100, 1 << 21, 3): (4, 2, False),
    (1, 1, 100000, 100000, 9000, 5): (2, 2, True),
    (2, 3, 70000, 66000, 2, 4): (4, 4, True),
    (12, 9, 6000, 6000, 131072, 4): (4, 5, False),   # 68 bits
    (6, 9, 6000, 6000, 262144, 4): (4, 5, False),    # 72 bits: part of the table, too
}

# Dealt positions, BLEU: few different tokens, (B, R, row, orders)
FEW_TOKENS = [(2, 1, 60000, 4), (16, 2, 12500, 4), (9, 3, 9000, 4), (4, 1, 30000, 3)]

# (B, R, row, 4-grams behind a beginning, beginnings)
CROWDED = [
    (4, 1, 30000, 1200, 1),     # 784 ids: three shares, by the partition's workgroup alone
    (4, 3, 30000, 900, 2),      # 592 ids
    (4, 1, 30000, 2500, 2),     # more shares, told of
    (2, 3, 30000, 6000, 1),
    (4, 8, 9000, 2000, 1),      # five counter words
    (2, 2, 70000, 3000, 4),     # counters of 32 bits
    (1, 1, 262144, 1500, 1),    # 1936 ids
    (1, 1, 262144, 15000, 3),
]
