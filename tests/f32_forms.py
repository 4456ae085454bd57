"""Shapes at which each form of the fp32 projection is planned (checked in
test_host_calls.py), for the GPU tests."""

# name, projected rows of a tile, vocabulary rows of a tile, the workload's overrides, seed
F32_FORMS = [
    # hidden sizes of whole 32-wide chunks, with a tail, of one chunk, and (d % 4 != 0) through 4-byte loads
    ("tile32", 32, 128, dict(B=1, L=40, K=4, d=100, V=32700, n_masked=8), 161),
    ("tile64_odd_d", 64, 128, dict(B=1, L=40, K=3, d=67, V=32661, n_masked=20), 162),
    ("tile96_tail", 96, 128, dict(B=2, L=40, K=3, d=116, V=32641, n_masked=15), 163),
    ("tile128_odd_chunks", 128, 128, dict(B=1, L=64, K=3, d=161, V=32700, n_masked=42), 164),
    ("tile128_two_row_tiles", 128, 128, dict(B=1, L=64, K=4, d=32, V=32650, n_masked=60), 165),
    ("tile64_row_split", 64, 128, dict(B=1, L=400, K=5, d=36, V=1500, n_masked=200), 166),
    ("small", 32, 64, dict(B=1, L=40, K=3, d=97, V=1025, n_masked=33), 167),
]
