"""Cases of the split channel products (inputs only), shared by their CPU and GPU tests.

Output multiplicities at the edges of the kernels' column tiles (16, 32, 64 and 128 wide, one tile
partly filled or two tiles), reductions that are no multiple of the 32-deep step, row counts on both
sides of the 128-row block, and enough few-row groups that the reduction is shared out.
"""

from tests.cases import make_case

# (irreps in, lmax, irreps out, K, nodes, edges)
CASES = [
    ("8x0e+8x1o", 1, "8x0e+4x1o", 4, 43, 500),        # 4 and 8 columns; 43 and 129 rows
    ("20x0e+12x1o", 1, "36x0e+72x1o", 5, 42, 300),    # 36 of 64 and 72 of 128 columns; 160-deep; 126 rows
    ("8x0e", 1, "132x0e+4x1o+100x1o", 8, 60, 300),    # two tiles of 128, and the wide adjoint-state kernel
    ("12x0e", 0, "16x0e", 3, 129, 700),               # 36-deep reduction
]
IDS = [f"{c[2]}-{c[4]}" for c in CASES]

# Three bf16 parts leave 2^-25 of an operand and six products 3 x 2^-25 of a term, and a 32-deep step
# adds one fp32 rounding: sums of n terms stay within a few sqrt(n) 2^-24 of their norm.  The longest
# reductions here have n = 1152 terms; 5e-6 of the largest output is eight times sqrt(n) 2^-24 / 3.
TOL = 5e-6


def case(i):
    a, lmax, c, K, N, E = CASES[i]
    return make_case((a, lmax, c, K), N, E, 300 + i)
