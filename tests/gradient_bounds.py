"""Bounds on outputs relative to their own size, for tests where a part of a sum may be lost: against max-abs bounds that are stated for whole workloads the
gradients of a small pack are small themselves."""
import numpy as np

# A value in bf16 mode is off by at most four roundings of 2^-9 each: of the scaled operand of the scores (scores below 2 here), of P or dS for the product,
# of O in delta, of the output (largest seen in the tests that use this: 4.7e-3 in dQ, 3.2e-3 in the others).  In fp32 mode by the rounding of scores, a random
# walk over 128 products that sum to 6 or less: sqrt(128) x 6 x 2^-24 (seen: 1.0e-6).
REL_BF16, REL_F32 = 4 * 2.0 ** -9, 4e-6
ROWS = 32


def worst_block(got, want, floor=0.1):
    """Largest 2-norm of the error over the 2-norm of the result, over blocks of 32 rows of one head ([T, H, d]); a block's norm counts `floor` times the whole
    output's root mean square in each of its elements on top (rows whose exact result is zero: the first row of a sample in dQ).  For dQ the floor is 1: the
    rounding of O reaches a row through delta, 2^-9 of dO . |O| whatever the differences dP - delta are, and a sample's second row can have two keys of nearly the
    same dP (seen: a row of a fortieth of its neighbours' size, off by 5 %)."""
    T, H, d = want.shape
    rms = float(np.sqrt(np.mean(want ** 2)))
    worst = 0.0
    for a in range(0, T, ROWS):
        e, w = (got[a:a + ROWS].astype(np.float64) - want[a:a + ROWS]), want[a:a + ROWS]
        err, size = np.sqrt((e ** 2).sum((0, 2))), np.sqrt((w ** 2).sum((0, 2)))
        worst = max(worst, float(np.max(err / (size + floor * rms * np.sqrt(w.shape[0] * d) + 1e-30))))
    return worst


def relative_error(name, got, want):
    return worst_block(got, want, 1.0 if name == "dQ" else 0.1)
