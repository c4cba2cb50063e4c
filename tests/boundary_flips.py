"""How far single entries of W_q - W that lie on a bf16 rounding boundary can move a step in its Gram-matrix form (no GPU needed).

The step stores d = W_q - W rounded to bf16.  A float32 evaluation of an entry whose exact value is next to the middle of two bf16
numbers may round the other way than the float64 oracle: one bf16 ulp of d, which on a large input channel is more than the noise
the parity tolerances are made for.  The noise of d: h is one exponential and one quotient, then the interval's product and sum
and the scale's product -- at most four roundings of 2^-24 of W_q -- and the difference with W."""
import numpy as np

from oracle import faar_oracle as fo

UNITS = 4.0


def flips(c, q, V0, beta, alpha):
    """-> (distance of every entry of d to its nearest boundary in units of 2^-24 (|W_q| + |W|), what a flip of it moves the
    loss by, Gm, d's ulp, dV / dG)."""
    sign, lo, hi, s = fo.interval_terms(c.W, q["s_global"], q["scales"])
    h = fo.h_beta(V0.astype(np.float64), beta)
    W = c.W.astype(np.float64)
    Wq = sign * (lo + h * (hi - lo)) * s
    d = Wq - W
    b = fo.bf16_round(d.astype(np.float32)).astype(np.float64)
    ulp = np.where(b != 0.0, 2.0 ** (np.floor(np.log2(np.maximum(np.abs(b), 2.0 ** -126))) - 7), 0.0)
    unit = 2.0 ** -24 * (np.abs(Wq) + np.abs(W))
    with np.errstate(divide="ignore", invalid="ignore"):
        dist = np.where((unit > 0.0) & (ulp > 0.0), (ulp / 2 - np.abs(d - b)) / unit, np.inf)
    X = c.Xq.astype(np.float64)
    Gm = X.T @ X
    G = 2.0 * alpha * (b @ Gm - (c.Y_fp.astype(np.float64) - X @ W.T).T @ X)
    loss = np.abs(G) * ulp + alpha * ulp ** 2 * np.diag(Gm)
    return dist, loss, Gm, ulp, sign * s * (hi - lo) * beta * h * (1.0 - h)


def allowance(c, q, V0, beta, alpha):
    """-> (loss, dV element by element): the most that flips of all entries within UNITS of a boundary change."""
    dist, loss, Gm, ulp, coef = flips(c, q, V0, beta, alpha)
    on = dist <= UNITS
    return float(loss[on].sum()), 2.0 * alpha * (np.where(on, ulp, 0.0) @ np.abs(Gm)) * np.abs(coef)
