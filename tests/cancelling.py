"""Inputs whose results are right only if the weights f and p are carried in fp32: the last key's V (K) and the last query's dO
(Q) are chosen so that a weighted sum cancels down to their own rounding, some 2^-9 of its terms; stored in bf16 it is then
known to 2^-18 of them, finer than weights of 16 bits give it."""
import numpy as np

from paper_2410_09397_amd import synth

N, D, SCALE = 3, 96, 96 ** -0.5
# columns 0 .. 31 form the scores; B: K is zero, so that Q is free; C: Q is zero, so that K is free
B, C = slice(32, 64), slice(64, 96)
# error of a sum in fp32 against the sum of the magnitudes of its terms: f and p are off by some 2^-22 (32 products, v_exp_f32, LSE
# rounded to fp32), no more than a few of which add up; 16 bits of a weight are off by up to 2^-18 = 3.8e-6
FP32_SUM = 1.2e-6


def bf16(x):
    return synth.round_to_bf16(np.asarray(x, np.float32)).astype(np.float64)


def inputs(heads, seed):
    """Q, K, V, dO [heads, N, D], O rounded to bf16, LSE rounded to fp32, and the sums that cancel: per name the weights
    [heads, N], the operands [heads, N, columns], bounds on the sizes of the weights' terms, the factor and where the result is."""
    rng = np.random.default_rng(seed)
    Q, K, V, dO = (bf16(rng.standard_normal((heads, N, D))) for _ in range(4))
    K[..., B] = 0
    Q[..., C] = 0
    f = np.exp(SCALE * np.einsum("hik,hjk->hij", Q, K))
    LSE = np.log(f.sum(-1)).astype(np.float32)
    f = np.exp(SCALE * np.einsum("hik,hjk->hij", Q, K) - LSE[..., None])

    def cancel(weights, operand):  # the last row of operand such that sum_t weights_t operand_t is nearly zero
        operand[:, -1] = bf16(-np.einsum("ht,htk->hk", weights[:, :-1], operand[:, :-1]) / weights[:, -1:])

    cancel(f[:, 0, :], V)
    cancel(f[:, :, 0], dO)
    O = bf16(np.einsum("hij,hjk->hik", f, V))
    dP, v = np.einsum("hik,hjk->hij", dO, V), (dO * O).sum(-1)
    p, p_size = f * (dP - v[..., None]), f * (np.abs(dP) + np.abs(v)[..., None])
    for part, weights, operand in ((B, p[:, :, 0], Q), (C, p[:, 0, :], K)):
        last = operand[..., part].copy()
        cancel(weights, last)
        operand[..., part] = last
    sums = {"O": (f[:, 0, :], V, f[:, 0, :], 1.0, slice(None)), "dV": (f[:, :, 0], dO, f[:, :, 0], 1.0, slice(None)),
            "dK": (p[:, :, 0], Q[..., B], p_size[:, :, 0], SCALE, B), "dQ": (p[:, 0, :], K[..., C], p_size[:, 0, :], SCALE, C)}
    return Q, K, V, dO, O, LSE, sums


def expected(sums, name):
    """The result of row 0 [heads, columns] and the largest difference that fp32 arithmetic and one rounding to bf16 leave."""
    w, x, size, factor, _ = sums[name]
    ref = factor * np.einsum("ht,htk->hk", w, x)
    terms = factor * np.einsum("ht,htk->hk", np.abs(size), np.abs(x))
    half_unit = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(ref), 1e-30))) - 8)
    return ref, half_unit + FP32_SUM * terms


def with_parts(sums, name, parts):
    """What the sum is with each weight as the sum of that many bf16 numbers."""
    w, x, _, factor, _ = sums[name]
    rest, total = w.astype(np.float32).astype(np.float64), 0.0
    for _ in range(parts):
        part = bf16(rest)
        total, rest = total + part, rest - part
    return bf16(factor * np.einsum("ht,htk->hk", total, x))
