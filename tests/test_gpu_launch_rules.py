"""Shapes on the far side of the rules that choose a kernel by the size of the call, with lengths that end inside a tile: the small
parity cases of the other files take the kernels for few blocks only.  Checked as the full-size workloads are: the complete forward
of sampled heads and sampled rows of the gradients against the oracle, and identities of the gradients on every head."""
import pytest

from paper_2410_09397_amd import synth
from tests.helpers import check, oracle_reference, to_dev, to_np
from tests.test_gpu_fullsize import check_at_full_size

pytestmark = pytest.mark.gpu

RULES = [
    # large d, product tiles of 256 x 256 in both directions (144 tiles forward, 432 backward); three row blocks, the last with 8 rows
    synth.Workload("wide_products_d512", 81, 1, 24, 520, 512, "bf16"),
    # the same under the causal rule (270 and 810 tiles): tiles of one to nine row blocks, the last with 2 rows
    synth.Workload("wide_products_d512_causal", 82, 1, 15, 2050, 512, "bf16", causal=True),
    # d = 1024 under the causal rule, backward tiles of 256 x 256 in four column blocks (360 and 480), the last row block with 6 rows; heads
    # that the 8 XCDs do and do not divide
    synth.Workload("wide_backward_d1024_causal", 84, 1, 6, 1030, 1024, "bf16", causal=True),
    synth.Workload("wide_backward_d1024_causal_8", 85, 1, 8, 1030, 1024, "bf16", causal=True),
    # 256 x 128 forward (72 tiles), 256 x 256 backward (216), four column tiles
    synth.Workload("wide_backward_d1024", 83, 1, 9, 300, 1024, "bf16"),
]


@pytest.mark.parametrize("w", RULES, ids=lambda w: w.name)
def test_large_calls_of_odd_length(w):
    check_at_full_size(w, w.index)


@pytest.mark.parametrize("causal,heads,n", [(False, 15, 700), (True, 24, 1030), (True, 25, 1030)])
def test_four_phases_at_d_256_with_wide_products(causal, heads, n):
    """One column tile, 135, 360 and 375 tiles of 256 x 256, against float64.  Bound: P, dS, O and the results are rounded to bf16 (2^-9 each),
    sums in fp32: the norm of the difference over that of the result stays below 2^-7."""
    import torch
    from paper_2410_09397_amd import attn
    print("case four phases d256", causal, heads, n, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + heads)
    Q, K, V, dO = (torch.randn((1, heads, n, 256), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4))
    O, LSE = attn.attn_fwd(Q, K, V, 1 / 16, causal=causal)
    grads = attn.attn_bwd(Q, K, V, O, dO, LSE, 1 / 16, causal=causal, tiling=attn.ATTN_BWD_FOUR_PHASE)
    for h in range(heads):
        q, k, v, g = (t[0, h].double() for t in (Q, K, V, dO))
        s = q @ k.T / 16
        if causal:
            s = s.masked_fill(torch.ones(n, n, device="cuda", dtype=torch.bool).triu(1), float("-inf"))
        P = torch.softmax(s, 1)
        dP = g @ v.T
        dS = P * (dP - (P * dP).sum(1, keepdim=True)) / 16
        for name, x, ref in zip(("dQ", "dK", "dV"), grads, (dS @ k, dS.T @ q, P.T @ g)):
            err = float((x[0, h].double() - ref).norm() / ref.norm())
            assert err <= 2.0 ** -7, (name, h, err)


@pytest.mark.parametrize("kind", ["full", "causal", "mask"])
@pytest.mark.parametrize("d", [64, 128])
def test_blocks_of_eight_waves_at_the_edges_of_their_tiles(d, kind):
    """Fused backward of few blocks: two groups of four waves take a block's tiles of 64 in turn, so odd and even numbers of tiles, a last
    tile of one row, and blocks with a single tile (causal, masked) or none (masked) that the second group sits out."""
    import numpy as np
    from paper_2410_09397_amd import attn
    for k, n in enumerate((257, 320, 321, 385, 448)):
        w = synth.Workload("eight_waves_d%d_n%d_%s" % (d, n, kind), 90 + k, 1, 3, n, d, "bf16", causal=kind == "causal", sparse=kind == "mask", extra_frac=0.5)
        print("case", w.name, flush=True)
        inp = synth.make_inputs(w)
        mask = None
        if kind == "mask":
            inp["keep"] = np.asarray(inp["keep"]).copy()
            inp["keep"][:, 1] = inp["keep"][1, :] = False  # a column and a row without a block
            mask = attn.BlockMask(inp["keep"], w.block, n)
        ref = oracle_reference(w, inp)
        Q, K, V, dO = (to_dev(inp[t], "bf16") for t in ("Q", "K", "V", "dO"))
        O_in, LSE_in = to_dev(ref["O_in"], "bf16"), to_dev(ref["LSE_in"], "f32")
        if mask is None:
            grads = attn.attn_bwd(Q, K, V, O_in, dO, LSE_in, w.scale, causal=w.causal)
        else:
            grads = attn.attn_bwd_blocksparse(Q, K, V, O_in, dO, LSE_in, w.scale, mask)
        for name, g, r in zip(("dQ", "dK", "dV"), grads, ref["iso"]):
            check(w.name, name, to_np(g), r, "bf16")


# fp32 arithmetic with the row sums formed in front (past the lines of work that the launch draws), at lengths that end inside a tile and at
# padded head dimensions; 16-byte and 4-byte rows in fp32
ROWS_IN_FRONT = [("f32", 33, 4, 901), ("f32", 80, 2, 1031), ("f32", 77, 2, 1031), ("f32", 128, 3, 517), ("f32", 115, 7, 401),
                 ("bf16", 40, 5, 1001), ("bf16", 96, 3, 1031), ("bf16", 120, 2, 901), ("bf16", 136, 2, 805), ("bf16", 192, 2, 750)]


@pytest.mark.parametrize("dtype,d,heads,n", ROWS_IN_FRONT)
def test_row_sums_in_front_against_the_oracle_and_the_masked_call(dtype, d, heads, n):
    """Against the oracle, and bit for bit against the call with a mask that keeps every block: up to d = 96 (fp32) and everywhere in bf16 that
    one forms the row sums inside.  Then the same with a NaN and an infinite key under the causal rule, whose rows are redone."""
    import numpy as np
    import torch
    from paper_2410_09397_amd import attn
    width = -(-d // 32) * 32
    assert heads * n * n * width >= (1e8 if dtype == "f32" and d > 96 else 2e8 if dtype == "f32" or d > 96 else 3e8)
    w = synth.Workload("rows_in_front_%s_d%d" % (dtype, d), 95, 1, heads, n, d, dtype)
    inp = synth.make_inputs(w)
    ref = oracle_reference(w, inp)
    Q, K, V, dO = (to_dev(inp[t], dtype) for t in ("Q", "K", "V", "dO"))
    O, LSE = to_dev(ref["O_in"], dtype), to_dev(ref["LSE_in"], "f32")
    grads = attn.attn_bwd(Q, K, V, O, dO, LSE, w.scale)
    for name, g, r in zip(("dQ", "dK", "dV"), grads, ref["iso"]):
        check(w.name, name, to_np(g), r, dtype)
    nblk = -(-n // 32)
    full, lower = np.ones((nblk, nblk), np.uint8), np.tril(np.ones((nblk, nblk), np.uint8))
    for g, m in zip(grads, attn.attn_bwd_blocksparse(Q, K, V, O, dO, LSE, w.scale, attn.BlockMask(full, 32, n))):
        assert torch.equal(g, m)
    K[0, 0, n - 40, 1], V[0, heads - 1, n // 2, d - 1] = float("nan"), float("inf")
    O, LSE = attn.attn_fwd(Q, K, V, w.scale, causal=True)
    causal = attn.attn_bwd(Q, K, V, O, dO, LSE, w.scale, causal=True)
    masked = attn.attn_bwd_blocksparse(Q, K, V, O, dO, LSE, w.scale, attn.BlockMask(lower, 32, n), causal=True)
    seen = torch.isfinite(causal[0][0, 0, : n - 40])
    assert seen.all()  # the queries before the NaN key do not see it
    for g, m in zip(causal[1:], masked[1:]):  # (redone rows of dQ add the keys of a list of blocks of 32 in another order)
        assert torch.equal(torch.isnan(g), torch.isnan(m)) and torch.equal(g.nan_to_num(0.0), m.nan_to_num(0.0))


# the same at twice the work, past the lines under the causal rule too, where a call counts for half
CAUSAL_ROWS_IN_FRONT = [("f32", 33, 8, 901), ("f32", 80, 4, 1031), ("f32", 77, 4, 1031), ("f32", 128, 6, 517), ("f32", 115, 14, 401),
                        ("bf16", 40, 10, 1001), ("bf16", 96, 6, 1031), ("bf16", 120, 4, 901), ("bf16", 136, 4, 805), ("bf16", 192, 4, 750)]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype,d,heads,n", CAUSAL_ROWS_IN_FRONT)
def test_row_sums_in_front_of_causal_calls_and_of_keys_that_are_not_finite(dtype, d, heads, n, causal):
    """Against the oracle, and bit for bit against the call with a mask that keeps every block (causal: every one below the diagonal): up to d = 96
    (fp32) and everywhere in bf16 that one forms the row sums inside.  Then the same with a NaN and an infinite key, whose rows are redone."""
    import numpy as np
    import torch
    from paper_2410_09397_amd import attn
    work = heads * n * n * (-(-d // 32) * 32) * (0.5 if causal else 1.0)
    assert work >= (1e8 if dtype == "f32" and d > 96 else 2e8 if dtype == "f32" or d > 96 else 3e8) and heads * n > 2048
    w = synth.Workload("rows_in_front_twice_%s_d%d%s" % (dtype, d, "_causal" if causal else ""), 95, 1, heads, n, d, dtype, causal=causal)
    print("case", w.name, flush=True)
    inp = synth.make_inputs(w)
    ref = oracle_reference(w, inp)
    Q, K, V, dO = (to_dev(inp[t], dtype) for t in ("Q", "K", "V", "dO"))
    O, LSE = to_dev(ref["O_in"], dtype), to_dev(ref["LSE_in"], "f32")
    nblk = -(-n // 32)
    mask = attn.BlockMask(np.tril(np.ones((nblk, nblk), np.uint8)) if causal else np.ones((nblk, nblk), np.uint8), 32, n)

    def both():
        return (attn.attn_bwd(Q, K, V, O, dO, LSE, w.scale, causal=causal), attn.attn_bwd_blocksparse(Q, K, V, O, dO, LSE, w.scale, mask, causal=causal))

    grads, masked = both()
    for name, g, r in zip(("dQ", "dK", "dV"), grads, ref["iso"]):
        check(w.name, name, to_np(g), r, dtype)
    for g, m in zip(grads, masked):
        assert torch.equal(g, m)
    K[0, 0, n - 40, 1], V[0, heads - 1, n // 2, d - 1] = float("nan"), float("inf")
    O, LSE = attn.attn_fwd(Q, K, V, w.scale, causal=causal)
    grads, masked = both()
    assert not all(bool(torch.isfinite(g).all()) for g in grads)
    if causal:
        assert torch.isfinite(grads[0][0, 0, : n - 40]).all()  # the queries before the NaN key do not see it
    for g, m in zip(grads[1:], masked[1:]):  # (redone rows of dQ add the keys of a list of blocks of 32 in another order)
        assert torch.equal(torch.isnan(g), torch.isnan(m)) and torch.equal(g.nan_to_num(0.0), m.nan_to_num(0.0))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,heads,n", [(64, 3, 333), (64, 5, 200), (128, 3, 250), (256, 4, 97), (512, 2, 130)])
def test_a_gradient_in_the_place_of_o(d, heads, n, causal):
    """The memory of O may be that of a gradient: the same bits as with four buffers.  (Calls that otherwise run in one launch, whose key blocks
    read O while others write gradients, and one of the four phases.)"""
    import torch
    from paper_2410_09397_amd import attn
    print("case gradient in the place of O", d, heads, n, causal, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    Q, K, V, dO = (torch.randn((1, heads, n, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4))
    O, LSE = attn.attn_fwd(Q, K, V, d ** -0.5, causal=causal)
    ref = attn.attn_bwd(Q, K, V, O, dO, LSE, d ** -0.5, causal=causal)
    for which in range(3):
        o = O.clone()
        out = [torch.empty_like(O) for _ in range(3)]
        out[which] = o
        attn.attn_bwd(Q, K, V, o, dO, LSE, d ** -0.5, causal=causal, out=tuple(out))
        for x, y in zip(out, ref):
            assert torch.equal(x, y)
