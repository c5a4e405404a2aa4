"""Sequence lengths around every tile edge of the kernels (1, 31 ... 257 rows), on each bf16 path and the fp32 one,
dense and causal: forward and isolated backward against the oracle; and properties of the gradients that hold at any
size, checked at the full size of the benchmark workloads where the oracle can only sample rows."""
import numpy as np
import pytest

from paper_2410_09397_amd import synth
from tests.helpers import LSE_TOL, check, oracle_reference, to_dev, to_np

pytestmark = pytest.mark.gpu

EDGE_LENGTHS = (1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 193, 255, 257)


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (256, "bf16"), (512, "bf16"), (40, "f32")])
def test_lengths_around_tile_edges(d, dtype):
    from paper_2410_09397_amd import attn
    for k, n in enumerate(EDGE_LENGTHS):
        for causal in (False, True):
            w = synth.Workload("edge_d%d_n%d%s" % (d, n, "_causal" if causal else ""), 400 + k, 1, 2, n, d, dtype,
                               causal=causal)
            print("case", w.name, flush=True)
            inp = synth.make_inputs(w)
            ref = oracle_reference(w, inp)
            Q, K, V, dO = (to_dev(inp[t], dtype) for t in ("Q", "K", "V", "dO"))
            O, LSE = attn.attn_fwd(Q, K, V, w.scale, causal=causal)
            check(w.name, "O", to_np(O), ref["O"], dtype)
            assert np.abs(to_np(LSE) - ref["LSE"]).max() <= LSE_TOL[dtype] * max(1.0, np.abs(ref["LSE"]).max())
            O_in, LSE_in = to_dev(ref["O_in"], dtype), to_dev(ref["LSE_in"], "f32")
            grads = attn.attn_bwd(Q, K, V, O_in, dO, LSE_in, w.scale, causal=causal)
            for name, g, r in zip(("dQ", "dK", "dV"), grads, ref["iso"]):
                check(w.name + " isolated", name, to_np(g), r, dtype)


@pytest.mark.parametrize("index", [2, 3, 4, 5])
def test_gradient_invariants_at_full_size(index):
    """Rows of f sum to 1 and rows of p sum to 0 (App. B.4), whatever the mask, so for every (batch, head) pair
    the column sums of dV equal those of dO, and <dQ, Q> = <dK, K> (both are scale * sum_ij p_ij s_ij / scale).
    Every element of the three outputs enters these sums (the sampled-row comparison with the oracle in
    test_gpu_fullsize.py sees 40 rows per tensor); observed: 7e-5 .. 1.4e-4 and 4e-6 .. 3e-5."""
    import torch
    from paper_2410_09397_amd import attn
    w = synth.workload(index)
    print("case invariants", w.name, flush=True)
    inp = synth.make_inputs(w)
    Q, K, V, dO = (to_dev(inp[t], w.dtype) for t in ("Q", "K", "V", "dO"))
    mask = attn.BlockMask(inp["keep"], w.block, w.n) if w.sparse else None
    O, LSE = attn.attn_fwd(Q, K, V, w.scale, causal=w.causal, mask=mask)
    if mask is not None:
        dQ, dK, dV = attn.attn_bwd_blocksparse(Q, K, V, O, dO, LSE, w.scale, mask, causal=w.causal)
    else:
        dQ, dK, dV = attn.attn_bwd(Q, K, V, O, dO, LSE, w.scale, causal=w.causal)
    torch.cuda.synchronize()
    f64 = lambda t: t.double()
    # column sums: n terms of unit size each, bf16 outputs -> errors of order 2^-9 * sqrt(n) against sums of order sqrt(n)
    sv, sg = f64(dV).sum(dim=2), f64(dO).sum(dim=2)
    err = float((sv - sg).abs().max() / sg.abs().max())
    print("invariant %s: column sums of dV against dO, max-normalised %.3e" % (w.name, err), flush=True)
    assert err <= 1e-3
    a, b = (f64(dQ) * f64(Q)).sum(dim=(2, 3)), (f64(dK) * f64(K)).sum(dim=(2, 3))
    # the two inner products are sums of n d terms with both signs: compare against the sum of magnitudes
    size = (f64(dQ).abs() * f64(Q).abs()).sum(dim=(2, 3))
    err2 = float(((a - b).abs() / size).max())
    print("invariant %s: <dQ,Q> against <dK,K>, relative to sum |dQ||Q| %.3e" % (w.name, err2), flush=True)
    assert err2 <= 3e-4


@pytest.mark.parametrize("d,bh,n", [(64, 24, 1400), (64, 20, 1000), (128, 24, 1500), (128, 37, 900), (256, 16, 1100), (256, 704, 300)])
def test_causal_block_order_covers_every_block(d, bh, n):
    """Under the causal rule the order in which workgroups take the blocks depends on how many there are (one round of the
    chip, a few, from eight rounds on head after head) and on whether the heads divide over the XCDs.  The order changes no
    arithmetic: with the heads the other way round every head has the same bits, and a call on a head alone (which may take
    blocks of another size) gives the same within the rounding of f, p and the results to bf16."""
    import torch
    from paper_2410_09397_amd import attn
    print("case", d, bh, n, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + bh + n)
    Q, K, V, dO = (torch.randn((1, bh, n, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4))

    def whole(Q, K, V, dO):
        nan = lambda t: torch.full_like(t, float("nan"))
        O, LSE, grads = nan(Q), torch.full((1, Q.shape[1], n), float("nan"), device="cuda"), (nan(Q), nan(Q), nan(Q))
        attn.attn_fwd(Q, K, V, d ** -0.5, causal=True, out=(O, LSE))
        attn.attn_bwd(Q, K, V, O, dO, LSE, d ** -0.5, causal=True, out=grads, tiling=attn.ATTN_BWD_TWO_KERNEL)
        return (O, LSE, *grads)

    out = whole(Q, K, V, dO)
    for t, u in zip(out, whole(*(t.flip(1).contiguous() for t in (Q, K, V, dO)))):
        assert torch.isfinite(t).all()
        assert torch.equal(t.flip(1), u)
    for h in sorted({0, 1, 7, bh // 2, bh - 1}):
        for t, u in zip(out, whole(*(t[:, h:h + 1].contiguous() for t in (Q, K, V, dO)))):
            assert_close_norm(t[:, h:h + 1], u, h)


def assert_close_norm(a, b, what):
    """Two evaluations that differ in the order of their fp32 sums, with f and p rounded to bf16 in between: each is 2.5e-3
    (2-norm) from float64 at most, so twice that lies between them at most; a block that is missing or taken from
    another place is off by the order of one."""
    err = float((a.double() - b.double()).norm() / b.double().norm())
    assert err <= 5e-3, (what, err)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("kind", ["full", "causal", "mask", "causal_mask"])
def test_query_blocks_of_64_and_128_agree(d, kind):
    """A call of few blocks takes query blocks of 64 with the keys split over two waves, a large one blocks of 128: many heads
    in one call against single heads of it, at lengths around the edges of both (the single heads meet the oracle above)."""
    import torch
    from paper_2410_09397_amd import attn
    causal, masked = kind.startswith("causal"), kind.endswith("mask")
    for n in (1, 32, 33, 64, 65, 97, 128, 129, 192, 200, 257, 391):
        blocks = (n + 127) // 128
        heads = (2 if causal and not masked else 1) * (128 if d == 256 else 256) // blocks + 3
        print("case", kind, d, n, heads, flush=True)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(d + n)
        Q, K, V, dO = (torch.randn((1, heads, n, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4))
        keep = np.random.default_rng(n).random((blocks, blocks)) < 0.6
        keep[0, :] = True
        if blocks > 1:
            keep[1, 0] = False  # a list of its own length for each block
        mask = attn.BlockMask(keep, 128, n) if masked else None

        def whole(Q, K, V, dO):
            O, LSE = attn.attn_fwd(Q, K, V, d ** -0.5, causal=causal, mask=mask)
            bwd = attn.attn_bwd if mask is None else attn.attn_bwd_blocksparse
            extra = () if mask is None else (mask,)
            return (O, LSE, *bwd(Q, K, V, O, dO, LSE, d ** -0.5, *extra, causal=causal))

        out = whole(Q, K, V, dO)
        for h in (0, heads // 2, heads - 1):
            for k, (t, u) in enumerate(zip(out, whole(*(t[:, h:h + 1].contiguous() for t in (Q, K, V, dO))))):
                t = t[:, h:h + 1]
                seen = torch.isfinite(u)  # (LSE of a query that sees no key is -inf)
                assert k == 1 or seen.all()
                assert torch.equal(t[~seen], u[~seen])
                if n > 1 or k not in (2, 3):  # (one key: dQ = dK = 0 up to rounding)
                    assert_close_norm(t[seen], u[seen], (n, h, k))


@pytest.mark.parametrize("d,heads,n", [(64, 24, 2000), (128, 16, 4096), (128, 24, 2000), (256, 12, 1990), (256, 16, 2048)])
def test_causal_calls_and_lower_triangular_masks_have_the_same_bits(d, heads, n):
    """Masks only select which tiles are visited: a lower-triangular block mask under the causal rule gives the bits of the causal
    call, also where the number of blocks decides how a kernel shares them out (the sizes lie on both sides of each line)."""
    import torch
    from paper_2410_09397_amd import attn
    print("case", d, heads, n, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + n)
    Q, K, V, dO = (torch.randn((1, heads, n, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4))
    nblk, scale = (n + 127) // 128, d ** -0.5
    mask = attn.BlockMask(np.tril(np.ones((nblk, nblk), np.uint8)), 128, n)
    O, LSE = attn.attn_fwd(Q, K, V, scale, causal=True)
    Om, LSEm = attn.attn_fwd(Q, K, V, scale, causal=True, mask=mask)
    assert torch.equal(O, Om) and torch.equal(LSE, LSEm)
    dense = attn.attn_bwd(Q, K, V, O, dO, LSE, scale, causal=True)
    masked = attn.attn_bwd_blocksparse(Q, K, V, O, dO, LSE, scale, mask, causal=True)
    for a, b in zip(dense, masked):
        assert torch.equal(a, b)


@pytest.mark.parametrize("d,queries", [(64, 64), (128, 64), (256, 64), (256, 128)])
@pytest.mark.parametrize("kind", ["full", "causal", "mask", "causal_mask"])
def test_pipelined_forward_against_float64(d, queries, kind):
    """The pipelined forward (eight waves at d = 64 and 128, query blocks of 64 and of 128 at d = 256) at lengths around its tiles of 64
    and 128 keys and its first and last steps, with a scale whose row maxima move along the row and a negative one."""
    import torch
    from paper_2410_09397_amd import attn
    causal, masked = kind.startswith("causal"), kind.endswith("mask")
    base = 64 if d == 256 else 768
    for i, n in enumerate([base, base + 1, base + 63, base + 65, base + 127, base + 128, base + 193, base + 320] + ([1, 5, 130, 897] if d == 256 else [])):
        nblk = (n + 127) // 128
        # the sides of the line that the launch draws: 64 queries up to 128 blocks of 128 at d = 256; eight waves up to 256 blocks of 64
        heads = 128 // nblk + 3 if queries == 128 else 3
        assert nblk * heads > 128 if queries == 128 else nblk * heads <= 128 and -(-n // 64) * heads <= 256
        scale = (-1 if i % 2 else 1) * (0.5 if i % 3 == 0 else d ** -0.5)
        print("case", kind, d, heads, n, scale, flush=True)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(d + n)
        Q, K, V = (torch.randn((1, heads, n, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
        K *= torch.linspace(0.2, 2.0, n, device="cuda").to(torch.bfloat16)[:, None]  # later keys have larger scores
        keep = np.random.default_rng(n).random((nblk, nblk)) < 0.6
        keep[np.arange(nblk), np.arange(nblk)] = True
        O, LSE = attn.attn_fwd(Q, K, V, scale, causal=causal, mask=attn.BlockMask(keep, 128, n) if masked else None)
        for h in (0, heads // 2, heads - 1):
            s = Q[0, h].double() @ K[0, h].double().T * scale
            if masked:
                s = s.masked_fill(~torch.from_numpy(keep).cuda().repeat_interleave(128, 0).repeat_interleave(128, 1)[:n, :n], float("-inf"))
            if causal:
                s = s.masked_fill(torch.ones(n, n, device="cuda", dtype=torch.bool).triu(1), float("-inf"))
            ref = torch.softmax(s, 1) @ V[0, h].double()
            # f and O are rounded to bf16 (2^-9 each) and the scores' 2^-24 grow with their size
            err = float((O[0, h].double() - ref).norm() / ref.norm())
            assert err <= 5e-3, (n, h, err)
            lse = torch.logsumexp(s, 1)
            # nothing is rounded to bf16 on the way: scores and their sum in fp32
            assert float(((LSE[0, h].double() - lse).abs() / lse.abs().clamp(min=1.0)).max()) <= 1e-5, (n, h)


@pytest.mark.parametrize("d", [512, 1024])
@pytest.mark.parametrize("causal", [False, True])
def test_large_d_forward_with_scores_of_any_size(d, causal):
    """exp(S) is written with a reference per row and chunk of 64 keys: rows of moderate, large positive, large negative and mixed scores,
    in blocks with and without each other, rows whose other chunks vanish beside one, and more than the 16 chunks that
    one thread of a row's sum takes first, with maxima that grow along the row, against float64."""
    import torch
    from paper_2410_09397_amd import attn
    for n in (1, 64, 65, 333, 700, 2100):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(d + n)
        Q, K, V = (torch.randn((1, 3, n, d), generator=gen, device="cuda") for _ in range(3))
        K[0, 2] *= torch.linspace(0.1, 25.0, n, device="cuda")[:, None]      # a reference of its own for every chunk, later ones larger
        Q[0, 0] *= torch.linspace(0.1, 60.0, n, device="cuda")[:, None]      # scores of -250 to 250 in the last rows
        Q[0, 1, n // 2:] = 12.0                                              # rows whose scores are large and of one sign
        K[0, 1] = K[0, 1].abs() * torch.where(torch.arange(n, device="cuda") % 97 < 60, 1.0, -1.0)[:, None]
        Q, K, V = (t.to(torch.bfloat16) for t in (Q, K, V))
        print("case large d scores", d, causal, n, flush=True)
        scale = d ** -0.5
        O, LSE = attn.attn_fwd(Q, K, V, scale, causal=causal)
        for h in range(3):
            s = Q[0, h].double() @ K[0, h].double().T * scale
            if causal:
                s = s.masked_fill(torch.ones(n, n, device="cuda", dtype=torch.bool).triu(1), float("-inf"))
            ref = torch.softmax(s, 1) @ V[0, h].double()
            rows = ((O[0, h].double() - ref).norm(dim=1) / ref.norm(dim=1)).max()
            # per row: f and O are rounded to bf16 (2^-9 each), and scores up to 500 are off by their 2^-22 in fp32 (their sum over d)
            assert float(rows) <= 2.0 ** -7, (n, h, float(rows))
            lse = torch.logsumexp(s, 1)
            assert float(((LSE[0, h].double() - lse).abs() / lse.abs().clamp(min=1.0)).max()) <= 1e-5


@pytest.mark.parametrize("d", [512, 1024])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("score", [16.0, -16.0, 40.0])
def test_large_d_forward_holds_the_range_of_the_values(d, causal, score):
    """Values near both ends of the exponent range with scores far from 0: the weights that meet them sum to about 1, so O is
    finite and keeps its precision wherever exp(S - LSE) V does."""
    import torch
    from paper_2410_09397_amd import attn
    for n in (130, 700, 1300):
        for size in (1e36, 1e-36):
            print("case range of V", d, causal, score, n, size, flush=True)
            gen = torch.Generator(device="cuda")
            gen.manual_seed(d + n)
            Q, K, V = (torch.randn((1, 2, n, d), generator=gen, device="cuda") for _ in range(3))
            Q = 1.0 + 0.1 * Q
            K = score * d ** -0.5 + 0.1 * K  # scores of `score` plus about 0.2
            Q, K, V = Q.to(torch.bfloat16), K.to(torch.bfloat16), (V * size).to(torch.bfloat16)
            O, _ = attn.attn_fwd(Q, K, V, d ** -0.5, causal=causal)
            for h in range(2):
                s = Q[0, h].double() @ K[0, h].double().T * d ** -0.5
                if causal:
                    s = s.masked_fill(torch.ones(n, n, device="cuda", dtype=torch.bool).triu(1), float("-inf"))
                ref = torch.softmax(s, 1) @ (V[0, h].double() / size)
                rows = ((O[0, h].double() / size - ref).norm(dim=1) / ref.norm(dim=1)).max()
                assert float(rows) <= 2.0 ** -7, (n, h, float(rows))  # as above


@pytest.mark.parametrize("d", [512, 1024])
def test_large_d_scores_are_rounded_the_same_in_every_tile(d):
    """The last row sees every key with and without the causal rule, but its last tile takes the body with the bound in one call and
    the body without it in the other: the same scores, so the same bits of O and LSE."""
    import torch
    from paper_2410_09397_amd import attn
    for size in (1.0, 4.0, 8.0):  # standard deviation of the scores
        gen = torch.Generator(device="cuda")
        gen.manual_seed(1)
        Q, K, V = (torch.randn((1, 16384 // d, 512, d), generator=gen, device="cuda") for _ in range(3))
        Q, K, V = ((t * f).to(torch.bfloat16) for t, f in ((Q, size), (K, 1.0), (V, 1.0)))
        print("case rounding of scores", d, size, flush=True)
        full, causal = (attn.attn_fwd(Q, K, V, d ** -0.5, causal=c) for c in (False, True))
        for x, y in zip(full, causal):
            assert torch.equal(x[:, :, -1], y[:, :, -1])


@pytest.mark.parametrize("d", [512, 1024])
@pytest.mark.parametrize("n", [65, 300, 1100])
def test_large_d_forward_shows_keys_that_are_nan(d, n):
    """A chunk of 64 keys that a row sees nothing but NaN of makes the row of O NaN (not 0); rows that do not see it, and other heads,
    keep their bits."""
    import torch
    from paper_2410_09397_amd import attn
    for causal, keys in ((False, slice(0, 64)), (True, slice(0, 64)), (False, slice(64 * ((n - 1) // 64), n)), (True, slice(n - 1, n))):
        print("case nan keys", d, n, causal, keys, flush=True)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(d + n)
        Q, K, V = (torch.randn((1, 2, n, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
        O, LSE = attn.attn_fwd(Q, K, V, d ** -0.5, causal=causal)
        K[0, 0, keys, 3] = float("nan")
        O_nan, LSE_nan = attn.attn_fwd(Q, K, V, d ** -0.5, causal=causal)
        alone = keys.start // 64 * 64 == keys.start  # the rows that see a key of it see none of its chunk that is finite
        first = keys.start if causal else 0
        if alone:  # (the first chunk's own rows have no other weight: no finite sum, a row of zeros)
            rows = O_nan[0, 0, max(first, 64 if causal and keys.start == 0 else 0):]
            assert bool(torch.isnan(rows).all())
        assert torch.equal(O_nan[0, 0, :first], O[0, 0, :first]) and torch.equal(LSE_nan[0, 0, :first], LSE[0, 0, :first])
        assert torch.equal(O_nan[0, 1], O[0, 1]) and torch.equal(LSE_nan[0, 1], LSE[0, 1])


@pytest.mark.parametrize("causal", [False, True])
def test_fp32_head_dimensions_around_the_last_sixteen_columns(causal):
    """fp32 head dimensions on both sides of the width from which the last 16 padded columns are left out, aligned and not,
    against float64 on the GPU."""
    import torch
    from paper_2410_09397_amd import attn
    for d in (1, 15, 16, 17, 32, 65, 72, 79, 80, 81, 96):
        for n in (33, 200):
            print("case fp32 width", causal, d, n, flush=True)
            gen = torch.Generator(device="cuda")
            gen.manual_seed(d + n)
            Q, K, V, dO = (torch.randn((2, 3, n, d), generator=gen, device="cuda") for _ in range(4))
            scale = d ** -0.5
            O, LSE = attn.attn_fwd(Q, K, V, scale, causal=causal)
            grads = attn.attn_bwd(Q, K, V, O, dO, LSE, scale, causal=causal)
            q, k, v, g = (t.double() for t in (Q, K, V, dO))
            s = torch.matmul(q, k.transpose(2, 3).contiguous()) * scale
            if causal:
                s = s.masked_fill(torch.ones(n, n, device="cuda", dtype=torch.bool).triu(1), float("-inf"))
            f = torch.softmax(s, 3)
            o = f @ v
            p = f * (torch.matmul(g, v.transpose(2, 3).contiguous()) - (g * o).sum(3, keepdim=True))
            want = (o, p @ k * scale, torch.matmul(p.transpose(2, 3).contiguous(), q) * scale, torch.matmul(f.transpose(2, 3).contiguous(), g))
            for got, ref in zip((O,) + tuple(grads), want):
                # fp32 sums of n + d terms: the bound that the other fp32 comparisons hold
                assert float((got.double() - ref).abs().max()) <= 3e-6 * max(float(ref.abs().max()), 1.0), (d, n)


def test_current_stream_is_the_one_that_torch_names():
    import torch
    from paper_2410_09397_amd import attn
    assert attn._stream(None) == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert attn._stream(None) == side.cuda_stream
    assert attn._stream(side) == side.cuda_stream
