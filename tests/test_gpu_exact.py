"""The fp32-arithmetic matrix-core kernels (fp32 tensors, bf16 tensors of any head dimension, block masks whose edge is a
multiple of the rows that a workgroup owns: 32 for bf16 up to d = 128, else 16) at the edges of their tiles: head dimensions on
both sides of every padded width, including those that are no multiple of 4 (fp32), and lengths around 16- and 32-row steps and
the turns of the eight waves that a workgroup has in calls of this size; larger calls, with four waves, further down, and with
them the FMA kernels that take the rest (here: bf16 d = 128 under blocks of 16).

Bounds: fp32 arithmetic on both storage types, so the error is that of sums of at most n + d terms in fp32, about
sqrt(n + d) 2^-24 = 1.5e-6 of the largest value at the sizes here (fp32 storage: the regression bound of tests/helpers, 3e-6); with
bf16 storage one rounding of the result comes on top: 8 significant bits, half a unit in the last place of a value just
above a power of two, 2^-8 of it at most."""
import numpy as np
import pytest

from paper_2410_09397_amd import synth
from tests.helpers import LSE_TOL, check, oracle_reference, to_dev, to_np

pytestmark = pytest.mark.gpu

BF16_BOUND = 2.0 ** -8 + 1e-5


def W(b, h, n, d, dtype, **kw):
    name = "exact_%s_d%d_n%d%s%s" % (dtype, d, n, "_causal" if kw.get("causal") else "", "_b%d" % kw["block"] if kw.get("sparse") else "")
    return synth.Workload(name, 500 + d, b, h, n, d, dtype, **kw)


CASES = (
    [W(1, 2, n, d, "f32", causal=c) for d, n in ((1, 17), (3, 64), (31, 65), (32, 16), (33, 127), (64, 33), (66, 129), (95, 200),
                                                (96, 1), (97, 63), (126, 130), (128, 257)) for c in (False, True)]
    + [W(1, 2, n, d, "bf16", causal=c) for d, n in ((8, 31), (32, 33), (40, 128), (56, 129), (72, 64), (96, 257), (120, 1),
                                                   (136, 95), (192, 130), (200, 65), (248, 127)) for c in (False, True)]
    + [W(1, 2, 300, 64, "bf16", sparse=True, block=64, extra_frac=0.4), W(2, 2, 500, 128, "bf16", sparse=True, block=16, extra_frac=0.2, causal=True),
       W(1, 2, 333, 256, "bf16", sparse=True, block=48, extra_frac=0.3), W(1, 3, 777, 80, "f32", sparse=True, block=32, extra_frac=0.2, causal=True,
                                                                        per_head_masks=True),
       W(1, 1, 400, 128, "f32", sparse=True, block=80, extra_frac=0.5)])


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_fp32_arithmetic_at_tile_edges(w):
    from paper_2410_09397_amd import attn
    print("case", w, flush=True)
    inp = synth.make_inputs(w)
    ref = oracle_reference(w, inp)
    tol = 3e-6 if w.dtype == "f32" else BF16_BOUND
    Q, K, V, dO = (to_dev(inp[t], w.dtype) for t in ("Q", "K", "V", "dO"))
    mask = attn.BlockMask(inp["keep"], w.block, w.n) if w.sparse else None
    O, LSE = attn.attn_fwd(Q, K, V, w.scale, causal=w.causal, mask=mask)
    check(w.name, "O", to_np(O), ref["O"], w.dtype, tol=tol)
    assert np.abs(to_np(LSE) - ref["LSE"]).max() <= LSE_TOL["f32"] * max(1.0, np.abs(ref["LSE"]).max())
    O_in, LSE_in = to_dev(ref["O_in"], w.dtype), to_dev(ref["LSE_in"], "f32")
    if mask is not None:
        grads = attn.attn_bwd_blocksparse(Q, K, V, O_in, dO, LSE_in, w.scale, mask, causal=w.causal)
    else:
        grads = attn.attn_bwd(Q, K, V, O_in, dO, LSE_in, w.scale, causal=w.causal)
    for name, g, r in zip(("dQ", "dK", "dV"), grads, ref["iso"]):
        if np.abs(r).max() > 0:  # a single row has dQ = dK = 0 up to rounding
            den = max(np.abs(r).max(), 1e-3)
            assert np.abs(to_np(g) - r).max() <= tol * den, (w.name, name, np.abs(to_np(g) - r).max() / den)


ROW_CASES = (
    [W(1, 2, n, d, "f32", causal=c) for d, n in ((129, 65), (130, 64), (200, 130), (257, 1), (509, 63), (512, 127)) for c in (False, True)]
    + [W(1, 2, n, d, "bf16", causal=c) for d, n in ((264, 65), (384, 130), (504, 3)) for c in (False, True)]
    + [W(1, 2, 300, d, dtype, sparse=True, block=b, extra_frac=0.3, causal=c)
       for d, dtype, b in ((40, "f32", 24), (128, "f32", 100), (130, "f32", 16), (200, "f32", 65), (64, "bf16", 24), (128, "bf16", 16),
                           (96, "bf16", 48), (256, "bf16", 100), (512, "bf16", 128)) for c in (False, True)]
    + [W(2, 2, 200, 100, "f32", sparse=True, block=7, extra_frac=0.2, causal=True, per_head_masks=True)])


@pytest.mark.parametrize("w", ROW_CASES, ids=lambda w: w.name)
def test_row_kernels(w):
    """What the matrix-core kernels do not take (head dimensions beyond theirs, mask edges that are no multiple of the rows that a
    workgroup owns) runs on the row-per-wave FMA kernels: head dimensions around the widths that they are built for."""
    test_fp32_arithmetic_at_tile_edges(w)


@pytest.mark.parametrize("d,dtype,n", [(80, "f32", 100), (64, "f32", 49), (30, "f32", 77), (96, "bf16", 100), (72, "bf16", 47), (200, "bf16", 81)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_invisible_rows_do_not_reach_results(d, dtype, n, value):
    """Under the causal rule the results of a query depend on no later key, whatever it holds, and those of a key on no
    earlier query: with the last keys (queries) not finite the others are what they are without."""
    import torch
    from paper_2410_09397_amd import attn
    print("case", d, dtype, n, value, flush=True)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + n)
    Q, K, V, dO = (torch.randn((1, 2, n, d), generator=gen, device="cuda").to(t) for _ in range(4))
    scale, cut = d ** -0.5, n - 5
    O, LSE = attn.attn_fwd(Q, K, V, scale, causal=True)
    dQ, dK, dV = attn.attn_bwd(Q, K, V, O, dO, LSE, scale, causal=True)
    K2, V2 = K.clone(), V.clone()
    K2[:, :, cut:] = value
    V2[:, :, cut:] = value
    O2, LSE2 = attn.attn_fwd(Q, K2, V2, scale, causal=True)
    dQ2, _, _ = attn.attn_bwd(Q, K2, V2, O, dO, LSE, scale, causal=True)
    bound = 3e-6 if dtype == "f32" else 2 * BF16_BOUND  # two results, each rounded once
    for a, b in ((O2, O), (LSE2, LSE), (dQ2, dQ)):
        a, b = a[:, :, :cut].float(), b[:, :, :cut].float()
        assert torch.isfinite(a).all()
        assert (a - b).abs().max() <= bound * max(1.0, float(b.abs().max()))
    assert not torch.isfinite(O2[:, :, cut:].float()).any()
    # a bias of minus infinity in the first column leaves a key without weight
    K3 = K.clone()
    Q3 = Q.clone()
    Q3[..., 0] = 1.0
    K3[:, :, 1, 0] = -float("inf")
    got = attn.attn_fwd(Q3, K3, V, scale, causal=True)[0].double()
    s = (Q3.double() @ K3.double().transpose(-1, -2).contiguous()) * scale
    s = s.masked_fill(torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1), -float("inf"))
    want = torch.softmax(s, -1) @ V.double()
    assert (got - want).abs().max() <= bound * float(want.abs().max())


@pytest.mark.parametrize("d,n", [(64, 100), (80, 49)])
def test_fp32_tensors_that_start_on_4_bytes(d, n):
    """fp32 tensors need no alignment beyond their own: the results are those of aligned copies."""
    import torch
    from paper_2410_09397_amd import attn
    print("case", d, n, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + n)
    aligned = [torch.randn((1, 2, n, d), generator=gen, device="cuda") for _ in range(4)]

    def shifted(t):
        return torch.cat([t.new_zeros(1), t.flatten()])[1:].view(t.shape)

    def both(Q, K, V, dO, like):
        O, LSE, grads = like(Q), torch.empty((1, 2, n), device="cuda"), tuple(like(t) for t in (Q, K, V))
        attn.attn_fwd(Q, K, V, d ** -0.5, causal=True, out=(O, LSE))
        attn.attn_bwd(Q, K, V, O, dO, LSE, d ** -0.5, causal=True, out=grads)
        return (O, LSE) + grads

    moved = [shifted(t) for t in aligned]
    assert all(t.data_ptr() % 16 == 4 for t in moved)
    for a, b in zip(both(*moved, shifted), both(*aligned, torch.empty_like)):
        assert (a - b).abs().max() <= 3e-6 * max(1.0, float(b.abs().max()))


@pytest.mark.parametrize("d,dtype,n", [(80, "f32", 100), (30, "f32", 77), (130, "f32", 100), (96, "bf16", 100), (200, "bf16", 81)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_invisible_queries_do_not_reach_key_gradients(d, dtype, n, value):
    """Under the causal rule dK and dV of a key depend on no earlier query, whatever Q, O and dO hold there; d = 130: the
    row-per-wave kernels."""
    import torch
    from paper_2410_09397_amd import attn
    print("case", d, dtype, n, value, flush=True)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + n)
    Q, K, V, dO = (torch.randn((1, 2, n, d), generator=gen, device="cuda").to(t) for _ in range(4))
    scale, cut = d ** -0.5, 5
    O, LSE = attn.attn_fwd(Q, K, V, scale, causal=True)
    _, dK, dV = attn.attn_bwd(Q, K, V, O, dO, LSE, scale, causal=True)
    Q2, dO2 = Q.clone(), dO.clone()
    Q2[:, :, :cut] = value
    dO2[:, :, :cut] = value
    _, dK2, dV2 = attn.attn_bwd(Q2, K, V, O, dO2, LSE, scale, causal=True)
    bound = 3e-6 if dtype == "f32" else 2 * BF16_BOUND  # two results, each rounded once
    for a, b in ((dK2, dK), (dV2, dV)):
        assert not torch.isfinite(a[:, :, :cut].float()).any()
        a, b = a[:, :, cut:].float(), b[:, :, cut:].float()
        assert torch.isfinite(a).all()
        assert (a - b).abs().max() <= bound * max(1.0, float(b.abs().max()))


@pytest.mark.parametrize("dtype,d,n,heads", [("f32", 128, 512, 8), ("bf16", 192, 512, 8)])
def test_steps_that_are_not_finite_take_a_few_finite_ones(dtype, d, n, heads):
    """A step that diverged (every value NaN) redoes its rows one by one, which ends with the first rows that it meets: it
    takes 2.6 (fp32) and 3 (bf16) times what a finite one takes; with every row summed to its end it was 15 and 30."""
    import torch
    from paper_2410_09397_amd import attn
    t = torch.float32 if dtype == "f32" else torch.bfloat16

    def step_us(tensors):
        Q, K, V, dO = tensors
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            O, LSE = attn.attn_fwd(Q, K, V, d ** -0.5)
            grads = attn.attn_bwd(Q, K, V, O, dO, LSE, d ** -0.5)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 1e3)
        return sorted(times)[3], grads

    finite, _ = step_us([torch.randn((1, heads, n, d), device="cuda").to(t) for _ in range(4)])
    nan, out = step_us([torch.full((1, heads, n, d), float("nan"), device="cuda", dtype=t) for _ in range(4)])
    print("step us, finite %.1f, NaN %.1f" % (finite, nan), flush=True)
    assert torch.isnan(out[1]).all() and torch.isnan(out[2]).all()
    assert nan <= 8 * finite


def reference(Q, K, V, dO, scale, causal, O_in=None):
    """O, LSE, dQ, dK, dV in float64, without a mask; the gradients with the O that the backward is given."""
    import torch
    Q, K, V, dO = (t.double() for t in (Q, K, V, dO))
    s = scale * (Q @ K.transpose(-1, -2).contiguous())
    if causal:
        s = s.masked_fill(torch.ones(s.shape[-2:], dtype=torch.bool, device=s.device).triu(1), -float("inf"))
    LSE = torch.logsumexp(s, -1)
    f = torch.exp(s - LSE[..., None])
    O = f @ V
    p = f * (dO @ V.transpose(-1, -2).contiguous() - ((O if O_in is None else O_in.double()) * dO).sum(-1, keepdim=True))
    t = lambda x: x.transpose(-1, -2).contiguous()
    return O, LSE, scale * (p @ K), scale * (t(p) @ Q), t(f) @ dO


def check_reference(case, out, ref, dtype):
    tol = 3e-6 if dtype == "f32" else BF16_BOUND
    for name, x, r in zip(("O", "LSE", "dQ", "dK", "dV"), out, ref):
        assert (x.double() - r).abs().max() <= (3e-6 if name == "LSE" else tol) * max(1.0, float(r.abs().max())), (case, name)


def check_call(dtype, d, h, n, causal, gen):
    """Forward, and backward on the rounded O and LSE, into outputs that hold NaN, against float64."""
    import torch
    from paper_2410_09397_amd import attn
    t, scale = torch.float32 if dtype == "f32" else torch.bfloat16, d ** -0.5
    Q, K, V, dO = (torch.randn((1, h, n, d), generator=gen, device="cuda").to(t) for _ in range(4))
    nan = lambda: torch.full_like(Q, float("nan"))
    O, LSE, grads = nan(), torch.full((1, h, n), float("nan"), device="cuda"), (nan(), nan(), nan())
    attn.attn_fwd(Q, K, V, scale, causal=causal, out=(O, LSE))
    ref = reference(Q, K, V, dO, scale, causal)
    O_in = ref[0].to(t)
    attn.attn_bwd(Q, K, V, O_in, dO, ref[1].float(), scale, causal=causal, out=grads)
    check_reference((dtype, d, h, n, causal), (O, LSE) + grads, ref[:2] + reference(Q, K, V, dO, scale, causal, O_in)[2:], dtype)


# heads and rows on both sides of the line between the row kernels and the matrix-core kernels, and of where they meet in
# one step (the backward has a line of its own)
@pytest.mark.parametrize("dtype,d,heads,rows", [("f32", 64, (1535, 1536), (1, 2, 3)), ("f32", 17, (3071, 3072), (2, 3)), ("f32", 128, (767, 768), (2, 6, 7)),
                                                ("bf16", 32, (2047, 2048), (4, 5)), ("bf16", 96, (682, 683), (4, 6, 7)), ("bf16", 192, (341, 342), (6, 7))])
@pytest.mark.parametrize("causal", [False, True])
def test_few_rows_in_many_heads(dtype, d, heads, rows, causal):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    for h in heads:
        for n in rows:
            print("case", dtype, d, h, n, causal, flush=True)
            check_call(dtype, d, h, n, causal, gen)


def test_more_heads_than_one_launch_has_workgroups_for():
    """2^23 heads of three rows: one workgroup of 256 threads per head and role would be 2^32 threads, which no launch has."""
    import torch
    from paper_2410_09397_amd import attn
    print("case 2^23 heads", flush=True)
    Q, K, V, dO = (torch.randn((4, 2 ** 21, 3, 1), device="cuda") for _ in range(4))
    O, LSE = attn.attn_fwd(Q, K, V, 1.0, causal=True)
    grads = attn.attn_bwd(Q, K, V, O, dO, LSE, 1.0, causal=True)
    check_reference("2^23 heads", (O, LSE) + grads, reference(Q, K, V, dO, 1.0, True), "f32")


@pytest.mark.parametrize("dtype,d", [("f32", 30), ("f32", 64), ("f32", 80), ("f32", 128), ("bf16", 32), ("bf16", 40), ("bf16", 96), ("bf16", 160)])
@pytest.mark.parametrize("causal", [False, True])
def test_more_than_two_workgroups_per_cu(dtype, d, causal):
    """From 513 workgroups on they have four waves instead of eight, and causal ones come in rounds of 256, every second one
    reversed: a second full round and one that is not full, in the forward (the backward has twice as many), and several."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    per_head = -(-200 // (32 if dtype == "bf16" and d <= 128 else 16))
    for blocks in (520, 1300):
        h = -(-blocks // per_head)
        print("case", dtype, d, h, causal, flush=True)
        check_call(dtype, d, h, 200, causal, gen)


@pytest.mark.parametrize("d,block,n,heads", [(64, 32, 300, 3), (128, 32, 200, 3), (128, 96, 500, 40)])
@pytest.mark.parametrize("causal", [False, True])
def test_bf16_mask_blocks_that_are_multiples_of_32(d, block, n, heads, causal):
    """Up to d = 128 a bf16 workgroup owns 32 rows, which a mask edge may not cut."""
    test_fp32_arithmetic_at_tile_edges(W(1, heads, n, d, "bf16", sparse=True, block=block, extra_frac=0.3, causal=causal))


@pytest.mark.parametrize("d", [96, 192])
def test_weights_are_carried_in_full(d):
    """Sums that cancel to 2^-9 of their terms: weights of 16 bits are four bounds off, of 8 bits thousands (tests/test_cancelling.py).
    96 columns as they are, and with as many zero ones behind them, where a workgroup owns 16 rows instead of 32."""
    import torch
    from paper_2410_09397_amd import attn
    from tests import cancelling
    Q, K, V, dO, O_in, LSE, sums = cancelling.inputs(64, 7)

    def dev(x):
        return to_dev(np.concatenate([x, np.zeros(x.shape[:2] + (d - cancelling.D,))], axis=2)[None], "bf16")

    Q, K, V, dO, O_in = (dev(x) for x in (Q, K, V, dO, O_in))
    got = {"O": attn.attn_fwd(Q, K, V, cancelling.SCALE)[0]}
    got["dQ"], got["dK"], got["dV"] = attn.attn_bwd(Q, K, V, O_in, dO, to_dev(LSE[None], "f32"), cancelling.SCALE)
    for name in sums:
        ref, bound = cancelling.expected(sums, name)
        worst = float((np.abs(to_np(got[name])[0, :, 0, :cancelling.D][:, sums[name][4]] - ref) / bound).max())
        print("cancelling d=%d %s: %.2f of the bound" % (d, name, worst), flush=True)
        assert worst <= 1.0, name
