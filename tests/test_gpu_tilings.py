"""GPU parity of every tiling of the fused backward (attn_bwd_tiling): each one against the float64
oracle on the same seeded inputs, and against each other where the arithmetic is the same."""
import numpy as np
import pytest

from paper_2410_09397_amd import synth
from tests.helpers import TOL, check, oracle_reference, rel_err, to_dev, to_np

pytestmark = pytest.mark.gpu

TWO_KERNEL, ONEPASS_K64, ONEPASS_K128, FOUR_PHASE, SPLIT_D = 1, 2, 3, 6, 7


def W(name, index, b, h, n, d, dtype="bf16", **kw):
    return synth.Workload(name, index, b, h, n, d, dtype, **kw)


CASES = [
    W("t_d128_causal", 131, 1, 2, 512, 128, causal=True, dO_std=0.1),
    W("t_d128_ragged", 132, 1, 3, 200, 128),
    W("t_d128_ragged_causal", 133, 2, 2, 333, 128, causal=True),
    W("t_d128_9tiles_ragged", 136, 1, 1, 570, 128),
    W("t_d128_8heads", 137, 2, 4, 256, 128, causal=True),
    W("t_d128_sparse", 141, 1, 2, 1024, 128, sparse=True, extra_frac=0.3),
    W("t_d128_sparse_causal_ragged", 144, 1, 2, 1100, 128, sparse=True, causal=True, extra_frac=0.4),
    W("t_d128_masks_per_head", 145, 2, 3, 900, 128, sparse=True, extra_frac=0.3, per_head_masks=True),
    W("t_d128_one_row", 162, 1, 2, 1, 128, causal=True),
    W("t_d128_65_rows", 163, 1, 1, 65, 128),
    W("t_d64", 121, 1, 2, 384, 64),
    W("t_d64_ragged_causal", 122, 2, 1, 333, 64, causal=True),
    W("t_d64_sparse_causal", 143, 1, 2, 768, 64, sparse=True, causal=True, extra_frac=0.5),
    W("t_d64_tiny", 123, 1, 1, 5, 64),
]


def tilings_for(d):
    return [ONEPASS_K64, ONEPASS_K128]


def run_bwd(w, mask, tiling, *args):
    from paper_2410_09397_amd import attn
    if mask is not None:
        return attn.attn_bwd_blocksparse(*args, w.scale, mask, causal=w.causal, tiling=tiling)
    return attn.attn_bwd(*args, w.scale, causal=w.causal, tiling=tiling)


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_one_pass_tilings_match_oracle(w):
    import torch
    from paper_2410_09397_amd import attn
    print("case", w, flush=True)
    inp = synth.make_inputs(w)
    ref = oracle_reference(w, inp)
    Q, K, V, dO = (to_dev(inp[t], w.dtype) for t in ("Q", "K", "V", "dO"))
    mask = attn.BlockMask(inp["keep"], w.block, w.n) if inp["keep"] is not None else None
    O_in, LSE_in = to_dev(ref["O_in"], w.dtype), to_dev(ref["LSE_in"], "f32")
    base = run_bwd(w, mask, TWO_KERNEL, Q, K, V, O_in, dO, LSE_in)
    for tiling in tilings_for(w.d):
        print("tiling", tiling, flush=True)
        grads = run_bwd(w, mask, tiling, Q, K, V, O_in, dO, LSE_in)
        torch.cuda.synchronize()
        for name, g, r in zip(("dQ", "dK", "dV"), grads, ref["iso"]):
            check("%s tiling %d" % (w.name, tiling), name, to_np(g), r, w.dtype)
        # the key-block owners of both tilings accumulate dK and dV over the same tiles in a fixed order
        again = run_bwd(w, mask, tiling, Q, K, V, O_in, dO, LSE_in)
        for a, b in zip(grads[1:], again[1:]):
            assert torch.equal(a, b), tiling
        # dQ: sums of the same terms in another order (a single row has dQ = 0 up to rounding)
        a, b = to_np(grads[0]), to_np(base[0])
        assert np.abs(a - b).max() <= 2e-2 * max(np.abs(b).max(), 1e-3)


OTHER_PATH = [
    # the four-phase scheme where the fused kernels are the default, the fused split-d kernels where it is
    (W("t4_d128_causal", 171, 1, 2, 512, 128, causal=True, dO_std=0.1), FOUR_PHASE),
    (W("t4_d256_ragged", 172, 1, 2, 333, 256), FOUR_PHASE),
    (W("t7_d512", 173, 1, 2, 384, 512), SPLIT_D),
    (W("t7_d512_ragged_causal", 174, 2, 1, 333, 512, causal=True), SPLIT_D),
    (W("t7_d512_one_row", 175, 1, 1, 1, 512, causal=True), SPLIT_D),
    (W("t7_d512_33_rows", 176, 1, 2, 33, 512), SPLIT_D),
    (W("t7_d256_causal", 177, 1, 2, 700, 256, causal=True), SPLIT_D),
]


@pytest.mark.parametrize("w,tiling", OTHER_PATH, ids=lambda x: x.name if hasattr(x, "name") else str(x))
def test_other_path_tilings_match_oracle(w, tiling):
    import torch
    print("case", w, "tiling", tiling, flush=True)
    inp = synth.make_inputs(w)
    ref = oracle_reference(w, inp)
    Q, K, V, dO = (to_dev(inp[t], w.dtype) for t in ("Q", "K", "V", "dO"))
    O_in, LSE_in = to_dev(ref["O_in"], w.dtype), to_dev(ref["LSE_in"], "f32")
    grads = run_bwd(w, None, tiling, Q, K, V, O_in, dO, LSE_in)
    torch.cuda.synchronize()
    for name, g, r in zip(("dQ", "dK", "dV"), grads, ref["iso"]):
        check("%s tiling %d" % (w.name, tiling), name, to_np(g), r, w.dtype)
    again = run_bwd(w, None, tiling, Q, K, V, O_in, dO, LSE_in)
    for a, b in zip(grads, again):
        assert torch.equal(a, b), tiling  # neither path has atomics


def test_unsupported_tilings_are_rejected():
    import torch
    from paper_2410_09397_amd import attn
    x = torch.zeros(1, 1, 128, 256, dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros(1, 1, 128, dtype=torch.float32, device="cuda")
    for tiling in (ONEPASS_K64, ONEPASS_K128):
        with pytest.raises(attn.AttnError) as e:
            attn.attn_bwd(x, x, x, x, x, lse, 1.0, tiling=tiling)
        assert e.value.status == attn.ATTN_ERR_UNSUPPORTED
    x64 = torch.zeros(1, 1, 128, 64, dtype=torch.bfloat16, device="cuda")
    for tiling in (FOUR_PHASE, SPLIT_D):
        with pytest.raises(attn.AttnError) as e:
            attn.attn_bwd(x64, x64, x64, x64, x64, lse, 1.0, tiling=tiling)
        assert e.value.status == attn.ATTN_ERR_UNSUPPORTED


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("kind", ["full", "causal", "mask", "causal_masks_per_head"])
def test_one_launch_and_two_have_the_same_bits(d, kind):
    """The library's choice runs the two owners of small calls side by side, with the row sums from a launch of their own: the same
    blocks, so the same bits as the two kernels, at the edges of the blocks, with query blocks of 64 and of 128 (many heads), in
    tensors whose heads are interleaved, and with more blocks than are ranked in one workgroup."""
    import torch
    from paper_2410_09397_amd import attn
    causal, masked = kind.startswith("causal"), "mask" in kind
    shapes = [(1, 1, 1), (1, 3, 63), (2, 4, 65), (1, 8, 128), (3, 1, 333), (1, 5, 700), (1, 1, 1025), (1, 40 if d == 256 else 70, 513)]
    if d == 64 and kind == "mask":
        shapes.append((1, 1, 128 * 257 + 5))
    for b, h, n in shapes:
        print("case", kind, d, b, h, n, flush=True)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(n)
        Q, K, V, dO = (torch.randn((b, n, h, d), generator=gen, device="cuda").to(torch.bfloat16).transpose(1, 2) for _ in range(4))
        mask = None
        if masked:
            nblk = (n + 127) // 128
            keep = np.random.default_rng(n).random((b * h, nblk, nblk) if "per_head" in kind else (nblk, nblk)) < min(0.5, 8 / nblk)
            keep[..., 0, 0] = True
            mask = attn.BlockMask(keep, 128, n)
        w = synth.Workload("one_launch", 190, b, h, n, d, "bf16", causal=causal)
        O, LSE = attn.attn_fwd(Q, K, V, w.scale, causal=causal, mask=mask, out=(torch.empty_like(Q), torch.empty((b, h, n), device="cuda")))
        args = (Q, K, V, O, dO, LSE)
        for x, y in zip(run_bwd(w, mask, 0, *args), run_bwd(w, mask, TWO_KERNEL, *args)):
            assert torch.isfinite(x).all() and torch.equal(x, y)
