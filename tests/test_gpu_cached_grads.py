"""The first 240 MB of a context's gradient chunks are stored by pack and, from 100 MB of sums on, loaded by accumulate without
non-temporal hints.  That changes no bit: tensors that are cut by that line, aligned and not, and chunks before, on and behind it."""
import pytest
import torch

from paper_2406_08334_amd import binding as B

from gpu_harness import hp_pair

pytestmark = pytest.mark.gpu

CACHED = 240 << 20


def gradients(n, dtype, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.empty(n, device="cuda").normal_(0.0, 1.0, generator=gen).to(dtype)


@pytest.mark.parametrize("shift", [0, 1])                            # elements the tensor is off the alignment
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_sums_on_both_sides_of_the_line(dtype, shift):
    line, n = CACHED // 4, 3 * 4096 + 7
    S = (line // 3 // 8 + 1) * 8                                     # the line falls into the end of the third of four chunks
    lo = line - 2 * S - n // 2                                       # of the tensor in that chunk, cut by the line
    n = min(n, S - lo)
    chunks = [torch.empty(S, device="cuda") for _ in range(4)]
    ctx = B.pt_ctx_create(B.PT_BF16 if dtype == torch.bfloat16 else B.PT_FP16, S, 4, None)
    B.pt_ctx_set_option(ctx, "grad_fp32", 1)
    src = gradients(2 * n + 16, dtype, 1 + shift)
    segs = [B.pt_segment(src.data_ptr() + 2 * shift, 0, n, lo, 2, 0), B.pt_segment(src.data_ptr() + 2 * (shift + n), 0, n, 5, 3, 1)]
    plan = B.pt_pack_plan_create(ctx, segs)
    try:
        parts = [(chunks[2], lo, src[shift:shift + n]), (chunks[3], 5, src[shift + n:shift + 2 * n])]
        want = [gradients(n, torch.float32, 7 + k) for k in range(2)]
        for (c, at, _), w in zip(parts, want):
            c[at:at + n] = w
        for k in range(3):                                           # overwritten, then added to twice; the norm with the last
            B.pt_chunk_accum_grads(ctx, plan, chunks, k == 0, k == 2)
            want = [g.float() if k == 0 else w + g.float() for w, (_, _, g) in zip(want, parts)]
            for (c, at, _), w in zip(parts, want):
                assert torch.equal(c[at:at + n], w), k
        B.pt_chunk_grad_sqnorm(ctx, None, 0, 4, B.PT_FINALIZE_CARRY)
        sq = sum(float(w.double().square().sum()) for w in want)
        assert abs(B.pt_step_report_read(ctx).sqnorm - sq) <= 1e-12 * sq          # fp64 sums in another order
    finally:
        torch.cuda.synchronize()
        B.pt_pack_plan_destroy(plan)
        B.pt_ctx_destroy(ctx)


@pytest.mark.parametrize("fp32", [False, True])
def test_update_on_both_sides_of_the_line(fp32):
    """A chunk with the line inside it (not on a tile's start), packed and updated with the hints and without any."""
    line, C = CACHED // (4 if fp32 else 2), 2
    S = line // C + 40 * 256 + 8
    gen = torch.Generator(device="cuda").manual_seed(3)
    base = {k: torch.empty(C, S, device="cuda").normal_(0.0, 0.01, generator=gen) for k in ("w", "m", "v")}
    base["v"].square_()
    src = gradients(C * S, torch.bfloat16, 5)
    got = []
    for nt in (2, 0):
        ctx = B.pt_ctx_create(B.PT_BF16, S, C, None)
        B.pt_ctx_set_option(ctx, "adamw_nt", nt)
        B.pt_ctx_set_option(ctx, "grad_fp32", int(fp32))
        B.pt_ctx_set_option(ctx, "adamw_zero_grads", int(fp32))
        segs = [B.pt_segment(src.data_ptr() + 2 * S * c, 0, S, 0, c, c) for c in range(C)]
        plan = B.pt_pack_plan_create(ctx, segs)
        a = {k: x.clone() for k, x in base.items()}
        a["p"] = a["w"].bfloat16()
        a["g"] = torch.zeros(C, S, dtype=torch.float32 if fp32 else torch.bfloat16, device="cuda")
        r = {k: [x[c] for c in range(C)] for k, x in a.items()}
        hp, _, _ = hp_pair()
        if fp32:
            B.pt_chunk_accum_grads(ctx, plan, r["g"], True, True)
        else:
            B.pt_chunk_pack_grads(ctx, plan, r["g"])
        assert torch.equal(a["g"].view(-1), src.to(a["g"].dtype))
        B.pt_chunk_grad_sqnorm(ctx, None, 0, C, True)
        B.pt_chunk_adamw_step(ctx, hp, 0, C, r["g"], r["w"], r["m"], r["v"], r["p"])
        B.pt_step_end(ctx)
        torch.cuda.synchronize()
        B.pt_pack_plan_destroy(plan)
        B.pt_ctx_destroy(ctx)
        got.append(a)
    assert not torch.equal(got[0]["w"], base["w"])
    for k in got[0]:
        assert torch.equal(got[0][k], got[1][k]), k
    if fp32:
        assert not got[0]["g"].any()
