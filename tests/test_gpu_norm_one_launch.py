"""The norm of a small arena without a context, in one launch, gives the bits of the context's two, at the edges of what one launch
takes: powers of two and their neighbours in workgroups per chunk, trees per chunk, chunks per wave, and the first sizes beyond."""
import math

import pytest
import torch

from paper_2406_08334_amd import binding as B

pytestmark = pytest.mark.gpu

BLOCK = 32768

# (workgroups per chunk, chunks): up to 512 per chunk, 1024 in all and 16 waves of partial sums in one launch
SHAPES = [(1, 1), (1, 16), (1, 17), (1, 1023), (1, 1024), (1, 1025), (2, 3), (2, 512), (3, 255), (3, 257), (5, 7), (32, 32), (33, 16), (33, 17),
          (63, 2), (64, 16), (65, 8), (65, 9), (128, 2), (511, 2), (512, 1), (512, 2), (513, 1)]


def both(g, dt, scale):
    C, S = g.shape
    out, inf = torch.full((2,), -1.0, dtype=torch.float64, device="cuda"), torch.full((1,), -1, dtype=torch.int32, device="cuda")
    B.pt_chunk_grad_sqnorm_noalloc(g, dt, S, C, scale, out, inf)
    ctx = B.pt_ctx_create(dt, S, C, B.pt_scaler_cfg(scale, 2.0, 0.5, 1000, 0))
    try:
        B.pt_chunk_grad_sqnorm(ctx, [g[c] for c in range(C)], 0, C, True)
        rep = B.pt_step_report_read(ctx)
    finally:
        B.pt_ctx_destroy(ctx)
    return (float(out[0]), float(out[1]), int(inf[0])), (rep.sqnorm, rep.norm, rep.found_inf)


@pytest.mark.parametrize("per,chunks", SHAPES)
def test_same_bits_as_two_launches(per, chunks):
    # short last workgroups keep the many-chunk arenas small
    S = BLOCK * (per - 1) + (8 * 37 if per * chunks > 64 else 8)
    gen = torch.Generator(device="cuda").manual_seed(per * 2048 + chunks)
    g = torch.empty(chunks, S, device="cuda").normal_(0.0, 3.0, generator=gen).half()
    for scale in (1.0, 1000.0):
        one, two = both(g, B.PT_FP16, scale)
        assert one == two
    g[chunks // 2, S - 1] = math.inf
    one, two = both(g, B.PT_FP16, 1.0)
    assert one == two and one[2] == 1
    g[0, 0] = math.nan
    one, two = both(g, B.PT_FP16, 1.0)
    assert one[2] == two[2] == 1 and math.isnan(one[0]) and math.isnan(two[0])


def test_call_after_call_of_other_sizes():
    """More calls than there are counters, sizes of one and of two launches in turn, on the current and on another stream; and a call captured
    (two launches) and replayed among them."""
    gen = torch.Generator(device="cuda").manual_seed(1)
    sizes = [(8, 1), (BLOCK * 3, 5), (BLOCK * 600, 1), (BLOCK * 100 + 8, 2)]
    gs = [torch.empty(C, S, device="cuda").normal_(0.0, 1.0, generator=gen).bfloat16() for S, C in sizes]
    want = [both(g, B.PT_BF16, 1.0)[1] for g in gs]
    out, inf = torch.zeros(2, dtype=torch.float64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")

    def check(k):
        assert (float(out[0]), float(out[1]), int(inf[0])) == want[k], k

    def call(k):
        S, C = sizes[k]
        B.pt_chunk_grad_sqnorm_noalloc(gs[k], B.PT_BF16, S, C, 1.0, out, inf)

    side = torch.cuda.Stream()
    for n in range(60):
        k = n % len(sizes)
        out.zero_()
        if n % 3 == 0:
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                call(k)
            torch.cuda.current_stream().wait_stream(side)
        else:
            call(k)
        check(k)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        call(1)
    for n in range(40):
        out.zero_()
        graph.replay()
        check(1)
        call(3)
        check(3)
