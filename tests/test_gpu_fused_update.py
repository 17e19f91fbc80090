"""An update of all chunks takes the step's scalar work along in its own launch (tests/pins/host_fused.cpp: when).  The same steps in a
context that has been captured into a graph, whose scalar kernel runs in front of the update, have to give every bit of them: sums,
norm, constants, step counter and loss scale, and the state."""
import pytest
import torch

from paper_2406_08334_amd import binding as B

from gpu_harness import ChunkedState, assert_same_bits, hp_pair

pytestmark = pytest.mark.gpu

INF = {torch.bfloat16: 0x7F80, torch.float16: 0x7C00}


def run(sizes, S, dtype, fp32, masked, captured, tries=None):
    scaler = B.pt_scaler_cfg(1024.0, 2.0, 0.5, 2, 0) if dtype == torch.float16 else None
    st = ChunkedState(sizes, S, dtype=dtype, grad_fp32=fp32, scaler=scaler)
    try:
        if captured:
            with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=torch.cuda.Stream()):
                B.pt_step_end(st.ctx)
        if tries is not None:
            B.pt_ctx_set_option(st.ctx, "update_test_tries", tries)
        B.pt_ctx_set_option(st.ctx, "adamw_zero_grads", int(fp32))
        if masked:
            st.set_no_decay(runs=[(0, 0, 3), (st.C - 1, S // 2 - 2, 5), (0, S - 1, 1), (0, 256, 512)])
        hp, _, _ = hp_pair()
        seen = []
        for t in range(1, 5):
            st.set_grads(t, scale=256.0 if scaler else 1.0)
            if t == 2:
                st.grad_src.view(torch.int16)[st.N // 2] = INF[dtype]
            if fp32:
                st.accum(False, True)
            else:
                st.pack()
            # the last step keeps the sum of a chunk that nothing packed in it
            st.norm(finalize=B.PT_FINALIZE_CARRY if t == 4 else B.PT_FINALIZE_STRICT)
            st.adamw(hp)
            r, c = B.pt_step_report_read(st.ctx), B.pt_update_consts_read(st.ctx)
            seen.append((repr(r.sqnorm), repr(r.norm), r.clip_coef, r.grad_mult, r.found_inf, r.step, r.loss_scale, r.good_steps,
                         tuple(c.c), c.skip))
            st.end()
            r = st.report()
            seen.append((r.step, r.loss_scale, r.good_steps))
        host = st.host_state()
        return seen, {k: host[k] for k in ("w", "m", "v", "p16") + (("g32",) if fp32 else ("g16",))}
    finally:
        st.close()


# plans whose sums wait for the update: a wave's partial sum covers 2048 elements (fp32 sums: 1024) of a tensor at most, and a unit 4096 of them
SHAPES = [
    ([1 << 16], 1 << 16),                                   # the smallest state that is taken along, one chunk
    ([70000], 1 << 15),                                     # three chunks, a padded end
    ([131072 * 2 + 8], 131072 * 2 + 8),                     # a partial sum more than two trees of 64
    ([512 * 2048 + 1], 1 << 21),                            # a row of 512 and one of the next
    ([4096 * 2048 + 1], (1 << 23) + 8),                     # a unit and one partial sum of the next
    ([4096 * 2048 * 3 - 5], 4096 * 2048 * 3),               # three units of one chunk
    ([1 << 18] * 7 + [(1 << 18) - 3], 1 << 18),             # eight chunks
    ([3, 1, 5] * 300 + [70000], 1 << 16),                   # many tiny tensors
    ([1 << 13] * 9, 1 << 13),                               # nine chunks: their sums are there already
    ([1 << 12] * 70, 1 << 12),                              # more chunks than a wave has lanes
]


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("dtype,fp32", [(torch.bfloat16, False), (torch.float16, False), (torch.bfloat16, True)])
@pytest.mark.parametrize("sizes,S", SHAPES)
def test_as_with_the_scalar_kernel_in_front(sizes, S, dtype, fp32, masked):
    want = run(sizes, S, dtype, fp32, masked, True)
    # 0 looks for what the first workgroup publishes: every wave that runs by then derives the constants by itself
    for tries in (None, 0):
        got = run(sizes, S, dtype, fp32, masked, False, tries)
        assert got[0] == want[0]
        for name, bits in want[1].items():
            assert_same_bits(got[1][name], bits, (name, tries))
