"""The kernels' own launch shapes at the sizes where they can go wrong: edges of tiles and of 128-byte lines,
remainders, the smallest inputs.  Each against the CPU oracle, bit for bit where the oracle has the same sequence."""
import numpy as np
import pytest
import torch

from paper_2406_08334_amd import binding as B

from gpu_harness import ChunkedState, assert_same_bits, hp_pair
from test_gpu_parity import run_oracle_f32seq

pytestmark = pytest.mark.gpu


# tile of the update: 256 elements; a line: 32 elements of an fp32 array, so S mod 32 != 0 puts every chunk of an arena at
# another place within its line
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("S,C,grid,masked", [
    (8, 5, 0, False), (24, 4, 0, True), (248, 3, 0, True), (256, 3, 0, False), (264, 5, 0, True), (512 + 8, 4, 0, False),
    (4096 * 3 + 40, 4, 0, True), (5000 * 8, 3, 0, True), (1 << 15, 3, 0, True),
    (264, 5, 1, True), (4096 + 8, 4, 7, False), (4096 + 24, 4, 20, True)])
def test_update_in_its_default_shape(orc, dtype, S, C, grid, masked):
    st = ChunkedState([S * C - 5], S, dtype=dtype)
    try:
        B.pt_ctx_set_option(st.ctx, "adamw_grid", grid)
        hp_b, hp_o, _ = hp_pair()
        runs = [(0, 0, 3), (C - 1, S - 1, 1), (1, 0, S), (2, S // 2 - 2, 5), (2, S // 2 + 3, 1)] if masked else []
        mask = st.set_no_decay(runs=runs) if masked else None
        host = st.host_state()
        for t in (1, 2, 3):
            st.set_grads(t)
            st.pack()
            B.pt_step_override(st.ctx, 0.0121, t == 3)            # the third step is skipped: nothing changes
            st.adamw(hp_b)
            st.end()
            host["g16"] = st.oracle_packed(orc)
            if t < 3:
                run_oracle_f32seq(orc, orc.consts_f32(hp_o, t, float(np.float32(0.0121))), host, st.orc_dtype, no_decay=mask)
            got = st.host_state()
            for name in ("g16", "w", "m", "v", "p16"):
                assert_same_bits(got[name], host[name], (name, t))
    finally:
        st.close()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("masked", [False, True])
def test_hints_by_the_size_of_the_gradient_chunks_change_no_bit(orc, dtype, masked):
    """A context whose 16-bit gradient chunks exceed the 256 MB Infinity Cache, of which pack stores the first 240 MB without
    non-temporal hints.  Only three of its chunks exist here: their bits are the oracle's."""
    S, n = 4096 * 3 + 40, 3
    C = (256 << 20) // (2 * S) + 1
    small = ChunkedState([S * n - 5], S, dtype=dtype)
    ctx = B.pt_ctx_create(small.pt_dtype, S, C, None)
    plan = B.pt_pack_plan_create(ctx, small.segs)
    try:
        assert 2 * S * C > 256 << 20 >= 2 * S * (C - 1)
        hp_b, hp_o, _ = hp_pair()
        runs = [(0, 0, 3), (n - 1, S - 1, 1), (1, 0, S), (2, S // 2 - 2, 5)] if masked else []
        mask = small.set_no_decay(runs=runs) if masked else None
        if masked:
            B.pt_ctx_set_no_decay(ctx, [B.pt_segment(0, 0, ln, off, c, 0) for c, off, ln in runs])
        host = small.host_state()
        for t in (1, 2):
            small.set_grads(t)
            B.pt_chunk_pack_grads(ctx, plan, small.rows(small.g16) + [None] * (C - n))
            B.pt_step_override(ctx, 0.0121, False)
            B.pt_chunk_adamw_step(ctx, hp_b, 0, n, small.rows(small.g16), small.rows(small.w), small.rows(small.m),
                                  small.rows(small.v), small.rows(small.p16))
            B.pt_step_end(ctx)
            host["g16"] = small.oracle_packed(orc)
            run_oracle_f32seq(orc, orc.consts_f32(hp_o, t, float(np.float32(0.0121))), host, small.orc_dtype, no_decay=mask)
            got = small.host_state()
            for name in ("g16", "w", "m", "v", "p16"):
                assert_same_bits(got[name], host[name], (name, t))
    finally:
        torch.cuda.synchronize()
        B.pt_pack_plan_destroy(plan)
        B.pt_ctx_destroy(ctx)
        small.close()
