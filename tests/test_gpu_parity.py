"""GPU parity: the HIP path (through the C-ABI binding) against the CPU oracle, element
by element, on the same seeded inputs.

Bars: pack/unpack and indexing bit-exact; gradient norm within relative 1e-5; fp32
master/m/v within 1e-6 of the fp64 oracle (scale-aware, see tests/tolerance.py);
16-bit parameters within one unit in the last place; and, with the device's own nine
fp32 constants handed to the oracle's fp32 operation sequence, every array bit-exact.
"""
import math

import numpy as np
import pytest
import torch

import oracle as O
from paper_2406_08334_amd import binding as B
from paper_2406_08334_amd import shapes, synth
from gpu_harness import ChunkedState, HP, assert_same_bits, hp_pair, same_bits, to_u16
from tolerance import ScaleTracker, check_p16, far_cap, ulp16_distance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    B.lib()                                    # fails loudly if the HIP library is missing
    yield
    torch.cuda.synchronize()


def ulp_diff32(a, b):
    a = np.asarray(a, np.float32).view(np.int32).astype(np.int64)
    b = np.asarray(b, np.float32).view(np.int32).astype(np.int64)
    return np.abs(a - b)


# ------------------------------------------------------------------------------- pack

RAGGED = [1, 3, 7, 8, 9, 17, 4099, 16384, 16385, 33, 100_003, 5, 2]      # odd sizes: misaligned sources
ALIGNED = [8, 4096, 16384 * 3, 40, 8 * 12345, 64]


@pytest.mark.parametrize("sizes,S", [(RAGGED, 16384 * 2 + 64), (RAGGED, 1024), (ALIGNED, 32768), ([5], 8),
                                     ([], 64), ([64], 64)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_pack_is_bit_exact_and_leaves_padding_alone(orc, sizes, S, dtype):
    st = ChunkedState(sizes, S, dtype=dtype, init_params=False)
    try:
        n = st.N
        bits = torch.randint(-32768, 32767, (max(n, 1),), dtype=torch.int16, device="cuda")
        st.grad_src.view(torch.int16).copy_(bits)
        st.g16.view(torch.int16).fill_(0x5A5A)               # sentinel: padding must survive
        st.pack()
        got = to_u16(st.g16)
        src = to_u16(st.grad_src)[:n]
        offs = np.cumsum([0] + list(sizes))
        want = orc.pack_dense([src[offs[i]:offs[i + 1]] for i in range(len(sizes))], S, n_chunks=st.C)
        assert same_bits(got.reshape(-1)[:n], want.reshape(-1)[:n])
        assert np.all(got.reshape(-1)[n:] == 0x5A5A)
        # inverse copy restores the tensors bit for bit
        st.grad_src.zero_()
        B.pt_chunk_unpack(st.ctx, st.plan, st.rows(st.g16))
        assert same_bits(to_u16(st.grad_src)[:n], src)
    finally:
        st.close()


def test_pack_gpt2_block_layout_against_oracle(orc):
    table, S = shapes.workload("gpt2_block_768")
    sizes = [n for _, n in table]
    st = ChunkedState(sizes, S, init_params=False)
    try:
        st.set_grads(1)
        st.pack()
        src = to_u16(st.grad_src)
        offs = np.cumsum([0] + sizes)
        want = orc.pack_dense([src[offs[i]:offs[i + 1]] for i in range(len(sizes))], S)
        assert same_bits(to_u16(st.g16), want)
        assert not to_u16(st.g16)[1, S - 1_300_736:].any()
    finally:
        st.close()


# ------------------------------------------------------------------------------- norm

@pytest.mark.parametrize("dtype,scaler", [(torch.bfloat16, None), (torch.float16, B.pt_scaler_cfg(65536.0, 2.0, 0.5, 2000, 0))])
@pytest.mark.parametrize("sizes,S", [(RAGGED, 32768 + 64), (ALIGNED, 32768), ([7_087_872], 1 << 22)])
def test_norm_fused_and_standalone_match_oracle(orc, dtype, scaler, sizes, S):
    st = ChunkedState(sizes, S, dtype=dtype, scaler=scaler, init_params=False)
    try:
        sigma = 65536.0 if scaler is not None else 1.0
        st.set_grads(1, scale=sigma)
        st.pack(); st.norm()
        r1 = st.report()
        g = st.oracle_packed(orc)                                    # the oracle's own packing of the sources
        assert_same_bits(to_u16(st.g16).reshape(-1), g, "g16")
        want = orc.sqnorm(g, st.orc_dtype, loss_scale=sigma, block=S, threads=8)
        assert r1.found_inf == 0
        assert abs(r1.sqnorm - want) <= 1e-12 * want                 # bar is 1e-5 on the norm
        assert abs(r1.norm - math.sqrt(want)) <= 1e-5 * math.sqrt(want)
        st.norm(recompute=True)
        r2 = st.report()
        assert abs(r2.sqnorm - want) <= 1e-12 * want
        # run-to-run bitwise reproducible
        st.pack(); st.norm()
        assert st.report().sqnorm == r1.sqnorm
        st.norm(recompute=True)
        assert st.report().sqnorm == r2.sqnorm
    finally:
        st.close()


def test_norm_closed_forms(orc):
    S = 1 << 20
    st = ChunkedState([4 * S], S, init_params=False)          # 2^22 ones -> norm 2048 exactly
    try:
        st.grad_src.fill_(1.0)
        st.pack(); st.norm()
        assert st.report().norm == 2048.0
        st.grad_src.zero_()
        st.pack(); st.norm()
        assert st.report().norm == 0.0 and st.report().found_inf == 0
        st.grad_src[3 * S + 12345] = -0.375
        st.pack(); st.norm()
        assert st.report().norm == 0.375
    finally:
        st.close()


@pytest.mark.parametrize("dtype,pats", [(torch.bfloat16, [0x7F80, 0xFF80, 0x7FC1]), (torch.float16, [0x7C00, 0xFC00, 0x7E00])])
def test_nonfinite_is_found_wherever_it_sits(orc, dtype, pats):
    sizes, S = RAGGED, 32768 + 64
    st = ChunkedState(sizes, S, dtype=dtype, init_params=False)
    try:
        n = st.N
        for k, pos in enumerate([0, 6, 16384 + 3, n - 1, n // 2, S - 1, S]):
            st.set_grads(1)
            st.grad_src.view(torch.int16)[pos] = np.array(pats[k % 3], np.uint16).view(np.int16).item()
            st.pack(); st.norm()
            assert st.report().found_inf == 1, pos
            st.norm(recompute=True)
            assert st.report().found_inf == 1, pos
        st.set_grads(1)
        st.grad_src.view(torch.int16)[5] = 0x7F7F if dtype == torch.bfloat16 else 0x7BFF   # largest finite
        st.pack(); st.norm()
        assert st.report().found_inf == 0
    finally:
        st.close()


# ------------------------------------------------------------------------------- AdamW

def run_oracle_f32seq(orc, consts, st_host, dtype, no_decay=None):
    orc.adamw_f32seq(consts, st_host["g16"], st_host["w"], st_host["m"], st_host["v"], st_host["p16"], dtype, threads=8,
                     no_decay=no_decay)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("S,C,threads,nt", [(4096 * 3 + 40, 3, 512, 1), (8, 2, 512, 2), (16384 * 8, 2, 512, 0), (4096, 1, 512, 1),
                                            (4096 * 3 + 40, 3, 256, 0), (16384 * 8 + 2048, 2, 256, 1)])
def test_adamw_kernel_isolated_is_bit_exact_against_f32_sequence(orc, dtype, S, C, threads, nt):
    st = ChunkedState([S * C - 5], S, dtype=dtype)
    try:
        B.pt_ctx_set_option(st.ctx, "adamw_threads", threads)
        B.pt_ctx_set_option(st.ctx, "adamw_nt", nt)          # with or without hints: same bits
        hp_b, hp_o, hpd = hp_pair()
        host = st.host_state()
        h64 = {k: a.copy() for k, a in host.items()}
        trk = ScaleTracker(host["w"], host["m"], hpd)
        gm = 0.0121
        for t in (1, 2, 3):
            st.set_grads(t)
            st.pack()
            B.pt_step_override(st.ctx, gm, False)
            st.adamw(hp_b)
            k = B.pt_update_consts_read(st.ctx)
            st.end()
            consts = np.array(list(k.c), dtype=np.float32)
            want_c = orc.consts_f32(hp_o, t, float(np.float32(gm)))
            # the device derives the very constants the oracle derives: the oracle runs on its own
            assert same_bits(consts, want_c) and k.skip == 0
            # ... and on its own packing of the same seeded source gradients
            g16 = orc.pack_dense([to_u16(st.grad_src[:st.N])], S, st.C).reshape(-1)
            assert_same_bits(to_u16(st.g16).reshape(-1), g16, ("g16", t))
            host["g16"] = g16.copy()
            run_oracle_f32seq(orc, want_c, host, st.orc_dtype)
            got = st.host_state()
            for name in ("w", "m", "v", "p16"):
                assert same_bits(got[name], host[name]), (name, t)
            # and the fp64 oracle bounds both
            orc.adamw_f64(hp_o, t, float(np.float32(gm)), g16, h64["w"], h64["m"], h64["v"], h64["p16"], st.orc_dtype, threads=8)
            trk.advance(t, orc.decode16(g16, st.orc_dtype).astype(np.float64) * float(np.float32(gm)), h64["v"])
            trk.check((got["w"], got["m"], got["v"]), (h64["w"], h64["m"], h64["v"]), tol=1e-6)
            far = check_p16(orc.decode16(got["p16"], st.orc_dtype), orc.decode16(h64["p16"], st.orc_dtype), h64["w"],
                            trk.W, dtype == torch.float16)
            assert far <= far_cap(got["p16"].size)
        # padding stayed exactly zero
        assert not got["w"][-5:].any() and not got["m"][-5:].any() and not got["v"][-5:].any() and not got["p16"][-5:].any()
    finally:
        st.close()


def test_adamw_is_bit_exact_where_intermediates_are_subnormal_or_extreme(orc):
    """Degenerate values of the update: gradients so small that g^2 and the variance are subnormal in
    fp32 or vanish, the smallest subnormal 16-bit words, huge finite gradients, weights of either zero,
    tiny and large magnitudes - every 16-bit exponent appears.  The device must follow the fp32 sequence
    (pinned against exact rational arithmetic, subnormals included) bit for bit: no flush to zero anywhere."""
    S = 8192 + 8
    st = ChunkedState([2 * S - 3], S, dtype=torch.bfloat16, init_params=False)
    try:
        hp_b, hp_o, _ = hp_pair()
        n = st.N
        rng = np.random.default_rng(3)
        # every finite bf16 pattern several times, in random order, as gradients; another draw as parameters
        pats = np.arange(1 << 16, dtype=np.uint16)
        finite = pats[(pats & 0x7F80) != 0x7F80]
        gw = rng.choice(finite, n).astype(np.uint16)
        pw = rng.choice(finite, n).astype(np.uint16)
        pw[(pw & 0x7F80) > 0x7000] &= np.uint16(0xBFFF)            # keep |w| below 2^98: w * decay stays finite
        st.grad_src[:n].view(torch.int16).copy_(torch.from_numpy(gw.view(np.int16)).cuda())
        st.p16.view(-1)[:n].view(torch.int16).copy_(torch.from_numpy(pw.view(np.int16)).cuda())
        st.w.copy_(st.p16.float())
        host = st.host_state()
        for t, gm in ((1, 1.0), (2, 2.0 ** -40), (3, 2.0 ** -75)):
            st.pack()
            B.pt_step_override(st.ctx, gm, False)
            st.adamw(hp_b)
            st.end()
            host["g16"] = st.oracle_packed(orc)
            run_oracle_f32seq(orc, orc.consts_f32(hp_o, t, gm), host, st.orc_dtype)
            got = st.host_state()
            for name in ("w", "m", "v", "p16"):
                assert_same_bits(got[name], host[name], (name, t))
        v = host["v"][:n]
        sub = (np.abs(v) > 0) & (np.abs(v) < np.float32(2.0 ** -126))
        assert sub.sum() > 100, "the case is meant to reach subnormal variances"
    finally:
        st.close()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_access_pattern_calibration_leaves_the_state_as_it_is(dtype):
    """pt_calib_adamw_pattern reads and rewrites the update's arrays without changing a bit (master,
    momentum, variance stored back as read; param16 re-derived from the master weight it already equals)."""
    S = 4096 * 4 + 8                                             # whole tiles and a ragged tail per chunk
    st = ChunkedState([3 * S - 11], S, dtype=dtype)
    try:
        hp_b, _, _ = hp_pair()
        with pytest.raises(B.PtError) as e:
            B.pt_calib_adamw_pattern(st.ctx, 0, st.C)            # no update has bound the pointers yet
        assert e.value.status == B.PT_ERR_STATE
        for t in (1, 2):
            st.set_grads(t)
            st.step(hp_b)
        before = st.host_state()
        for unroll, nt in ((0, 2), (0, 0), (4, 1), (1, 2), (8, 0)):      # 0: the library's own shape
            B.pt_ctx_set_option(st.ctx, "adamw_unroll", unroll)
            B.pt_ctx_set_option(st.ctx, "adamw_nt", nt)
            B.pt_calib_adamw_pattern(st.ctx, 0, st.C)
            B.pt_calib_adamw_pattern(st.ctx, 1, 2)
        after = st.host_state()
        for name in ("g16", "w", "m", "v", "p16"):
            assert_same_bits(after[name], before[name], name)
        with pytest.raises(B.PtError):
            B.pt_calib_adamw_pattern(st.ctx, 2, 2)
    finally:
        st.close()


def test_adamw_golden_tiny_case(orc):
    from test_oracle_golden import load_golden
    rec = load_golden()
    p16_0 = np.frombuffer(rec["p16_0"], dtype=np.uint16).copy()
    n, S = p16_0.size, 16
    st = ChunkedState([n], S, init_params=False)
    try:
        st.p16.view(-1)[:n].view(torch.int16).copy_(torch.from_numpy(p16_0.view(np.int16)).cuda())
        st.w.copy_(st.p16.float())
        hp_b, _, _ = hp_pair()
        for s in (1, 2, 3):
            g = np.frombuffer(rec[f"g16_{s}"], dtype=np.uint16).copy()
            st.grad_src.view(torch.int16).copy_(torch.from_numpy(g.view(np.int16)).cuda())
            rep = st.step(hp_b)
            want_norm = np.frombuffer(rec[f"norm_{s}"], dtype=np.float64)[0]
            assert abs(rep.norm - want_norm) <= 1e-12 * want_norm
        got = st.host_state()
        w = np.frombuffer(rec["w_final"], np.float32); m = np.frombuffer(rec["m_final"], np.float32)
        v = np.frombuffer(rec["v_final"], np.float32); p = np.frombuffer(rec["p16_final"], np.uint16)
        assert np.all(np.abs(got["v"][:n] - v) <= 1e-6 * np.abs(v))
        assert np.all(np.abs(got["m"][:n] - m) <= 1e-6 * np.abs(m) + 1e-12)
        assert np.all(np.abs(got["w"][:n] - w) <= 1e-6 * np.abs(w) + 1e-10)
        assert ulp16_distance(got["p16"][:n], p).max() <= 1
    finally:
        st.close()


def end_to_end(orc, sizes, S, dtype, steps, grad_std=1e-3, scaler_b=None, scaler_o=None, inf_step=None,
               outlier_every=0, recompute_norm=False, no_decay_tensors=None):
    st = ChunkedState(sizes, S, dtype=dtype, scaler=scaler_b)
    try:
        hp_b, hp_o, hpd = hp_pair()
        mask = st.set_no_decay(tensors=no_decay_tensors) if no_decay_tensors is not None else None
        host = st.host_state()
        ost = orc.new_state(scaler_o)
        trk = ScaleTracker(host["w"], host["m"], hpd)
        fa = {k: a.copy() for k, a in host.items()}            # fp32-sequence shadow fed with GPU scalars
        reports = []
        for s in range(1, steps + 1):
            sigma = ost.loss_scale
            st.set_grads(s, std=grad_std, scale=sigma, outlier_every=outlier_every)
            if inf_step == s:
                e = synth.pick_element(synth.SEED_INF, s, st.N)
                st.grad_src.view(torch.int16)[e] = 0x7C00 if dtype == torch.float16 else 0x7F80
            st.pack()
            st.norm(recompute=recompute_norm)
            st.adamw(hp_b)
            rep = B.pt_step_report_read(st.ctx)
            k = B.pt_update_consts_read(st.ctx)
            st.end()
            g16 = st.oracle_packed(orc)                              # the oracle packs the seeded sources itself
            assert_same_bits(to_u16(st.g16).reshape(-1), g16, ("g16", s))
            orep = orc.step(hp_o, scaler_o, ost, g16, host["w"], host["m"], host["v"], host["p16"], S,
                            st.orc_dtype, threads=8, no_decay=mask)
            reports.append((rep, orep))
            assert rep.found_inf == orep.found_inf
            assert rep.loss_scale == orep.loss_scale_used
            after = B.pt_step_report_read(st.ctx)
            assert after.step == ost.t and after.loss_scale == ost.loss_scale and after.good_steps == (ost.good_steps if scaler_o else after.good_steps)
            got = st.host_state()
            if orep.found_inf:
                assert k.skip == 1
                for name in ("w", "m", "v", "p16"):
                    assert_same_bits(got[name], fa[name], name)       # untouched, bit for bit
                continue
            assert abs(rep.norm - orep.norm) <= 1e-5 * orep.norm
            assert abs(rep.norm - orep.norm) <= 1e-12 * orep.norm     # what the fp64 reduction really gives
            assert abs(rep.clip_coef - orep.clip_coef) <= 1e-12 * orep.clip_coef
            assert abs(rep.grad_mult - orep.grad_mult) <= 6e-8 * orep.grad_mult
            trk.advance(ost.t, orc.decode16(g16, st.orc_dtype).astype(np.float64) * orep.grad_mult, host["v"])
            trk.check((got["w"], got["m"], got["v"]), (host["w"], host["m"], host["v"]), tol=1e-6)
            far = check_p16(orc.decode16(got["p16"], st.orc_dtype), orc.decode16(host["p16"], st.orc_dtype),
                            host["w"], trk.W, dtype == torch.float16)
            assert far <= far_cap(got["p16"].size)          # beyond one ulp only where w's terms cancel
            # the oracle's own norm gives the very constants the device derived (the two norms agree to
            # 1e-15, far inside the fp32 rounding of grad_mult), so the fp32 sequence runs on the oracle's
            consts = orc.consts_f32(hp_o, ost.t, orep.grad_mult)
            assert same_bits(np.array(list(k.c), dtype=np.float32), consts)
            fa["g16"] = g16
            run_oracle_f32seq(orc, consts, fa, st.orc_dtype, no_decay=mask)
            for name in ("w", "m", "v", "p16"):
                assert_same_bits(got[name], fa[name], (name, s))
        return reports
    finally:
        st.close()


def test_end_to_end_gpt2_block_bf16_three_steps(orc):
    table, S = shapes.workload("gpt2_block_768")
    reps = end_to_end(orc, [n for _, n in table], S, torch.bfloat16, steps=3)
    for rep, orep in reps:
        assert abs(orep.norm - 2.662) < 0.01 and rep.clip_coef < 1.0      # 1e-3 * sqrt(7,087,872)


def test_end_to_end_ragged_with_outliers_and_recomputed_norm(orc):
    reps = end_to_end(orc, RAGGED + [300_000], 65536 + 8, torch.bfloat16, steps=3, grad_std=1e-2,
                      outlier_every=1000, recompute_norm=True)
    assert all(r.clip_coef < 1.0 for r, _ in reps)


def test_end_to_end_fp16_loss_scaling_with_a_skipped_step(orc):
    sb = B.pt_scaler_cfg(65536.0, 2.0, 0.5, 2000, 0)
    so = orc.ScalerCfg(65536.0, 2.0, 0.5, 2000, 1)
    reps = end_to_end(orc, [1_000_000, 333, 4096 * 9], 1 << 18, torch.float16, steps=6, scaler_b=sb, scaler_o=so,
                      inf_step=3)
    assert [r.found_inf for r, _ in reps] == [0, 0, 1, 0, 0, 0]
    assert [r.loss_scale for r, _ in reps] == [65536.0] * 3 + [32768.0] * 3


def test_loss_scale_growth_on_device(orc):
    sb = B.pt_scaler_cfg(4.0, 2.0, 0.5, 3, 0)
    st = ChunkedState([256], 64, dtype=torch.float16, scaler=sb, init_params=False)
    try:
        hp_b, _, _ = hp_pair()
        scales = []
        for _ in range(7):
            st.step(hp_b)
            scales.append(st.report().loss_scale)
        assert scales == [4.0, 4.0, 8.0, 8.0, 8.0, 16.0, 16.0]
        st.grad_src.view(torch.int16)[3] = np.array(0xFC00, np.uint16).view(np.int16).item()
        for want in (8.0, 4.0, 2.0, 1.0, 1.0):
            st.step(hp_b)
            r = st.report()
            assert r.loss_scale == want and r.good_steps == 0 and r.step == 7
        B.pt_ctx_set_state(st.ctx, 11, 128.0, 2)
        r = st.report()
        assert (r.step, r.loss_scale, r.good_steps) == (11, 128.0, 2)
    finally:
        st.close()


# ------------------------------------------------------------------- streamed == resident

def run_mixed(sizes, S, n_persist, n_slots, steps, dtype=torch.bfloat16, scaler=None, inf_step=None, host_update=False,
              no_decay_runs=None, orc=None, in_place=True):
    """Chunks [0, n_persist) resident, the rest in pinned host memory: streamed, in place over the link or through
    n_slots chunk buffers, or (host_update) updated by host threads.  With `orc` the oracle takes every step beside the device on
    the same seeded inputs (its own pack, norm, constants and fp32 sequence) and the final state of ALL
    chunks - resident, streamed or host-updated - must equal the oracle's bit for bit."""
    st = ChunkedState(sizes, S, dtype=dtype, scaler=scaler)
    try:
        hp_b, hp_o, _ = hp_pair()
        mask = None
        if no_decay_runs is not None:
            mask = st.set_no_decay(runs=no_decay_runs)
        C = st.C
        host = {}
        if orc is not None:
            shadow = st.host_state()
            sc_o = None if scaler is None else orc.ScalerCfg(scaler.init_scale, scaler.growth, scaler.backoff,
                                                             scaler.growth_interval, 1)
            ost = orc.new_state(sc_o)
        if n_persist < C:
            if not host_update:
                B.pt_stream_reserve(st.ctx, n_slots)
                B.pt_ctx_set_option(st.ctx, "stream_in_place", 2 if in_place else 0)
            for name, arena in (("g16", st.g16), ("p16", st.p16), ("w", st.w), ("m", st.m), ("v", st.v)):
                host[name] = [torch.empty(S, dtype=arena.dtype).pin_memory() for _ in range(n_persist, C)]
            for name, arena in (("p16", st.p16), ("w", st.w), ("m", st.m), ("v", st.v)):
                for i, c in enumerate(range(n_persist, C)):
                    host[name][i].copy_(arena[c])
                arena[n_persist:].fill_(7)                      # device copies of streamed chunks are not used
        for s in range(1, steps + 1):
            sigma = 65536.0 if scaler is not None else 1.0
            st.set_grads(s, scale=sigma)
            if inf_step == s:
                st.grad_src.view(torch.int16)[st.N // 3] = 0x7C00 if dtype == torch.float16 else 0x7F80
            if orc is not None:
                orc.step(hp_o, sc_o, ost, st.oracle_packed(orc), shadow["w"], shadow["m"], shadow["v"], shadow["p16"], S,
                         st.orc_dtype, use_f32seq=True, threads=4, no_decay=mask)
            st.pack()                                            # partials are taken on the GPU ...
            for i, c in enumerate(range(n_persist, C)):          # ... before the chunk is offloaded
                host["g16"][i].copy_(st.g16[c])
            torch.cuda.synchronize()
            st.norm()
            if n_persist < C and not host_update:
                B.pt_chunk_stream_step(st.ctx, hp_b, n_persist, C - n_persist, host["g16"], host["w"], host["m"],
                                       host["v"], host["p16"])
            if n_persist > 0:
                st.adamw(hp_b, 0, n_persist)
            if n_persist < C and host_update:          # host threads work while the GPU kernel runs
                B.pt_chunk_host_adamw_step(st.ctx, hp_b, n_persist, C - n_persist, host["g16"], host["w"], host["m"],
                                           host["v"], host["p16"], 5)
            st.end()
        torch.cuda.synchronize()
        out = {}
        for name, arena in (("p16", st.p16), ("w", st.w), ("m", st.m), ("v", st.v)):
            full = arena.clone()
            for i, c in enumerate(range(n_persist, C)):
                full[c].copy_(host[name][i])
            out[name] = full.cpu()
        out["report"] = st.report()
        if orc is not None:
            for name in ("p16", "w", "m", "v"):
                got = to_u16(out[name]).reshape(-1) if out[name].element_size() == 2 else out[name].numpy().reshape(-1)
                assert_same_bits(got, shadow[name], (name, "against the oracle", n_persist, n_slots, host_update))
            assert out["report"].step == ost.t and out["report"].loss_scale == ost.loss_scale
        return out
    finally:
        st.close()


@pytest.mark.parametrize("dtype,scaler,inf_step", [(torch.bfloat16, None, None),
                                                   (torch.float16, B.pt_scaler_cfg(65536.0, 2.0, 0.5, 2000, 0), 2)])
def test_streamed_and_host_updated_chunks_equal_the_oracle_and_the_resident_bits(orc, dtype, scaler, inf_step):
    sizes, S = [6 * 40_000 - 24], 40_000                        # 6 chunks, last one padded
    ref = run_mixed(sizes, S, 6, 2, steps=3, dtype=dtype, scaler=scaler, inf_step=inf_step, orc=orc)
    for n_persist, n_slots, in_place in ((3, 2, False), (0, 2, False), (0, 3, False), (2, 3, False), (5, 2, False),
                                         (0, 2, True), (2, 2, True), (5, 2, True)):
        got = run_mixed(sizes, S, n_persist, n_slots, steps=3, dtype=dtype, scaler=scaler, inf_step=inf_step, orc=orc,
                        in_place=in_place)
        for name in ("p16", "w", "m", "v"):
            assert torch.equal(got[name].view(torch.int16 if got[name].element_size() == 2 else torch.int32),
                               ref[name].view(torch.int16 if ref[name].element_size() == 2 else torch.int32)), \
                (name, n_persist, n_slots, in_place)
        assert got["report"].step == ref["report"].step and got["report"].loss_scale == ref["report"].loss_scale
    # the paper's placement: non-persistent chunks updated by host threads, same bits again
    for n_persist in (3, 0, 5):
        got = run_mixed(sizes, S, n_persist, 2, steps=3, dtype=dtype, scaler=scaler, inf_step=inf_step, host_update=True,
                        orc=orc)
        for name in ("p16", "w", "m", "v"):
            assert torch.equal(got[name].view(torch.int16 if got[name].element_size() == 2 else torch.int32),
                               ref[name].view(torch.int16 if ref[name].element_size() == 2 else torch.int32)), \
                ("host", name, n_persist)
        assert got["report"].step == ref["report"].step and got["report"].loss_scale == ref["report"].loss_scale


# ------------------------------------------------------------------------------- errors

def test_error_paths_return_codes_and_leave_the_context_usable():
    st = ChunkedState([1000], 512, init_params=True)
    try:
        hp_b, _, _ = hp_pair()
        with pytest.raises(B.PtError) as e:
            st.adamw(hp_b)                                       # no finalized norm yet
        assert e.value.status == B.PT_ERR_STATE
        with pytest.raises(B.PtError) as e:
            B.pt_chunk_grad_sqnorm(st.ctx, None, 1, 2, True)     # range outside the context
        assert e.value.status == B.PT_ERR_INVALID_ARG
        st.pack(); st.norm()
        with pytest.raises(B.PtError) as e:
            B.pt_chunk_adamw_step(st.ctx, hp_b, 0, 3, st.rows(st.g16), st.rows(st.w), st.rows(st.m), st.rows(st.v),
                                  st.rows(st.p16))
        assert e.value.status == B.PT_ERR_INVALID_ARG
        bad = [st.w[0][1:], st.w[1]]                             # 4-byte aligned only
        with pytest.raises(B.PtError) as e:
            B.pt_chunk_adamw_step(st.ctx, hp_b, 0, 2, st.rows(st.g16), bad, st.rows(st.m), st.rows(st.v), st.rows(st.p16))
        assert e.value.status == B.PT_ERR_ALIGNMENT
        with pytest.raises(B.PtError) as e:
            B.pt_chunk_adamw_step(st.ctx, hp_b, 0, 2, st.rows(st.g16), [st.w[0], None], st.rows(st.m), st.rows(st.v),
                                  st.rows(st.p16))
        assert e.value.status == B.PT_ERR_INVALID_ARG
        with pytest.raises(B.PtError) as e:
            B.pt_chunk_stream_step(st.ctx, hp_b, 0, 1, [st.g16[0]], [st.w[0]], [st.m[0]], [st.v[0]], [st.p16[0]])
        assert e.value.status == B.PT_ERR_STATE                  # no chunk buffers reserved
        with pytest.raises(B.PtError) as e:
            B.pt_stream_reserve(st.ctx, 1)
        assert e.value.status == B.PT_ERR_INVALID_ARG
        # overlapping segments / overrun are refused when the plan is built
        s0 = B.pt_segment(st.grad_src.data_ptr(), 0, 100, 0, 0, 0)
        s1 = B.pt_segment(st.grad_src.data_ptr(), 0, 100, 50, 0, 0)
        with pytest.raises(B.PtError) as e:
            B.pt_pack_plan_create(st.ctx, [s0, s1])
        assert e.value.status == B.PT_ERR_INVALID_ARG and "overlap" in str(e.value)
        s2 = B.pt_segment(st.grad_src.data_ptr(), 0, 100, 500, 0, 0)
        with pytest.raises(B.PtError) as e:
            B.pt_pack_plan_create(st.ctx, [s2])
        assert e.value.status == B.PT_ERR_INVALID_ARG and "overruns" in str(e.value)
        with pytest.raises(B.PtError) as e:
            B.pt_chunk_pack_grads(st.ctx, st.plan, [None, None])
        assert e.value.status == B.PT_ERR_INVALID_ARG
        # a second plan on a chunk that this step's plan has packed would replace its share of the norm: refused
        other = B.pt_pack_plan_create(st.ctx, [B.pt_segment(st.grad_src.data_ptr(), 0, 64, 0, 0, 0)])
        with pytest.raises(B.PtError) as e:
            B.pt_chunk_pack_grads(st.ctx, other, st.rows(st.g16))
        assert e.value.status == B.PT_ERR_STATE and "another plan" in str(e.value)
        st.pack()                                                # the step's own plan may pack again
        st.norm()
        # after all that the step still completes normally
        st.adamw(hp_b); st.end()
        assert st.report().step == 1
        B.pt_chunk_pack_grads(st.ctx, other, st.rows(st.g16))    # a new step: any one plan per chunk
        with pytest.raises(B.PtError) as e:
            st.pack()
        assert e.value.status == B.PT_ERR_STATE
        B.pt_pack_plan_destroy(other)                            # ... and a plan that is gone stands in nobody's way
        st.pack(); st.norm(); st.adamw(hp_b); st.end()
        assert st.report().step == 2
    finally:
        st.close()


def test_finalize_refuses_chunks_without_a_sum_from_this_step(orc):
    """Three chunks, a plan that fills only the first two: a strict finalize must refuse (chunk 2 would enter
    the norm with whatever an earlier step left), PT_FINALIZE_CARRY takes the old value on purpose, and
    pt_step_end makes every sum stale again."""
    S = 4096
    st = ChunkedState([3 * S - 8], S)
    try:
        hp_b, _, _ = hp_pair()
        st.set_grads(1)
        two = B.pt_pack_plan_create(st.ctx, [s for s in st.segs if s.chunk < 2])
        B.pt_chunk_pack_grads(st.ctx, two, st.rows(st.g16))
        with pytest.raises(B.PtError) as e:
            st.norm()
        assert e.value.status == B.PT_ERR_STATE and "chunk 2" in str(e.value)
        st.norm(finalize=B.PT_FINALIZE_CARRY)                   # chunk 2 never had gradients: its sum is the initial zero
        words = to_u16(st.grad_src[:2 * S])
        want = orc.sqnorm(words, st.orc_dtype, block=S)
        assert abs(st.report().sqnorm - want) <= 1e-12 * want
        st.adamw(hp_b, 0, 2); st.end()
        with pytest.raises(B.PtError) as e:                      # a new step: the old sums no longer count
            st.norm()
        assert e.value.status == B.PT_ERR_STATE and "chunk 0" in str(e.value)
        B.pt_chunk_grad_sqnorm(st.ctx, st.rows(st.g16), 2, 1, False)   # recompute chunk 2 alone ...
        B.pt_chunk_pack_grads(st.ctx, two, st.rows(st.g16))            # ... the plan covers 0 and 1
        st.norm()
        assert abs(st.report().sqnorm - want) <= 1e-12 * want
        st.end()
        B.pt_pack_plan_destroy(two)
    finally:
        st.close()


# --------------------------------------------------- paper-faithful (no-split, grouped) layout

@pytest.mark.parametrize("separate_allocs", [True, False])
def test_grouped_layout_pack_and_step_against_oracle(orc, separate_allocs):
    from oracle import layout as OL
    # embedding, three "blocks" (one larger than the others), tail tensors; odd sizes on purpose
    sizes = [40_000, 5, 9_000, 9_001, 77, 9_000, 30_011, 3, 9_000, 9_000, 64, 1_000, 17]
    gids = [None, None, 0, 0, 0, 1, 1, 1, 2, 2, 2, None, None]
    S, n_chunks, waste = B.pt_chunk_size_search(sizes, gids, 0, 1 << 14, 1 << 10)
    assert (S, n_chunks, waste) == OL.chunk_size_search(sizes, gids, 0, 1 << 14, 1 << 10)
    place, _, _ = OL.layout_grouped(sizes, gids, S)
    segs, C, _ = B.pt_layout_grouped(sizes, gids, S)
    N = sum(sizes)
    dev = "cuda"
    if separate_allocs:
        tensors = [torch.empty(n, dtype=torch.bfloat16, device=dev) for n in sizes]
    else:
        flat = torch.empty(N, dtype=torch.bfloat16, device=dev)
        offs = np.cumsum([0] + sizes[:-1]).tolist()
        tensors = [flat[o:o + n] for o, n in zip(offs, sizes)]
    for s in segs:
        s.src = tensors[s.tensor].data_ptr()
    ctx = B.pt_ctx_create(B.PT_BF16, S, C, None)
    plan = B.pt_pack_plan_create(ctx, segs)
    try:
        g16 = torch.zeros(C, S, dtype=torch.bfloat16, device=dev)
        p16 = torch.zeros(C, S, dtype=torch.bfloat16, device=dev)
        rows = lambda a: [a[c] for c in range(C)]

        def scatter(per_tensor_u16):                       # the oracle's placements, applied with numpy
            out = np.zeros((C, S), np.uint16)
            for t, pl in enumerate(place):
                if pl is not None:
                    out[pl[0], pl[1]:pl[1] + sizes[t]] = per_tensor_u16[t]
            return out

        # parameters: generated per tensor, placed by the oracle's layout
        params = [synth.normal_16(synth.SEED_PARAMS, 0, t, 0, n, 0.02, torch.bfloat16, dev) for t, n in enumerate(sizes)]
        p_host = scatter([to_u16(x) for x in params])
        p16.view(torch.int16).copy_(torch.from_numpy(p_host.view(np.int16)).to(dev))
        w = p16.float(); m = torch.zeros_like(w); v = torch.zeros_like(w)
        hp_b, hp_o, hpd = hp_pair()
        host = dict(p16=p_host.reshape(-1).copy(), w=w.cpu().numpy().reshape(-1).copy(),
                    m=np.zeros(C * S, np.float32), v=np.zeros(C * S, np.float32))
        ost = orc.new_state(None)
        trk = ScaleTracker(host["w"], host["m"], hpd)
        for step in (1, 2):
            for t, n in enumerate(sizes):
                synth.normal_16(synth.SEED_GRADS, step, t, 0, n, 1e-2, torch.bfloat16, dev, out=tensors[t])
            want_g = scatter([to_u16(x) for x in tensors])
            g16.view(torch.int16).fill_(0)
            B.pt_chunk_pack_grads(ctx, plan, rows(g16))
            assert same_bits(to_u16(g16), want_g)                       # pack: bit-exact, gaps untouched
            B.pt_chunk_grad_sqnorm(ctx, None, 0, C, True)
            B.pt_chunk_adamw_step(ctx, hp_b, 0, C, rows(g16), rows(w), rows(m), rows(v), rows(p16))
            rep = B.pt_step_report_read(ctx)
            B.pt_step_end(ctx)
            orep = orc.step(hp_o, None, ost, want_g.reshape(-1), host["w"], host["m"], host["v"], host["p16"], S,
                            orc.BF16, threads=4)
            assert abs(rep.norm - orep.norm) <= 1e-12 * orep.norm and rep.clip_coef < 1.0
            trk.advance(step, orc.decode16(want_g.reshape(-1), orc.BF16).astype(np.float64) * orep.grad_mult, host["v"])
            got = (w.cpu().numpy().reshape(-1), m.cpu().numpy().reshape(-1), v.cpu().numpy().reshape(-1))
            trk.check(got, (host["w"], host["m"], host["v"]), tol=1e-6)
            check_p16(orc.decode16(to_u16(p16).reshape(-1), orc.BF16), orc.decode16(host["p16"], orc.BF16), host["w"],
                      trk.W, False)
        # updated parameters go back to the model's tensors through the inverse copy
        for x in tensors:
            x.zero_()
        B.pt_chunk_unpack(ctx, plan, rows(p16))
        back = to_u16(p16)
        for t, pl in enumerate(place):
            if pl is not None:
                assert same_bits(to_u16(tensors[t]), back[pl[0], pl[1]:pl[1] + sizes[t]])
    finally:
        torch.cuda.synchronize()
        B.pt_pack_plan_destroy(plan)
        B.pt_ctx_destroy(ctx)


# ----------------------------------------------------- the step is capturable in a HIP graph

def test_whole_step_replays_from_a_hip_graph_bit_for_bit():
    """The hot calls neither allocate nor synchronise once the pointer tables are bound, so a
    step can be captured and replayed; every replay matches the eager path bit for bit, with
    eager work and synchronisations between replays."""
    sizes, S = [300_000, 4099, 65_536], 1 << 16
    a = ChunkedState(sizes, S)                 # eager
    b = ChunkedState(sizes, S)                 # captured
    try:
        hp_b, _, _ = hp_pair()
        side = torch.cuda.Stream()

        def step_on(st, stream):
            B.pt_chunk_pack_grads(st.ctx, st.plan, st.rows(st.g16), stream)
            B.pt_chunk_grad_sqnorm(st.ctx, None, 0, st.C, True, stream)
            B.pt_chunk_adamw_step(st.ctx, hp_b, 0, st.C, st.rows(st.g16), st.rows(st.w), st.rows(st.m), st.rows(st.v),
                                  st.rows(st.p16), stream)
            B.pt_step_end(st.ctx, stream)

        for st in (a, b):
            st.set_grads(1)
        torch.cuda.synchronize()
        step_on(a, torch.cuda.current_stream())
        with torch.cuda.stream(side):
            step_on(b, side)                   # binds the pointer tables outside the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            step_on(b, torch.cuda.current_stream())
        torch.cuda.synchronize()
        # the capture itself did not run anything: b is still one step behind nothing, same as a
        for s in (2, 3, 4, 5):
            for st in (a, b):
                st.set_grads(s)
            torch.cuda.synchronize()
            step_on(a, torch.cuda.current_stream())
            graph.replay()
            torch.cuda.synchronize()
            ha, hb = a.host_state(), b.host_state()
            for name in ("g16", "w", "m", "v", "p16"):
                assert_same_bits(hb[name], ha[name], (name, s))
            ra, rb = a.report(), b.report()
            assert (ra.step, ra.norm, ra.found_inf) == (rb.step, rb.norm, rb.found_inf) and ra.step == s
    finally:
        a.close(); b.close()


# ------------------------------------------------------------- hyper-parameter corners, resume

@pytest.mark.parametrize("kw", [dict(max_norm=0.0), dict(lr=0.0), dict(beta1=0.0, beta2=0.0), dict(weight_decay=0.0),
                                dict(eps=1e-3, max_norm=1e9), dict(lr=3e-2, beta1=0.5, beta2=0.999, weight_decay=1.0)])
def test_hyper_parameter_corners_end_to_end(orc, kw):
    st = ChunkedState([70_000, 33, 8_200], 1 << 15)
    try:
        hp_b, hp_o, hpd = hp_pair(**kw)
        host = st.host_state()
        fa = {k: a.copy() for k, a in host.items()}
        ost = orc.new_state(None)
        trk = ScaleTracker(host["w"], host["m"], hpd)
        for s in (1, 2, 3):
            st.set_grads(s, std=1e-2)
            st.pack(); st.norm(); st.adamw(hp_b)
            rep = B.pt_step_report_read(st.ctx)
            k = B.pt_update_consts_read(st.ctx)
            st.end()
            g16 = st.oracle_packed(orc)
            assert_same_bits(to_u16(st.g16).reshape(-1), g16, ("g16", s))
            orep = orc.step(hp_o, None, ost, g16, host["w"], host["m"], host["v"], host["p16"], st.S, orc.BF16, threads=4)
            assert abs(rep.clip_coef - orep.clip_coef) <= 1e-12 * orep.clip_coef
            if hpd["max_norm"] <= 0 or hpd["max_norm"] > 1e6:
                assert rep.clip_coef == 1.0 and rep.grad_mult == 1.0
            got = st.host_state()
            trk.advance(s, orc.decode16(g16, orc.BF16).astype(np.float64) * orep.grad_mult, host["v"])
            trk.check((got["w"], got["m"], got["v"]), (host["w"], host["m"], host["v"]), tol=1e-6)
            consts = orc.consts_f32(hp_o, ost.t, orep.grad_mult)            # the oracle's own constants
            assert same_bits(np.array(list(k.c), dtype=np.float32), consts)
            fa["g16"] = g16
            run_oracle_f32seq(orc, consts, fa, orc.BF16)
            for name in ("w", "m", "v", "p16"):
                assert_same_bits(got[name], fa[name], (name, s, kw))
    finally:
        st.close()


def test_resume_from_saved_state_gives_the_same_bits():
    sizes, S = [50_000, 4_100], 1 << 14
    sb = B.pt_scaler_cfg(1024.0, 2.0, 0.5, 2, 0)              # grows every 2 good steps: the state matters
    a = ChunkedState(sizes, S, dtype=torch.float16, scaler=sb)
    b = None
    try:
        hp_b, _, _ = hp_pair()
        scale = 1024.0
        for s in (1, 2, 3):
            a.set_grads(s, scale=scale)
            a.step(hp_b)
            scale = a.report().loss_scale
        r = a.report()
        assert (r.step, r.loss_scale, r.good_steps) == (3, 2048.0, 1)
        snap = {k: getattr(a, k).clone() for k in ("p16", "w", "m", "v")}
        # a fresh context resumed from the saved arrays and the three saved scalars
        b = ChunkedState(sizes, S, dtype=torch.float16, scaler=sb, init_params=False)
        for k, t in snap.items():
            getattr(b, k).copy_(t)
        B.pt_ctx_set_state(b.ctx, r.step, r.loss_scale, r.good_steps)
        for s in (4, 5, 6):
            for st in (a, b):
                st.set_grads(s, scale=scale)
                st.step(hp_b)
            assert a.report().loss_scale == b.report().loss_scale
            scale = a.report().loss_scale
        ha, hb = a.host_state(), b.host_state()
        for name in ("w", "m", "v", "p16"):
            assert_same_bits(hb[name], ha[name], name)
        ra, rb = a.report(), b.report()
        assert (ra.step, ra.loss_scale, ra.good_steps) == (rb.step, rb.loss_scale, rb.good_steps) == (6, 8192.0, 0)
    finally:
        a.close()
        if b is not None:
            b.close()


# ------------------------------------------------------------------------- arena placement

def test_spread_arenas_gives_zeroed_tensors_and_returns_the_spacers():
    from paper_2406_08334_amd.arena import spread_arenas
    torch.cuda.empty_cache()
    free0, _ = torch.cuda.mem_get_info()
    specs = [((3, 1 << 20), torch.bfloat16), ((3, 1 << 20), torch.float32), ((5,), torch.float32)]
    for gap in (0, 64 << 20, None):
        arenas = spread_arenas(specs, gap_bytes=gap)
        assert [tuple(a.shape) for a in arenas] == [(3, 1 << 20), (3, 1 << 20), (5,)]
        assert [a.dtype for a in arenas] == [torch.bfloat16, torch.float32, torch.float32]
        assert all(a.is_cuda and a.is_contiguous() and not bool(a.view(-1).any()) for a in arenas)
        assert all(a.data_ptr() % 256 == 0 for a in arenas)
        free1, _ = torch.cuda.mem_get_info()
        assert free0 - free1 < (1 << 30)               # the spacers (up to 20 GiB each) went back to the driver
        del arenas
        torch.cuda.empty_cache()
