"""GPU parity on inputs the layouts never produce, long runs and concurrent contexts:
random segment tables (gaps, partial tensors, shuffled order, odd alignments) through pack,
unpack and accumulate; forty steps with loss-scale back-offs and growths, bit for bit;
two contexts stepping on two streams at once."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2406_08334_amd import binding as B
from paper_2406_08334_amd import synth

from gpu_harness import ChunkedState, hp_pair, to_u16, same_bits, assert_same_bits

pytestmark = pytest.mark.gpu


def random_table(rng, C, S, n_tensors, max_len):
    """Segments at random, non-overlapping places: every chunk is cut into random pieces, a random
    subset of the pieces receives a random sub-range of a random tensor."""
    sizes = [int(rng.integers(1, max_len)) for _ in range(n_tensors)]
    table = []
    for c in range(C):
        cuts = np.unique(np.concatenate(([0, S], rng.integers(0, S, 24))))
        for lo, hi in zip(cuts[:-1], cuts[1:]):
            if rng.random() < 0.35:
                continue                                            # a gap
            t = int(rng.integers(0, n_tensors))
            n = int(min(hi - lo, sizes[t]))
            n = int(rng.integers(1, n + 1))
            so = int(rng.integers(0, sizes[t] - n + 1))
            table.append((t, so, n, c, int(lo)))
    order = rng.permutation(len(table))
    return sizes, [table[i] for i in order]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("seed,C,S", [(1, 3, 40_000), (2, 2, 8192 * 3 + 8), (3, 5, 1000)])
def test_random_segment_tables_through_pack_unpack_and_norm(orc, dtype, seed, C, S):
    rng = np.random.default_rng(seed)
    sizes, table = random_table(rng, C, S, n_tensors=9, max_len=30_000)
    orc_dtype = orc.BF16 if dtype == torch.bfloat16 else orc.FP16
    # tensors: random finite 16-bit patterns
    host_t = []
    for n in sizes:
        w = rng.integers(0, 1 << 16, n, dtype=np.uint16)
        exp = 0x7F80 if dtype == torch.bfloat16 else 0x7C00
        w[(w & exp) == exp] &= np.uint16(0x3FFF)                   # no inf / NaN
        host_t.append(w)
    dev_t = [torch.from_numpy(w.view(np.int16)).cuda().view(dtype) for w in host_t]
    ctx = B.pt_ctx_create(B.PT_BF16 if dtype == torch.bfloat16 else B.PT_FP16, S, C, None)
    plan = None
    try:
        segs = [B.pt_segment(dev_t[t].data_ptr(), so, n, co, c, t) for t, so, n, c, co in table]
        plan = B.pt_pack_plan_create(ctx, segs)
        chunks = torch.full((C, S), 0.5, dtype=dtype, device="cuda")       # sentinel in the gaps
        sent = int(to_u16(chunks[0, :1])[0])
        B.pt_chunk_pack_grads(ctx, plan, [chunks[c] for c in range(C)])
        B.pt_chunk_grad_sqnorm(ctx, None, 0, C, B.PT_FINALIZE_CARRY)     # a random table may leave a chunk untouched
        rep = B.pt_step_report_read(ctx)
        want = np.full((C, S), sent, np.uint16)
        orc.pack_segments([(host_t[t], so, n, c, co) for t, so, n, c, co in table], want)
        assert_same_bits(to_u16(chunks), want, "pack")
        covered = np.zeros((C, S), np.uint16)
        orc.pack_segments([(host_t[t], so, n, c, co) for t, so, n, c, co in table], covered)
        want_sq = orc.sqnorm(covered.reshape(-1), orc_dtype, block=S, threads=4)      # gaps hold zero here
        assert rep.found_inf == 0 and abs(rep.sqnorm - want_sq) <= 1e-12 * want_sq
        # inverse copy into fresh tensors: exactly the covered source ranges come back
        back = [torch.full((n,), 0.25, dtype=dtype, device="cuda") for n in sizes]
        q = int(to_u16(back[0][:1])[0])
        segs_b = [B.pt_segment(back[t].data_ptr(), so, n, co, c, t) for t, so, n, c, co in table]
        plan_b = B.pt_pack_plan_create(ctx, segs_b)
        B.pt_chunk_unpack(ctx, plan_b, [chunks[c] for c in range(C)])
        torch.cuda.synchronize()
        B.pt_pack_plan_destroy(plan_b)
        exp_back = [np.full(n, q, np.uint16) for n in sizes]
        for t, so, n, c, co in table:          # a source range used twice receives equal words both times
            exp_back[t][so:so + n] = host_t[t][so:so + n]
        for t in range(len(sizes)):
            assert_same_bits(to_u16(back[t]), exp_back[t], ("unpack", t))
    finally:
        torch.cuda.synchronize()
        if plan is not None:
            B.pt_pack_plan_destroy(plan)
        B.pt_ctx_destroy(ctx)


@pytest.mark.parametrize("seed,C,S", [(4, 3, 40_000), (5, 2, 4096 * 5 + 24)])
def test_random_segment_tables_through_accumulate(orc, seed, C, S):
    rng = np.random.default_rng(seed)
    sizes, table = random_table(rng, C, S, n_tensors=7, max_len=25_000)
    ctx = B.pt_ctx_create(B.PT_BF16, S, C, None)
    B.pt_ctx_set_option(ctx, "grad_fp32", 1)
    plan = None
    try:
        dev_t = [torch.empty(n, dtype=torch.bfloat16, device="cuda") for n in sizes]
        segs = [B.pt_segment(dev_t[t].data_ptr(), so, n, co, c, t) for t, so, n, c, co in table]
        plan = B.pt_pack_plan_create(ctx, segs)
        acc = torch.full((C, S), -3.0, dtype=torch.float32, device="cuda")
        want = np.full(C * S, -3.0, np.float32)
        for k in range(3):
            host_t = []
            for i, n in enumerate(sizes):
                dev_t[i].normal_(0, 1.0, generator=None)
                host_t.append(to_u16(dev_t[i]).copy())
            B.pt_chunk_accum_grads(ctx, plan, [acc[c] for c in range(C)], k == 0, k == 2)
            for t, so, n, c, co in table:
                view = want[c * S + co: c * S + co + n]
                part = view.copy()
                orc.accum_f32(host_t[t][so:so + n], part, orc.BF16, overwrite=(k == 0))
                view[:] = part
            assert_same_bits(acc.cpu().numpy().reshape(-1), want, ("accumulate", k))
        B.pt_chunk_grad_sqnorm(ctx, None, 0, C, B.PT_FINALIZE_CARRY)
        rep = B.pt_step_report_read(ctx)
        cov = np.zeros(C * S, np.float32)
        for t, so, n, c, co in table:
            cov[c * S + co: c * S + co + n] = want[c * S + co: c * S + co + n]
        want_sq = orc.sqnorm_f32(cov, block=S, threads=4)
        assert abs(rep.sqnorm - want_sq) <= 1e-12 * want_sq
    finally:
        torch.cuda.synchronize()
        if plan is not None:
            B.pt_pack_plan_destroy(plan)
        B.pt_ctx_destroy(ctx)


def test_forty_steps_with_loss_scale_events_stay_bit_exact(orc):
    """growth every 3 good steps, an inf every 7th step: back-offs and growths interleave; the GPU
    state follows the oracle's fp32 sequence bit for bit through all of it"""
    sb = B.pt_scaler_cfg(1024.0, 2.0, 0.5, 3, 0)
    so = orc.ScalerCfg(1024.0, 2.0, 0.5, 3, 1)
    S = 4096 * 2 + 40
    st = ChunkedState([2 * S + 1000, 77], S, dtype=torch.float16, scaler=sb)
    try:
        hp_b, hp_o, _ = hp_pair(lr=3e-4)
        host = st.host_state()
        ost = orc.new_state(so)
        scales = []
        for s in range(1, 41):
            sigma = ost.loss_scale
            scales.append(sigma)
            st.set_grads(s, scale=sigma)
            if s % 7 == 0:
                st.grad_src.view(torch.int16)[(s * 131) % st.N] = 0x7C00
            st.pack(); st.norm(); st.adamw(hp_b)
            rep = B.pt_step_report_read(st.ctx)
            k = B.pt_update_consts_read(st.ctx)
            st.end()
            g16 = st.oracle_packed(orc)                              # the oracle packs the seeded sources itself
            assert_same_bits(to_u16(st.g16).reshape(-1), g16, ("g16", s))
            # the whole step in the oracle, fp32 sequence, its own norm, constants and loss-scale machine
            orep = orc.step(hp_o, so, ost, g16, host["w"], host["m"], host["v"], host["p16"], st.S, orc.FP16,
                            use_f32seq=True, threads=4)
            assert rep.found_inf == orep.found_inf == int(s % 7 == 0) and rep.loss_scale == orep.loss_scale_used == sigma
            if not orep.found_inf:
                assert same_bits(np.array(list(k.c), np.float32), orc.consts_f32(hp_o, ost.t, orep.grad_mult))
            after = B.pt_step_report_read(st.ctx)
            assert (after.step, after.loss_scale, after.good_steps) == (ost.t, ost.loss_scale, ost.good_steps), s
            got = st.host_state()
            for name in ("w", "m", "v", "p16"):
                assert_same_bits(got[name], host[name], (name, s))
        assert ost.t == 35 and len(set(scales)) >= 3            # the scale really moved both ways
    finally:
        st.close()


def test_two_contexts_on_two_streams_do_not_disturb_each_other(orc):
    sizes, S = [300_000, 4099, 65_536], 1 << 16
    solo = [ChunkedState(sizes, S, seed=i) for i in (0, 1)]
    duo = [ChunkedState(sizes, S, seed=i) for i in (0, 1)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    try:
        hp_b, _, _ = hp_pair()

        def step_on(st, stream):
            B.pt_chunk_pack_grads(st.ctx, st.plan, st.rows(st.g16), stream)
            B.pt_chunk_grad_sqnorm(st.ctx, None, 0, st.C, True, stream)
            B.pt_chunk_adamw_step(st.ctx, hp_b, 0, st.C, st.rows(st.g16), st.rows(st.w), st.rows(st.m), st.rows(st.v),
                                  st.rows(st.p16), stream)
            B.pt_step_end(st.ctx, stream)

        for s in (1, 2, 3, 4):
            for st in solo + duo:
                st.set_grads(s)
            torch.cuda.synchronize()
            for st in solo:                                     # one after the other, default stream
                step_on(st, torch.cuda.current_stream())
                torch.cuda.synchronize()
            for st, stream in zip(duo, streams):                # both enqueued before either is waited for
                step_on(st, stream)
            torch.cuda.synchronize()
        for a, b in zip(solo, duo):
            ha, hb = a.host_state(), b.host_state()
            for name in ("g16", "w", "m", "v", "p16"):
                assert_same_bits(hb[name], ha[name], name)
            assert a.report().norm == b.report().norm
    finally:
        for st in solo + duo:
            st.close()


def test_stream_reserve_tries_its_copy_streams_out_and_ends_with_a_pair_that_overlaps():
    """A stream keeps the copy engine of its first copy, and two copy streams that took the same one carry one
    direction of the link at a time.  pt_stream_reserve makes the first copies itself, side by side, then measures
    (one copy up, one down, both at once) and replaces a pair that does not overlap.  Here: a process that has created
    and destroyed other streams right before, several contexts in a row - every reservation must end with an
    overlapping pair; the replacement forced from the host; and small chunk buffers, which skip the test."""
    S = 1 << 22                                   # 64 MiB chunk buffers: large enough to measure
    ctxs = []
    try:
        for k in range(3):
            junk = [torch.cuda.Stream() for _ in range(k + 1)]
            for s in junk:
                with torch.cuda.stream(s):
                    torch.zeros(8, device="cuda")
            torch.cuda.synchronize()
            del junk
            ctx = B.pt_ctx_create(B.PT_BF16, S, 4, None)
            ctxs.append(ctx)
            B.pt_stream_reserve(ctx, 2)
            st = B.pt_stream_status(ctx)
            print(f"[stream self-test] context {k}: {st}", flush=True)
            assert st["duplex_tested"] and st["duplex_ok"] and 1 <= st["attempts"] <= 6, st
        # the replacement itself, forced from the host: two stream pairs rejected whatever they measure, the third
        # kept; the streamed update through the replaced stream still gives the resident bits
        forced = B.pt_ctx_create(B.PT_BF16, S, 4, None)
        ctxs.append(forced)
        B.pt_ctx_set_option(forced, "stream_in_place", 0)          # through the copy streams
        B.pt_ctx_set_option(forced, "stream_test_reject", 2)
        B.pt_stream_reserve(forced, 2)
        st = B.pt_stream_status(forced)
        assert st["duplex_tested"] and st["duplex_ok"] and st["attempts"] == 3, st
        hp_b, _, _ = hp_pair()
        dev = {k: torch.zeros(2, S, dtype=dt, device="cuda") for k, dt in
               (("g", torch.bfloat16), ("p", torch.bfloat16), ("w", torch.float32), ("m", torch.float32), ("v", torch.float32))}
        synth.normal_16(synth.SEED_GRADS, 1, 0, 0, 2 * S, 1e-3, torch.bfloat16, "cuda", out=dev["g"].view(-1))
        synth.normal_16(synth.SEED_PARAMS, 0, 0, 0, 2 * S, 0.02, torch.bfloat16, "cuda", out=dev["p"].view(-1))
        dev["w"].copy_(dev["p"])
        host = {k: [t[c].cpu().pin_memory() for c in range(2)] for k, t in dev.items()}
        rows = lambda k: [dev[k][0], dev[k][1]]

        def step_and_compare(tag):
            B.pt_chunk_grad_sqnorm(forced, [dev["g"][0], dev["g"][1], None, None], 0, 2, False)
            B.pt_chunk_grad_sqnorm(forced, None, 0, 4, B.PT_FINALIZE_CARRY)
            B.pt_chunk_stream_step(forced, hp_b, 2, 2, host["g"], host["w"], host["m"], host["v"], host["p"])
            B.pt_chunk_adamw_step(forced, hp_b, 0, 2, rows("g"), rows("w"), rows("m"), rows("v"), rows("p"))
            B.pt_step_end(forced)
            torch.cuda.synchronize()
            for k in ("w", "m", "v", "p"):
                for c in range(2):
                    view = torch.int16 if k == "p" else torch.int32
                    assert torch.equal(host[k][c].view(view), dev[k][c].cpu().view(view)), (tag, k, c)
        step_and_compare("first step")
        assert B.pt_stream_status(forced)["rebuilds"] == 0
        # A step that ran with its two directions behind each other makes the next call replace the side streams;
        # here the verdict on the finished step is forced from the host.  Same bits through the new streams.
        B.pt_ctx_set_option(forced, "stream_test_unhealthy", 1)
        step_and_compare("step after the verdict")
        st = B.pt_stream_status(forced)
        assert st["rebuilds"] == 1 and st["duplex_tested"], st
        step_and_compare("a further step")
        assert B.pt_stream_status(forced)["rebuilds"] == 1
        small = B.pt_ctx_create(B.PT_BF16, 4096, 2, None)
        ctxs.append(small)
        B.pt_stream_reserve(small, 2)
        assert B.pt_stream_status(small) == {"duplex_tested": False, "duplex_ok": False, "attempts": 0, "rebuilds": 0}
    finally:
        torch.cuda.synchronize()
        for ctx in ctxs:
            B.pt_ctx_destroy(ctx)


@pytest.mark.parametrize("dtype,grad_fp32", [(torch.bfloat16, False), (torch.float16, True)])
@pytest.mark.parametrize("S,n_host", [(8, 1), (1024, 3), (5000, 17)])      # one unit; whole tiles; ragged, two launches
@pytest.mark.parametrize("memory", ["pinned", "shared", "offset", "pageable"])
@pytest.mark.parametrize("inf", [False, True])
def test_streamed_update_by_the_kind_of_host_memory(dtype, grad_fp32, S, n_host, memory, inf):
    """Pinned and aligned arrays are updated in place (also where gradient and parameters share one), pinned ones off the
    alignment and pageable ones through the chunk buffers: the bits of the resident update, skipped steps included."""
    if memory == "shared" and grad_fp32:
        pytest.skip("fp32 gradients and 16-bit parameters are two arrays")
    st = ChunkedState([S * n_host - 3 if S > 8 else 5], S, dtype=dtype, grad_fp32=grad_fp32)
    try:
        assert st.C == n_host
        hp_b, _, _ = hp_pair()
        st.set_no_decay(runs=[(c, 1, S // 2) for c in range(n_host)])
        st.set_grads(1)
        if grad_fp32:
            st.accum(True, True)
        else:
            st.pack()
        arenas = {"g": st.grads, "w": st.w, "m": st.m, "v": st.v, "p": st.p16}

        def host_copy(row):
            if memory == "pageable":
                return row.cpu()
            off = 1 if memory == "offset" else 0
            t = torch.empty(S + off, dtype=row.dtype, pin_memory=True)[off:]
            return t.copy_(row)
        host = {k: [host_copy(a[c]) for c in range(n_host)] for k, a in arenas.items()}
        if memory == "shared":
            host["p"] = host["g"]
        B.pt_stream_reserve(st.ctx, 2)
        B.pt_step_override(st.ctx, 0.5, inf)
        stream = lambda: B.pt_chunk_stream_step(st.ctx, hp_b, 0, n_host, host["g"], host["w"], host["m"], host["v"], host["p"])
        B.pt_ctx_set_option(st.ctx, "stream_in_place", 2)
        if memory in ("pinned", "shared"):
            stream()
        else:
            with pytest.raises(B.PtError) as e:
                stream()
            assert e.value.status == B.PT_ERR_UNSUPPORTED
            B.pt_ctx_set_option(st.ctx, "stream_in_place", 1)
            stream()
        torch.cuda.synchronize()
        st.adamw(hp_b)
        st.end()
        torch.cuda.synchronize()
        for k in ("w", "m", "v", "p"):
            for c in range(n_host):
                bits = torch.int16 if k == "p" else torch.int32
                assert torch.equal(host[k][c].view(bits), arenas[k][c].cpu().view(bits)), (k, c)
    finally:
        st.close()


@pytest.mark.parametrize("tiles", [1, 511, 4096, 4097, 8193])        # one workgroup's lanes, one workgroup, segments
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("inf", [False, True])
def test_norm_of_many_partial_sums(tiles, dtype, inf):
    """The sum over a chunk's partials in one workgroup or in segments, several plans of one step put off together, from
    two streams: against the sum in 64 bits.  Squares of 16-bit words are exact there and every partial is a sum of
    non-negative terms, so n terms in any order are within n * 2^-53 of each other."""
    S = max(8, (tiles - 1) * 1024 + 8)
    C = 3
    ctx = B.pt_ctx_create(B.PT_BF16 if dtype == torch.bfloat16 else B.PT_FP16, S, C, None)
    plans = []
    try:
        B.pt_ctx_set_option(ctx, "pack_tile_elems", 1024)
        src = torch.empty(C, S, dtype=dtype, device="cuda")
        synth.normal_16(synth.SEED_GRADS, 1, 0, 0, C * S, 1e-2, dtype, "cuda", out=src.view(-1))
        if inf:
            src[1, S - 1] = float("inf")
        dst = torch.zeros(C, S, dtype=dtype, device="cuda")
        plans = [B.pt_pack_plan_create(ctx, [B.pt_segment(src[c].data_ptr(), 0, S, 0, c, c) for c in cs]) for cs in ((0, 2), (1,))]
        rows = [dst[c] for c in range(C)]
        side = torch.cuda.Stream()
        torch.cuda.synchronize()

        def want():
            return float(src.double().square().sum())

        def check(rep):
            assert rep.found_inf == int(inf)
            assert inf or abs(rep.sqnorm - want()) <= C * S * 2.0 ** -53 * want()
        B.pt_chunk_pack_grads(ctx, plans[0], rows)
        B.pt_chunk_pack_grads(ctx, plans[1], rows, side)
        torch.cuda.current_stream().wait_stream(side)
        B.pt_chunk_grad_sqnorm(ctx, None, 0, C, True)
        check(B.pt_step_report_read(ctx))
        assert torch.equal(dst.view(torch.int16), src.view(torch.int16))
        B.pt_step_end(ctx)
        # a finalize that waits takes the sums as they were when it was asked for
        old = want()
        for k in range(2):
            B.pt_chunk_pack_grads(ctx, plans[k], rows)
        B.pt_chunk_grad_sqnorm(ctx, None, 0, C, True)
        src[0] *= 2
        side.wait_stream(torch.cuda.current_stream())
        B.pt_chunk_pack_grads(ctx, plans[0], rows, side)
        torch.cuda.current_stream().wait_stream(side)
        # the report reads what the finalize published: the pack that came after it is not in the norm
        rep = B.pt_step_report_read(ctx)
        assert rep.found_inf == int(inf) and (inf or abs(rep.sqnorm - old) <= C * S * 2.0 ** -53 * old)
        B.pt_step_end(ctx)
        # recomputed from the chunks, in two calls that are put off together
        B.pt_chunk_grad_sqnorm(ctx, rows, 0, 2, False)
        B.pt_chunk_grad_sqnorm(ctx, rows, 2, 1, True)
        check(B.pt_step_report_read(ctx))
        B.pt_step_end(ctx)
    finally:
        torch.cuda.synchronize()
        for p in plans:
            B.pt_pack_plan_destroy(p)
        B.pt_ctx_destroy(ctx)


def test_plan_destroyed_before_its_partial_sums_were_read():
    """The sums of a plan that is destroyed before the norm is finalized still enter it."""
    st = ChunkedState([5000, 3000], 4096)
    try:
        st.set_grads(1, std=1e-2)
        st.pack()
        B.pt_pack_plan_destroy(st.plan)
        st.plan = B.pt_pack_plan_create(st.ctx, st.segs)
        st.norm()
        want = float(st.grad_src.double().square().sum())
        assert abs(st.report().sqnorm - want) <= 8000 * 2.0 ** -53 * want
    finally:
        st.close()


@pytest.mark.parametrize("S,C", [(8, 1), (8, 17), (32768 * 513, 3), (4096 * 32768, 1), (4096 * 32768 + 8, 1)])   # to two segments
@pytest.mark.parametrize("inf", [False, True])
def test_norm_without_a_context_by_size(S, C, inf):
    """Chunks of one block, of more than a lane's share, of one and of two segments: the same bits as the context's recompute, call
    after call."""
    g = torch.empty(C, S, dtype=torch.bfloat16, device="cuda")
    synth.normal_16(synth.SEED_GRADS, 1, 0, 0, C * S, 1e-3, torch.bfloat16, "cuda", out=g.view(-1))
    if inf:
        g[C - 1, S - 1] = float("-inf")
    ctx = B.pt_ctx_create(B.PT_BF16, S, C, None)
    try:
        B.pt_chunk_grad_sqnorm(ctx, [g[c] for c in range(C)], 0, C, True)
        rep = B.pt_step_report_read(ctx)
        for _ in range(3):
            out, found = torch.zeros(2, dtype=torch.float64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
            B.pt_chunk_grad_sqnorm_noalloc(g, B.PT_BF16, S, C, 1.0, out, found)
            assert int(found[0]) == rep.found_inf == int(inf)
            assert inf or (float(out[0]), float(out[1])) == (rep.sqnorm, rep.norm)
        want = float(g.double().square().sum())
        assert inf or abs(rep.sqnorm - want) <= C * S * 2.0 ** -53 * want
    finally:
        B.pt_ctx_destroy(ctx)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 505, 1023, 1024, 1025, 2047, 2048, 2049, 4099])
def test_pack_unpack_and_accumulate_at_the_edges_of_a_tile(dtype, n):
    """Every alignment of the tensor against the chunk (in elements), lengths around one wave's tile, with the words
    around the tensor's place left alone."""
    S = 8192
    gaps = [(s, d) for s in range(8) for d in range(8)]
    C = len(gaps)
    src = torch.zeros(C, S, dtype=dtype, device="cuda")
    synth.normal_16(synth.SEED_GRADS, 1, 0, 0, C * S, 1e-2, dtype, "cuda", out=src.view(-1))
    segs = [B.pt_segment(src[c].data_ptr(), s, n, d, c, c) for c, (s, d) in enumerate(gaps)]
    for fp32 in (False, True):
        ctx = B.pt_ctx_create(B.PT_BF16 if dtype == torch.bfloat16 else B.PT_FP16, S, C, None)
        plan = None
        try:
            B.pt_ctx_set_option(ctx, "grad_fp32", int(fp32))
            plan = B.pt_pack_plan_create(ctx, segs)
            dst = torch.full((C, S), 3.0, dtype=torch.float32 if fp32 else dtype, device="cuda")
            want = dst.clone()
            for c, (s, d) in enumerate(gaps):
                want[c, d:d + n] = src[c, s:s + n]
            rows = [dst[c] for c in range(C)]
            if fp32:
                B.pt_chunk_accum_grads(ctx, plan, rows, True, False)
                assert torch.equal(dst, want)
                B.pt_chunk_accum_grads(ctx, plan, rows, False, True)
                for c, (s, d) in enumerate(gaps):
                    want[c, d:d + n] += src[c, s:s + n].float()
            else:
                B.pt_chunk_pack_grads(ctx, plan, rows)
            assert torch.equal(dst, want)
            B.pt_chunk_grad_sqnorm(ctx, None, 0, C, True)
            sq = sum(float(want[c, d:d + n].double().square().sum()) for c, (s, d) in enumerate(gaps))
            assert abs(B.pt_step_report_read(ctx).sqnorm - sq) <= C * n * 2.0 ** -53 * sq
            if not fp32:
                back = src.clone()
                for c, (s, d) in enumerate(gaps):
                    src[c, s:s + n] = 0
                B.pt_chunk_unpack(ctx, plan, rows)
                assert torch.equal(src, back)
        finally:
            torch.cuda.synchronize()
            if plan is not None:
                B.pt_pack_plan_destroy(plan)
            B.pt_ctx_destroy(ctx)


@pytest.mark.parametrize("n", [(240 << 19) - 5, (240 << 19) + 3, (240 << 19) + 5 * 8192 + 1])
def test_unpack_around_what_the_cache_keeps(n):
    """The first 240 MB of unpacked words are stored in another way than what follows; the tensor lies off the chunks' alignment."""
    S = 1 << 25
    C = -(-n // S)
    chunks = torch.randint(-2 ** 15, 2 ** 15, (C, S), dtype=torch.int16, device="cuda")
    flat = torch.zeros(n + 2, dtype=torch.int16, device="cuda")
    segs, _ = B.pt_layout_dense([n], S)
    for s in segs:
        s.src = flat.data_ptr() + 2
    ctx = B.pt_ctx_create(B.PT_BF16, S, C, None)
    plan = B.pt_pack_plan_create(ctx, segs)
    try:
        for _ in range(2):
            flat.zero_()
            B.pt_chunk_unpack(ctx, plan, [chunks[c] for c in range(C)])
            assert torch.equal(flat[1:n + 1], chunks.view(-1)[:n]) and int(flat[0]) == int(flat[-1]) == 0
    finally:
        torch.cuda.synchronize()
        B.pt_pack_plan_destroy(plan)
        B.pt_ctx_destroy(ctx)


@pytest.mark.parametrize("C", [1, 48, 49, 192, 193])        # 5 pointers a chunk: one launch of 240, two, four, a copy
def test_chunk_pointers_of_any_number_reach_the_device(C):
    """Many small chunks give what one large chunk gives, also after every chunk has moved."""
    many, one = ChunkedState([8 * C], 8), ChunkedState([8 * C], 8 * C)
    try:
        assert many.C == C and one.C == 1
        hp_b, _, _ = hp_pair()
        for step in (1, 2):
            for st in (many, one):
                st.set_grads(step, std=1.0)
                st.pack()
                B.pt_step_override(st.ctx, 0.5, False)
                st.adamw(hp_b)
                st.end()
            for k in ("g16", "w", "m", "v", "p16"):
                bits = torch.int16 if k in ("g16", "p16") else torch.int32
                assert torch.equal(getattr(many, k).view(-1).view(bits), getattr(one, k).view(-1).view(bits)), (step, k)
                # the old places hold something else from now on
                old = getattr(many, k)
                setattr(many, k, old.clone())
                old.fill_(7)
    finally:
        many.close()
        one.close()


@pytest.mark.parametrize("pending", [False, True])       # nothing packed at the capture; an eager pack right before it
def test_graph_of_norm_update_and_step_end_replayed_behind_eager_packs(pending):
    """A plan of more than eight chunks is reduced by its own call: a graph that was captured without the pack sees the sums
    of whatever plan packed in front of the replay, and plans may come and go.  Against the same steps without a graph."""
    sizes, S, C = [9 * 4096 - 5], 4096, 9
    a, b = ChunkedState(sizes, S), ChunkedState(sizes, S)          # replayed, eager
    side = torch.cuda.Stream()
    try:
        assert a.C == C
        hp, _, _ = hp_pair(max_norm=0.05)
        for st in (a, b):                                          # a first step binds every pointer
            st.set_grads(1)
            st.step(hp)
        for st in (a, b):
            st.set_grads(2)
        if pending:
            a.pack()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            B.pt_chunk_grad_sqnorm(a.ctx, None, 0, C, B.PT_FINALIZE_CARRY)
            a.adamw(hp)
            a.end()
        for step in range(2, 7):
            if step > 2 or not pending:
                for st in (a, b):
                    B.pt_pack_plan_destroy(st.plan)
                    st.grad_src = st.grad_src.clone()              # the gradients have moved
                    for g in st.segs:
                        g.src = st.grad_src.data_ptr()
                    st.plan = B.pt_pack_plan_create(st.ctx, st.segs)
                    st.set_grads(step, std=1e-3 * step)
                a.pack()
            graph.replay()
            torch.cuda.synchronize()
            rb = b.step(hp)
            ra = a.report()
            assert (ra.norm, ra.found_inf) == (rb.norm, rb.found_inf), step
            for k in ("g16", "w", "m", "v", "p16"):
                bits = torch.int16 if k in ("g16", "p16") else torch.int32
                assert torch.equal(getattr(a, k).view(bits), getattr(b, k).view(bits)), (step, k)
    finally:
        torch.cuda.synchronize()
        a.close()
        b.close()


def non_coherent_pinned(n, dtype):
    """n elements of pinned host memory that the device caches between synchronisations (hipHostMallocNonCoherent), and
    what gives it back."""
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))
    p = ctypes.c_void_p()
    size = n * torch.empty(0, dtype=dtype).element_size()
    assert hip.hipHostMalloc(ctypes.byref(p), ctypes.c_size_t(size), ctypes.c_uint(0x80000000)) == 0
    t = torch.frombuffer((ctypes.c_char * size).from_address(p.value), dtype=dtype)
    return t, lambda: hip.hipHostFree(p)


@pytest.mark.parametrize("kind", ["coherent", "non-coherent", "graph"])
def test_streamed_update_in_place_step_after_step(kind):
    """Two contexts on streams of their own, four steps without a wait between them, new gradients in host memory each time;
    memory the device caches; the same steps replayed from a graph.  Against a resident copy of the same state, bit for bit."""
    S, n = 5000, 3
    B.lib()
    free, pairs = [], []
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    hp, _, _ = hp_pair()
    try:
        for seed in (0, 1):
            st, ref = ChunkedState([S * n - 3], S, seed=seed), ChunkedState([S * n - 3], S, seed=seed)
            pairs.append((st, ref, {}))
            for k, a in (("g", st.g16), ("p", st.p16), ("w", st.w), ("m", st.m), ("v", st.v)):
                pairs[-1][2][k] = []
                for c in range(n):
                    if kind == "non-coherent":
                        t, give_back = non_coherent_pinned(S, a.dtype)
                        free.append(give_back)
                    else:
                        t = torch.empty(S, dtype=a.dtype, pin_memory=True)
                    pairs[-1][2][k].append(t.copy_(a[c]))
            B.pt_stream_reserve(st.ctx, 2)
            B.pt_ctx_set_option(st.ctx, "stream_in_place", 2)

        def step(st, host, stream):
            B.pt_step_override(st.ctx, 0.5, False, stream)
            B.pt_chunk_stream_step(st.ctx, hp, 0, n, host["g"], host["w"], host["m"], host["v"], host["p"], stream)
            B.pt_step_end(st.ctx, stream)
        graphs = []
        if kind == "graph":
            for (st, _, host), stream in zip(pairs, streams):
                torch.cuda.synchronize()
                graphs.append(torch.cuda.CUDAGraph())
                with torch.cuda.graph(graphs[-1], stream=stream):
                    step(st, host, torch.cuda.current_stream())
        for t in (1, 2, 3, 4):
            for st, ref, host in pairs:
                ref.set_grads(t)
                ref.pack()
                torch.cuda.synchronize()
                for c in range(n):
                    host["g"][c].copy_(ref.g16[c])
            for i, ((st, ref, host), stream) in enumerate(zip(pairs, streams)):      # both enqueued before either is waited for
                if graphs:
                    with torch.cuda.stream(stream):
                        graphs[i].replay()
                else:
                    step(st, host, stream)
            for stream in streams:
                stream.synchronize()
            for st, ref, host in pairs:
                B.pt_step_override(ref.ctx, 0.5, False)
                ref.adamw(hp)
                ref.end()
                for k, a in (("p", ref.p16), ("w", ref.w), ("m", ref.m), ("v", ref.v)):
                    bits = torch.int16 if k == "p" else torch.int32
                    for c in range(n):
                        assert torch.equal(host[k][c].view(bits), a[c].cpu().view(bits)), (kind, t, k, c)
    finally:
        torch.cuda.synchronize()
        for st, ref, _ in pairs:
            st.close()
            ref.close()
        pairs.clear()
        for give_back in free:
            give_back()
