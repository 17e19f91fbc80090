"""A step ends in the launch that derives its constants - here the update itself - without a launch of its own behind it, unless
something of the same step still depends on the step counter or the loss scale, or the context has been captured into a graph.
Either way leads to the values of the machine written out here; every sequence runs in a context of each kind."""
import pytest
import torch

from paper_2406_08334_amd import binding as B

from gpu_harness import ChunkedState, assert_same_bits, hp_pair

pytestmark = pytest.mark.gpu

C = 3
SIZES = [4096, (1 << 19) + 8]       # elements of a chunk: below 6144 tiles of the update altogether, and above
GROWTH_INTERVAL = 2
INF_STEPS = (3, 6)


class Machine:
    """Step counter and loss scale as pt_step_end documents them, and the number of the update in flight."""

    def __init__(self):
        self.step, self.scale, self.good, self.found, self.t = 0, 1024.0, 0, 0, 0

    def update(self):
        self.t = self.step + 1

    def end(self):
        if self.found:
            self.scale, self.good = max(self.scale * 0.5, 1.0), 0
        else:
            self.step, self.good = self.step + 1, self.good + 1
            if self.good == GROWTH_INTERVAL:
                self.scale, self.good = self.scale * 2.0, 0

    def check(self, st, hp, where):
        r = B.pt_step_report_read(st.ctx)
        assert (r.step, r.loss_scale, r.good_steps, r.found_inf) == (self.step, self.scale, self.good, self.found), where
        if self.t:
            c5 = B.pt_update_consts_read(st.ctx).c[5]
            assert abs(c5 * (1.0 - hp.beta1 ** self.t) / hp.lr - 1.0) < 1e-6, (where, "t")     # one rounding to fp32: 6e-8
        return r.sqnorm, r.norm, r.clip_coef, r.grad_mult


def make(captured, S):
    st = ChunkedState([S * C - 5], S, dtype=torch.float16, scaler=B.pt_scaler_cfg(1024.0, 2.0, 0.5, GROWTH_INTERVAL, 0))
    if captured:                            # from here on its steps end in a kernel of their own (tests/pins/host_calls.cpp counts them)
        with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=torch.cuda.Stream()):
            B.pt_step_end(st.ctx)
    return st


def set_grads(st, t):
    st.set_grads(t, scale=256.0)
    if t in INF_STEPS:
        st.grad_src.view(torch.int16)[t * 100] = 0x7C00


def between(st, kind, hp, hp2, model):
    """What happens between the update and the step's end, on the device and in the machine; returns whether the step is over by then, and
    the hyper-parameters last used."""
    if kind == "pack":
        st.pack()
    elif kind == "recompute":               # a norm of the same step that finds an inf: the step counts as skipped
        st.g16.view(torch.int16)[1, 7] = 0x7C00
        st.norm(recompute=True)
        model.found = 1
    elif kind == "finalize":
        st.norm(finalize=B.PT_FINALIZE_CARRY)
        st.adamw(hp2)
        return False, hp2
    elif kind == "override":
        B.pt_step_override(st.ctx, 0.25, False)
        st.adamw(hp)
        model.found = 0
    elif kind == "skip":
        B.pt_step_override(st.ctx, 0.25, True)
        model.found = 1
    elif kind == "state":
        B.pt_ctx_set_state(st.ctx, 40, 64.0, 1)
        model.step, model.scale, model.good = 40, 64.0, 1
    elif kind == "hyper-parameters":
        st.adamw(hp2)
        return False, hp2
    elif kind == "in parts":
        st.adamw(hp, 1, 2)
    elif kind == "graph":                   # the end alone in a graph, replayed: the kernel sees that the step has ended
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            B.pt_step_end(st.ctx)
        model.check(st, hp, "captured, not run")
        for _ in range(3):                  # the second and third end steps of their own, on the same found_inf
            g.replay()
            model.end()
        torch.cuda.synchronize()
        return True, hp
    return False, hp


@pytest.mark.parametrize("S", SIZES)
@pytest.mark.parametrize("kind", ["nothing", "pack", "recompute", "finalize", "override", "skip", "state", "hyper-parameters",
                                  "in parts", "graph"])
def test_the_step_ends_with_its_constants_or_behind_the_update(kind, S):
    states = [make(captured, S) for captured in (False, True)]
    hp, _, _ = hp_pair()
    hp2, _, _ = hp_pair(lr=3e-3, beta1=0.5, beta2=0.7, max_norm=0.1)
    models = [Machine() for _ in states]
    try:
        for t in range(1, 8):
            seen = []
            for st, model in zip(states, models):
                set_grads(st, t)
                model.found = int(t in INF_STEPS)
                st.pack()
                st.norm()
                st.adamw(hp)
                model.update()
                seen.append([model.check(st, hp, (kind, t, "open"))])          # before the step's end
                over, last = between(st, kind if t > 1 else "nothing", hp, hp2, model)
                if not over:
                    seen[-1].append(model.check(st, last, (kind, t, "still open")))
                    st.end()
                    model.end()
                seen[-1].append(model.check(st, last, (kind, t, "over")))
            assert seen[0] == seen[1], t
            a, b = (st.host_state() for st in states)
            for name in ("g16", "w", "m", "v", "p16"):
                assert_same_bits(a[name], b[name], (kind, t, name))
    finally:
        torch.cuda.synchronize()
        for st in states:
            st.close()


@pytest.mark.parametrize("S", SIZES)
def test_step_end_in_a_graph_behind_eager_updates(S):
    """The step end alone, captured on a fresh context and replayed in every step: Adam's t and the loss scale move."""
    st, model = make(False, S), Machine()
    hp, _, _ = hp_pair()
    try:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            B.pt_step_end(st.ctx)
        for t in range(1, 9):
            set_grads(st, t)
            model.found = int(t in INF_STEPS)
            st.pack()
            st.norm(finalize=B.PT_FINALIZE_CARRY)
            st.adamw(hp)
            model.update()
            model.check(st, hp, (t, "open"))
            g.replay()
            model.end()
            torch.cuda.synchronize()
            model.check(st, hp, (t, "over"))
    finally:
        st.close()


@pytest.mark.parametrize("S", SIZES)
@pytest.mark.parametrize("first", ["eager step", "replay"])
def test_graph_captured_in_a_step_that_has_ended_early(first, S):
    """Norm, update and step end are captured between an update and its step end, then replayed with eager steps in between."""
    st, model = make(False, S), Machine()
    hp, _, _ = hp_pair()

    def gradients(t):
        set_grads(st, t)
        model.found = int(t in INF_STEPS)
        st.pack()

    def eager(t):
        gradients(t)
        st.norm()
        st.adamw(hp)
        model.update()
        model.check(st, hp, (t, "open"))
        st.end()
        model.end()
        model.check(st, hp, (t, "eager"))

    try:
        eager(1)
        gradients(2)
        st.norm()
        st.adamw(hp)
        model.update()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            st.norm(finalize=B.PT_FINALIZE_CARRY)
            st.adamw(hp)
            B.pt_step_end(st.ctx)
        model.check(st, hp, "captured, not run")
        if first == "eager step":
            st.end()
            model.end()
            model.check(st, hp, "ended")
        for t in range(3, 12):
            if t % 3 == 0 and (first == "eager step" or t > 3):
                eager(t)
                continue
            gradients(t)
            st.report()                     # a small plan's sums wait for an eager call
            g.replay()
            model.update()
            model.end()
            torch.cuda.synchronize()
            model.check(st, hp, (t, "replayed"))
    finally:
        st.close()
