"""A step ends in the launch that derives its constants, without a launch of its own behind the update - unless something of
the same step still depends on the step counter or the loss scale, or the context has been captured into a graph.  Either way
gives the same bits: every sequence runs in a context of each kind."""
import pytest
import torch

from paper_2406_08334_amd import binding as B

from gpu_harness import ChunkedState, assert_same_bits, hp_pair

pytestmark = pytest.mark.gpu

S, C = 4096, 3
GROWTH_INTERVAL = 2


def make(captured):
    st = ChunkedState([S * C - 5], S, dtype=torch.float16, scaler=B.pt_scaler_cfg(1024.0, 2.0, 0.5, GROWTH_INTERVAL, 0))
    if captured:                            # from here on its steps end in a kernel of their own
        with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=torch.cuda.Stream()):
            B.pt_step_end(st.ctx)
    return st


def report(st):
    r = B.pt_step_report_read(st.ctx)
    return (r.sqnorm, r.norm, r.clip_coef, r.loss_scale, r.grad_mult, r.found_inf, r.step, r.good_steps)


def between(st, kind, hp, hp2):
    """What happens between the update and the step's end; True if the step is over by then."""
    if kind == "pack":
        st.pack()
    elif kind == "recompute":               # a norm of the same step that finds an inf: the step counts as skipped
        st.g16.view(torch.int16)[1, 7] = 0x7C00
        st.norm(recompute=True)
    elif kind == "finalize":
        st.norm(finalize=B.PT_FINALIZE_CARRY)
        st.adamw(hp2)
    elif kind == "override":
        B.pt_step_override(st.ctx, 0.25, False)
        st.adamw(hp)
    elif kind == "skip":
        B.pt_step_override(st.ctx, 0.25, True)
    elif kind == "state":
        B.pt_ctx_set_state(st.ctx, 40, 64.0, 1)
    elif kind == "hyper-parameters":
        st.adamw(hp2)
    elif kind == "in parts":
        st.adamw(hp, 1, 2)
    elif kind == "graph":                   # the end alone in a graph, replayed: the kernel sees that the step has ended
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            B.pt_step_end(st.ctx)
        for _ in range(3):                  # the second and third end steps of their own, on the same found_inf
            g.replay()
        torch.cuda.synchronize()
        return True
    return False


@pytest.mark.parametrize("kind", ["nothing", "pack", "recompute", "finalize", "override", "skip", "state", "hyper-parameters",
                                  "in parts", "graph"])
def test_the_step_ends_with_its_constants_or_behind_the_update(kind):
    states = [make(captured) for captured in (False, True)]
    hp, _, _ = hp_pair()
    hp2, _, _ = hp_pair(lr=3e-3, beta1=0.5, beta2=0.7, max_norm=0.1)
    try:
        scale, good, step = 1024.0, 0, 0
        for t in range(1, 8):
            seen = []
            for st in states:
                st.set_grads(t, scale=256.0)
                if t in (3, 6):
                    st.grad_src.view(torch.int16)[t * 100] = 0x7C00
                st.pack()
                st.norm()
                st.adamw(hp)
                seen.append([report(st)])              # the step is still open: before its end
                over = between(st, kind if t > 1 else "nothing", hp, hp2)
                if not over:
                    seen[-1].append(report(st))
                    st.end()
                seen[-1].append(report(st))
            assert seen[0] == seen[1], t
            if kind in ("nothing", "pack", "in parts"):         # the machine itself
                assert seen[0][0][3] == seen[0][1][3] == scale and seen[0][0][6:] == (step, good), t
                if t in (3, 6):
                    scale, good = max(scale * 0.5, 1.0), 0
                else:
                    step, good = step + 1, good + 1
                    if good == GROWTH_INTERVAL:
                        scale, good = scale * 2.0, 0
                assert seen[0][-1][3] == scale and seen[0][-1][6:] == (step, good), t
            a, b = (st.host_state() for st in states)
            for name in ("g16", "w", "m", "v", "p16"):
                assert_same_bits(a[name], b[name], (kind, t, name))
    finally:
        torch.cuda.synchronize()
        for st in states:
            st.close()
