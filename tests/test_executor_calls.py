"""The HIP calls the executor makes, checked without a device (tests/fake_hip.py)."""
import pytest

from tests.fake_hip import ADDR, calls

CALLER, OTHER = 7 << 8, 8 << 8  # the program's streams


def _stage(qe, use_graphs, on_caller, microbatches=4):
    ctx = qe.Context(microbatches, use_graphs=use_graphs, replay_on_caller=on_caller)
    st, layer = ctx.qe_layer_register(0, 0, 256, 256, 64, ADDR, qe.F32, 4, 0)
    assert st == "OK"
    return ctx, layer


def _fwd(ctx, qe, layer, m, caller=CALLER):
    return ctx.qe_fp8_linear_fwd(layer, qe.key(0, 0, m, 0), ADDR, qe.F32, 64, ADDR, qe.F32, caller=caller)[0]


# ------------------------------------------------------------------ an action that fails part-way
def part_way(qe, hip, use_graphs, on_caller, fault):
    """The second F fails after its first kernel (or at its completion event); then each way on."""
    got = {}
    for way in ("sync", "destroy", "caller", "next"):
        ctx, layer = _stage(qe, use_graphs, on_caller)
        if use_graphs:
            assert ctx.qe_prebuild_graphs(64, qe.F32, qe.F32, qe.F32, qe.F32) == "OK"
        assert _fwd(ctx, qe, layer, 0) == "OK"
        hip.drain(CALLER)
        assert hip.pending() == 0
        if fault == "launch":
            hip.fail_launch(2)
        else:  # the first record of a two-way action is the caller's edge
            hip.fail_record(1 if on_caller else 2)
        assert _fwd(ctx, qe, layer, 1) == "HIP"
        before = hip.pending()
        if way == "sync":
            assert ctx.qe_sync() == "OK"
        elif way == "caller":  # what the program enqueues next may overwrite the action's buffers
            hip.drain(CALLER)
        elif way == "next":    # the next action, from another stream
            assert ctx.qe_abort_epoch() == "OK" and ctx.qe_arena_rebuild() == "OK"
            assert _fwd(ctx, qe, layer, 0, OTHER) == "OK"
            hip.drain(OTHER)
        hip.clear()
        after = hip.pending()
        ctx.close()
        frees = [int(w[1].split("=")[1]) for w in hip.log("free")]
        got[way] = [before, after, max(frees)]
    return got


@pytest.mark.parametrize("fault", ["launch", "record"])
@pytest.mark.parametrize("on_caller", [False, True], ids=["graph_stream", "caller_stream"])
@pytest.mark.parametrize("use_graphs", [0, 1], ids=["eager", "graphs"])
def test_action_that_fails_part_way_is_waited_for(use_graphs, on_caller, fault):
    """An action whose second launch (or completion event) fails has its first kernels in flight: qe_sync, the
    caller's stream, the next action and the destruction of the context still come after them."""
    got = calls(part_way, use_graphs, on_caller, fault)
    for way, (before, after, at_free) in got.items():
        if fault == "launch":
            assert before == 1, way
        if way != "destroy":
            assert after == 0, way
        assert at_free == 0, way
