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


# ------------------------------------------------------------------ how a captured chain is replayed
DIRECT, EXECUTABLE = 1, 2  # use_graphs


def replays(qe, hip, use_graphs, on_caller, graph_inputs, k, tokens):
    """Four F of one slot: the first one, with the weights, from a graph of its own, then three with other inputs
    each, nothing waited for between."""
    ctx = qe.Context(1, use_graphs=use_graphs, replay_on_caller=on_caller, graph_inputs=graph_inputs)
    st, layer = ctx.qe_layer_register(0, 0, 256, k, tokens, ADDR, qe.F32, 4, 0)
    assert st == "OK"
    for i in range(4):
        st, _ = ctx.qe_fp8_linear_fwd(layer, qe.key(0, 0, 0, 0), ADDR << i, qe.F32, tokens, ADDR, qe.F32, caller=CALLER)
        assert st == "OK"
        assert ctx.qe_abort_epoch() == "OK" and ctx.qe_arena_rebuild() == "OK"  # frees the slot
    state = ctx.qe_get_state()
    ctx.close()
    return [{kind: hip.log(kind) for kind in ("capture", "launch", "instantiate", "graph_launch", "set_params", "exec_destroy")},
            state["captures"], state["rebinds"], state["replays"]]


@pytest.mark.parametrize("on_caller", [False, True], ids=["graph_stream", "caller_stream"])
def test_short_chains_are_replayed_launch_by_launch(on_caller):
    log, captures, rebinds, n = calls(replays, DIRECT, on_caller, 0, 256, 64)
    assert (captures, rebinds, n) == (2, 2, 4)
    assert len(log["capture"]) == 2 * 2 and len(log["launch"]) == 4 * 2
    assert not log["instantiate"] and not log["graph_launch"] and not log["set_params"]


# 2^17 rows of 2^16 codes are four 2 GiB blocks and a bit (a chain of six kernels); 2^18 are nine (ten)
@pytest.mark.parametrize("use_graphs,k,tokens,kernels", [(EXECUTABLE, 256, 64, 2), (DIRECT, 1 << 16, 1 << 18, 10),
                                                         (DIRECT, 1 << 16, 1 << 17, 0)])
@pytest.mark.parametrize("on_caller", [False, True], ids=["graph_stream", "caller_stream"])
def test_executables_are_rebound_after_their_replay(on_caller, use_graphs, k, tokens, kernels):
    """Chains of nine kernels and more, and all with use_graphs = 2, are instantiated; their nodes are rewritten
    with no replay of theirs in flight.  (0 kernels: the chain stays below nine.)"""
    log, captures, rebinds, n = calls(replays, use_graphs, on_caller, 0, k, tokens)
    assert (captures, rebinds, n) == (2, 2, 4)
    if kernels == 0:
        assert len(log["capture"]) == 2 * 6 and not log["instantiate"] and len(log["launch"]) == 4 * 6
        return
    assert len(log["capture"]) == 2 * kernels and not log["launch"]
    assert log["instantiate"] == [["instantiate", "kernels=%d" % kernels]] * 2
    assert [w[2] for w in log["graph_launch"]] == ["kernels=%d" % kernels] * 4
    assert log["set_params"] == [["set_params", "pending=0"]] * 2  # the cast's input
    assert log["exec_destroy"] == [["exec_destroy", "pending=0"]] * 2


@pytest.mark.parametrize("on_caller", [False, True], ids=["graph_stream", "caller_stream"])
def test_recaptured_executables_go_after_their_replay(on_caller):
    log, captures, rebinds, n = calls(replays, EXECUTABLE, on_caller, 1, 256, 64)
    assert (captures, rebinds, n) == (4, 0, 4)
    assert len(log["instantiate"]) == 4 and len(log["graph_launch"]) == 4 and not log["set_params"]
    assert log["exec_destroy"] == [["exec_destroy", "pending=0"]] * 4
