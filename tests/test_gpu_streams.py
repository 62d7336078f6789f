"""Calls are enqueued on the stream that torch has as the current one, in the calling thread, or on the one that is passed."""
import threading

import pytest
import torch

import gen
import paper_2308_14352_amd as moeq
from helpers import build_layer_pair

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("how", ("current", "passed", "thread"))
@pytest.mark.parametrize("columns", (False, True), ids=("canonical", "columns"))
def test_calls_wait_for_the_work_ahead_of_them_on_their_stream(how, columns):
    cfg = gen.tiny_config("c1", 256, 512, n_experts=4, n_layers=1, group=32)
    layer, _, _, _ = build_layer_pair(cfg, 0, DEV, [2, 4, 8, 4], want_oracle=False, columns=columns)
    x = gen.hidden(cfg, 0, 0, 3, DEV)
    gate = torch.full((3,), 0.5, device=DEV)
    calls = lambda v, **kw: [moeq.moe_layer_forward(layer, v, ws=ws, **kw), moeq.moe_expert_ffn_q(layer, 1, v, gate=gate, ws=ws, **kw),
                             *moeq.moe_router_topk(layer, v, ws=ws, **kw)]
    ws = torch.empty(layer.workspace_bytes(3), dtype=torch.uint8, device=DEV)
    want = calls(x)
    late = torch.zeros_like(x)
    torch.cuda.synchronize()
    side, got = torch.cuda.Stream(), []

    def run():
        with torch.cuda.stream(side):
            torch.cuda._sleep(20_000_000)            # some 10 ms: on another stream the calls would read zeros
            late.copy_(x)
            if how != "passed":
                got.extend(calls(late))
        if how == "passed":
            got.extend(calls(late, stream=side))

    if how == "thread":
        t = threading.Thread(target=run)
        t.start()
        t.join()
    else:
        run()
    side.synchronize()
    assert len(got) == 4 and all(torch.equal(a, b) for a, b in zip(got, want))
