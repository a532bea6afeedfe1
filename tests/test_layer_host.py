"""Which methods and which library calls a whole-layer pass goes through, on the host: the library is replaced by a recorder."""
import pytest

import paper_2512_07710_amd as moe
from paper_2512_07710_amd import binding

CALLS = ("moe_route", "moe_route_replay", "moe_quantize_fp8", "moe_route_quantize", "moe_route_replay_quantize",
         "moe_expert_ffn_fp8", "moe_expert_ffn_fp8_gather", "moe_combine")
BUFFERS = ("topk_idx", "topk_w", "offsets", "perm", "inv_perm", "xq", "xs", "xq_tok", "xs_tok", "y_perm", "y")
WEIGHTS = dict.fromkeys(("W1q", "W3q", "W2q", "s1", "s3", "s2"))


class _Stream:
    def wait_stream(self, other):
        pass


def _bare(cls, overlap=False):
    layer = object.__new__(cls)                                # no GPU here: only what the passes read
    layer.T, layer.d, layer.E, layer.k, layer.F, layer.N = 3, 128, 4, 2, 128, 6
    layer.ctx, layer.side_ctx = "ctx", "side"
    layer.stream, layer.side_stream, layer.overlap_quantize = _Stream(), _Stream(), overlap
    for name in BUFFERS:
        setattr(layer, name, name)
    layer.close = lambda: None
    return layer


@pytest.fixture
def log(monkeypatch):
    calls = []
    for name in CALLS:
        monkeypatch.setattr(binding, name, lambda *a, _n=name: calls.append(_n))
    return calls


def _forward(layer, mode, **kw):
    if mode == "routed":
        return layer.forward_routed("x", "W_r", "bias", WEIGHTS, **kw)
    return layer.forward_replay("x", "ids", "gates", WEIGHTS, **kw)


@pytest.mark.parametrize("mode,route", [("routed", "moe_route"), ("replay", "moe_route_replay")])
def test_plain_layer_takes_the_joint_call(log, mode, route):
    assert _forward(_bare(moe.MoELayer), mode) == "y"
    assert log == [route + "_quantize", "moe_expert_ffn_fp8_gather", "moe_combine"]
    log.clear()
    _forward(_bare(moe.MoELayer), mode, fused=False)
    assert log == [route, "moe_quantize_fp8", "moe_expert_ffn_fp8", "moe_combine"]
    log.clear()
    _forward(_bare(moe.MoELayer, overlap=True), mode)
    assert log == ["moe_quantize_fp8", route, "moe_expert_ffn_fp8_gather", "moe_combine"]


@pytest.mark.parametrize("overlap", [False, True])
@pytest.mark.parametrize("how", ["subclass", "instance", "class"])
@pytest.mark.parametrize("mode,stage", [("routed", "route"), ("routed", "quantize_tokens"), ("replay", "route_replay"),
                                        ("replay", "quantize_tokens")])
def test_a_replaced_stage_is_called(log, monkeypatch, mode, stage, how, overlap):
    """A routing or quantising method that a subclass, an instance or a wrapper on the class replaces is called with what the pass was
    given, whatever the size of the batch, and the stages beside it run as calls of their own."""
    seen = []
    original = getattr(moe.MoELayer, stage)

    def wrapper(self, *args):
        seen.append(args)
        return original(self, *args)

    cls = moe.MoELayer
    if how == "subclass":
        cls = type("Wrapped", (moe.MoELayer,), {stage: wrapper})
    elif how == "class":
        monkeypatch.setattr(moe.MoELayer, stage, wrapper)
    layer = _bare(cls, overlap)
    if how == "instance":
        setattr(layer, stage, lambda *args: wrapper(layer, *args))
    assert _forward(layer, mode) == "y"
    assert seen == [{"route": ("x", "W_r", "bias"), "route_replay": ("x", "ids", "gates"), "quantize_tokens": ("x",)}[stage]]
    route = "moe_route" if mode == "routed" else "moe_route_replay"
    assert sorted(log[:2]) == sorted([route, "moe_quantize_fp8"]) and log[2:] == ["moe_expert_ffn_fp8_gather", "moe_combine"]
