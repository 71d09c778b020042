"""Selected experts without a valid slot, where the expert kernels split their
work: their terms are left out of the output and nothing else changes, the
status says why (bit 0: slot -1, bit 1: a slot past the pool), and what they
would have written is not read (the workspace starts as NaN bytes).

Decode down: runs of concatenated k-steps that start in, end in and cross such
an expert, also where several workgroups share a row tile.  One-token calls:
the selection inside gate/up reports routed and shared experts.  Prefill: narrow
down tiles over several k-chunks."""
import numpy as np
import pytest

import oracle
from gpu_layer import Layer, LazyBlobs, assert_ffn_close, check_routing, ffn_error, decode_rel_floor
from mira_inputs import MoEConfig

pytestmark = pytest.mark.gpu


def _cfg(cid, T, C, R, E, k, S=0, act="bf16"):
    return MoEConfig(f"missing_{cid}", cid, T=T, C=C, R=R, E=E, k=k, S=S, act=act, zipf_s=0.5)


class _Without:
    """The layer's blobs, with experts of zero weights and scales for the missing ones."""

    def __init__(self, lay, missing):
        self.blobs, self.missing, self.size = LazyBlobs(lay), missing, lay.stride

    def __len__(self):
        return len(self.blobs)

    def __getitem__(self, e):
        return np.zeros(self.size, dtype=np.uint8) if e in self.missing else self.blobs[e]


def run_without(lay, slots, flags=0):
    """One call with the table entries `slots` {expert: slot}, checked against the oracle."""
    c = lay.cfg
    for e, s in slots.items():
        lay.table[e] = s
    res = lay.run(flags, ws_fill=0xFF)
    assert res["status"][0] == sum({1 if s < 0 else 2 for s in slots.values()})
    x, wr, b = lay.oracle_inputs()
    check_routing(res, lay, oracle.router_logits(x, wr, b))
    shared = [blob for s, blob in enumerate(lay.shared_blobs()) if c.E + s not in slots]
    ref = oracle.moe_forward(x, wr, b, _Without(lay, slots), c.k, c.C, c.R, shared_blobs=shared, idx=res["idx"],
                             fmt=lay.fmt)["out"]
    assert_ffn_close(res["out"], ref, f"{c.name} {lay.fmt} without {slots}")
    return res, ffn_error(res["out"], ref)[0]


DOWN = [
    # two and four workgroups per row tile; one per tile
    ("shared_by_2", _cfg(791, 2, 64, 1408, 64, 6, S=2), "int8"),
    ("shared_by_4", _cfg(792, 11, 192, 768, 64, 6, S=1, act="f32"), "int8"),
    ("shared_by_4_int4", _cfg(793, 16, 128, 640, 64, 6, S=2), "int4"),
    ("whole", _cfg(794, 5, 192, 832, 7, 3, S=1), "int8"),
    ("split", _cfg(795, 9, 64, 6208, 4, 2, S=1), "int8"),
]


@pytest.mark.parametrize("which", ["first", "last", "routed_and_shared"])
@pytest.mark.parametrize("cfg,fmt", [pytest.param(c, f, id=i) for i, c, f in DOWN])
def test_down_runs(mira, cfg, fmt, which):
    lay = Layer(cfg, fmt=fmt)
    hit = np.flatnonzero(lay.run()["counts"][:cfg.E])
    past = lay.n_slots + 3
    slots = {"first": {int(hit[0]): -1}, "last": {int(hit[-1]): past},
             "routed_and_shared": {int(hit[len(hit) // 2]): past, int(hit[0]): -1, cfg.E: -1}}[which]
    _, err = run_without(lay, slots)
    assert err < decode_rel_floor(cfg.T), err


@pytest.mark.parametrize("fmt", ["int8", "int4"])
@pytest.mark.parametrize("slots", [{8: -1}, {9: 10}, {8: -1, 9: 99}, {8: 99, 9: -1, "top": -1}], ids=str)
def test_one_token_shared(mira, fmt, slots):
    """Experts 8 and 9 are the shared ones; "top" is the token's first choice."""
    lay = Layer(_cfg(796, 1, 256, 384, 8, 2, S=2), fmt=fmt)
    top = int(lay.run()["idx"][0][0])
    _, err = run_without(lay, {top if e == "top" else e: s for e, s in slots.items()})
    assert err < decode_rel_floor(1), err


@pytest.mark.parametrize("missing", [0, 1])
def test_narrow_prefill_chunks(mira, missing):
    run_without(Layer(_cfg(797, 70, 192, 8192, 2, 1, S=1)), {missing: -1, 2: 7})
