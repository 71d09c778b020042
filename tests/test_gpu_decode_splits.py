"""Decode calls at the edges of the expert kernels' work splits, against the
oracle (run_and_check: routing bit-exact, every output row within the bars, and
the decode floor).

Down projection: up to 96 k-steps (64 entries of R) per expert the waves split
the concatenated k-steps of all non-empty experts, above that each expert's;
an expert of at most one token group runs the one-group body.

Gate/up: an expert's own token count (1 to 5, to 10, above) chooses the body
in a call of several groups (INT8 up to 15 tokens, INT4 always); INT4 keeps the
digits of one-group experts in LDS up to hidden 4096.

Routing: large routers (more than 16 experts and 96 KB of rows) compute their
logits in a launch of their own; a whole one-token call with at most 64 experts
selects inside the gate/up kernel (up to 16 experts: if its tiles are few).
Descriptors are ordered by token count, up to five tokens by expert."""
import numpy as np
import pytest

import oracle
from gpu_layer import Layer, LazyBlobs, assert_ffn_close, decode_rel_floor, run_and_check
from mira_inputs import MoEConfig

pytestmark = pytest.mark.gpu


def _cfg(cid, T, C, R, E, k, S=0, act="bf16"):
    return MoEConfig(f"split_{cid}", cid, T=T, C=C, R=R, E=E, k=k, S=S, act=act, zipf_s=0.5)


DOWN = [
    # more than 64 non-empty experts (descriptors counted in two passes), some
    # with one token and shared ones with 16
    ("many_experts", _cfg(701, 16, 128, 128, 120, 8, S=2), "int8"),
    ("many_experts_int4", _cfg(702, 16, 128, 256, 120, 8, S=1), "int4"),
    # one k-step in all: 15 (13) waves without work
    ("one_step", _cfg(703, 1, 64, 64, 1, 1), "int8"),
    ("two_steps_int4", _cfg(704, 9, 128, 128, 1, 1), "int4"),
    # the largest ffn with concatenated k-steps and the next one
    ("last_flat", _cfg(705, 9, 64, 6144, 4, 2), "int8"),
    ("first_split", _cfg(706, 9, 64, 6208, 4, 2), "int8"),
    ("last_flat_one", _cfg(707, 1, 64, 6144, 4, 2), "int8"),
    ("first_split_int4", _cfg(708, 6, 128, 6272, 4, 2), "int4"),
    # several workgroups per row tile, one per 150 k-steps (experts reachable *
    # R/64), as the CUs allow: the last whole tile, the first shared by two, by
    # four (more waves than some hold steps), two at the largest hidden size
    ("last_whole", _cfg(710, 2, 64, 1344, 64, 6, S=2), "int8"),
    ("first_shared", _cfg(711, 2, 64, 1408, 64, 6, S=2), "int8"),
    ("shared_by_4_int4", _cfg(712, 16, 128, 640, 64, 6, S=2), "int4"),
    ("shared_by_4", _cfg(715, 11, 192, 768, 64, 6, S=1, act="f32"), "int8"),
    ("shared_2048", _cfg(713, 2, 2048, 6144, 16, 4, act="f32"), "int8"),
    ("whole_2112", _cfg(714, 2, 2112, 6144, 16, 4), "int8"),
    # runs that start and end inside experts
    ("ragged_runs", _cfg(709, 5, 192, 832, 7, 3, S=1, act="f32"), "int8"),
]


@pytest.mark.parametrize("cfg,fmt", [pytest.param(c, f, id=i) for i, c, f in DOWN])
def test_down_split(mira, cfg, fmt):
    _, errs, _, _ = run_and_check(Layer(cfg, fmt=fmt))
    assert errs[0] < decode_rel_floor(cfg.T), errs


GATEUP = [
    # every group size from 1 to T in one call: shared experts with T tokens,
    # popular and rare routed ones
    ("t10", _cfg(721, 10, 192, 128, 24, 3, S=1), "int8"),
    ("t11", _cfg(722, 11, 192, 192, 6, 2, S=1), "int8"),
    ("t15", _cfg(723, 15, 192, 192, 12, 4, S=1), "int8"),
    ("t16", _cfg(724, 16, 192, 192, 12, 4, S=1), "int8"),
    # the largest hidden size with three workgroups per CU and the next one
    ("three_per_cu", _cfg(730, 8, 1024, 192, 12, 4, S=1), "int8"),
    ("three_per_cu_3", _cfg(731, 13, 1024, 128, 12, 4, S=1, act="f32"), "int8"),
    ("two_per_cu", _cfg(732, 8, 1088, 192, 12, 4, S=1), "int8"),
    ("two_per_cu_3", _cfg(733, 13, 1088, 128, 12, 4, S=1), "int8"),
    ("t10_int4", _cfg(725, 10, 256, 128, 24, 3, S=1), "int4"),
    ("t16_int4", _cfg(726, 16, 384, 256, 12, 4, S=1), "int4"),
    ("t6_int4_f32", _cfg(727, 6, 128, 128, 12, 2, act="f32"), "int4"),
    # the largest hidden size with digits in LDS and the next one
    ("lds_last", _cfg(728, 7, 4096, 128, 5, 2), "int4"),
    ("lds_none", _cfg(729, 16, 4224, 128, 5, 2), "int4"),
]


@pytest.mark.parametrize("cfg,fmt", [pytest.param(c, f, id=i) for i, c, f in GATEUP])
def test_gateup_groups(mira, cfg, fmt):
    _, errs, _, _ = run_and_check(Layer(cfg, fmt=fmt))
    assert errs[0] < decode_rel_floor(cfg.T), errs


ROUTE = [
    # the last router in one launch and the first in two (bf16: 96 KB = 24 x 2048)
    ("one_launch", _cfg(741, 3, 2048, 64, 23, 2), 0),
    ("two_launches", _cfg(742, 3, 2048, 64, 24, 2), 0),
    ("two_launches_16", _cfg(743, 16, 1024, 64, 64, 6, S=1), 0),
    # more than 64 pairs and more than 64 experts, a ragged last expert tile
    ("many", _cfg(744, 16, 512, 64, 100, 8), 0),
    ("f32", _cfg(745, 7, 1088, 64, 30, 3, act="f32"), 0),
    ("f32_one_launch", _cfg(746, 5, 320, 64, 7, 3, act="f32"), 0),
    # fp32 with a wave per token and expert (at most 16) and the next call in 4 x 4
    # tiles; columns past the last whole pass of either
    ("f32_single", _cfg(757, 4, 576, 64, 4, 2, act="f32"), 0),
    ("f32_single_one", _cfg(758, 1, 1088, 64, 16, 3, act="f32"), 0),
    ("f32_tiles", _cfg(759, 3, 1088, 64, 6, 2, act="f32"), 0),
    ("f32_split_one", _cfg(760, 1, 2112, 64, 29, 3, act="f32"), 0),
    # fp32 columns past the last whole pass, ragged token and expert quads
    ("f32_prefill", _cfg(747, 37, 576, 64, 21, 4, act="f32"), 0),
    # one token: rank counting (E < 2k) and repeated maxima, at their border
    ("one_k_of_2k", _cfg(748, 1, 128, 64, 12, 6, S=2), 0),
    ("one_k_above", _cfg(749, 1, 128, 64, 11, 6), 0),
    ("one_64", _cfg(750, 1, 256, 64, 64, 16, S=3), 0),
    # every group size up to T, in both descriptor forms; equal sizes
    ("sizes", _cfg(753, 16, 128, 64, 20, 3, S=2), 0),
    ("sizes_many", _cfg(754, 16, 128, 64, 40, 8, S=2), 0),
    # expert order up to five tokens, sizes above; shared experts at either end
    ("order_5", _cfg(734, 5, 128, 64, 12, 4, S=3), 0),
    ("order_6", _cfg(735, 6, 128, 64, 12, 4, S=3), 0),
    ("sizes_equal", _cfg(755, 16, 128, 64, 8, 8, S=3), 0),
    ("sizes_254", _cfg(756, 16, 64, 64, 250, 16, S=4), 0),
    # the most tiles (12 per CU) of a call of 16 experts that selects inside
    # gate/up, and the next one
    ("one_tiles_last", _cfg(736, 1, 64, 6144, 16, 8), 0),
    ("one_tiles_next", _cfg(737, 1, 64, 6208, 16, 8), 0),
    ("one_all", _cfg(751, 1, 128, 64, 9, 2, S=1, act="f32"), 1),
    ("three_all", _cfg(752, 3, 128, 64, 40, 5), 1),
]


@pytest.mark.parametrize("cfg,softmax_all", [pytest.param(c, f, id=i) for i, c, f in ROUTE])
def test_route_split(mira, cfg, softmax_all):
    """Routing and output against the oracle, and the one-shot call against the
    two-phase call (which runs the general kernels) bit for bit."""
    lay = Layer(cfg)
    flags = mira.MIRA_FLAG_SOFTMAX_ALL if softmax_all else 0
    res = lay.run(flags)
    two = lay.run(flags, two_phase=True, ws_fill=0xFF)
    for name, v in res.items():
        assert np.array_equal(v, two[name]), name
    if not softmax_all:
        run_and_check(lay, res=res)
        return
    # the oracle's helper checks renormalised weights; these sum to less.  The
    # selection is the sort of the logits, and weights and output are the oracle's
    # under it
    x, wr, b = lay.oracle_inputs()
    lg = res["logits"].astype(np.float64)
    assert np.max(np.abs(lg - oracle.router_logits(x, wr, b)) / np.maximum(1.0, np.abs(lg))) < 2e-5
    for t in range(cfg.T):
        assert res["idx"][t].tolist() == sorted(range(cfg.E), key=lambda e: (-lg[t, e], e))[:cfg.k], t
    ref = oracle.moe_forward(x, wr, b, LazyBlobs(lay), cfg.k, cfg.C, cfg.R, shared_blobs=lay.shared_blobs(),
                             norm_topk=False, idx=res["idx"])
    assert np.max(np.abs(res["w"] - ref["w"])) < 2e-5
    assert_ffn_close(res["out"], ref["out"], cfg.name)


@pytest.mark.parametrize("softmax_all", [0, 1])
@pytest.mark.parametrize("cfg", [
    # rank counting (E < 2k) and repeated maxima, shared experts, the most experts
    pytest.param(_cfg(783, 1, 256, 256, 12, 7, S=2), id="counting"),
    pytest.param(_cfg(784, 1, 384, 384, 64, 6, S=3), id="maxima"),
    pytest.param(_cfg(785, 1, 4096, 128, 8, 2), id="lds_last"),
    pytest.param(_cfg(786, 1, 128, 256, 9, 2, S=1, act="f32"), id="f32"),
])
def test_one_token_int4_selection(mira, cfg, softmax_all):
    """A one-token INT4 call, which selects inside gate/up, against the two-phase
    call (a selection kernel) bit for bit, and against the oracle."""
    lay = Layer(cfg, fmt="int4")
    flags = mira.MIRA_FLAG_SOFTMAX_ALL if softmax_all else 0
    res = lay.run(flags, ws_fill=0xFF)
    two = lay.run(flags, two_phase=True, ws_fill=0xFF)
    for name, v in res.items():
        assert np.array_equal(v, two[name]), name
    if not softmax_all:
        run_and_check(lay, res=res)
