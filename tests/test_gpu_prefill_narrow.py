"""Prefill down projection in 128-row tiles, against the oracle (run_and_check:
routing bit-exact, every output row within the bars).

With m = P/128 + G + 1 token tiles (P positions, G groups) and ks k-chunks
(R/4096, 1 to 4) at most, the narrow tiles run where 2 * m * ceil(C/512) * ks
does not exceed the 256 CUs."""
import pytest

from gpu_layer import Layer, run_and_check
from mira_inputs import MoEConfig

pytestmark = pytest.mark.gpu


def _cfg(cid, T, C, R, E, k, S=0, act="bf16"):
    return MoEConfig(f"narrow_{cid}", cid, T=T, C=C, R=R, E=E, k=k, S=S, act=act, zipf_s=0.5)


CASES = [
    # the last narrow call of this shape and the first wide one; C is not a
    # multiple of either tile
    ("last_narrow", _cfg(761, 2112, 1472, 128, 8, 2)),
    ("first_wide", _cfg(762, 2176, 1472, 128, 8, 2)),
    # half a tile of rows; fewer stages than the ring holds, in one pass and two
    ("one_stage", _cfg(763, 17, 64, 64, 2, 1)),
    ("two_stages", _cfg(764, 33, 192, 128, 3, 2, S=1)),
    ("one_stage_f32", _cfg(765, 65, 64, 64, 2, 1, act="f32")),
    ("f32", _cfg(766, 129, 1024, 832, 5, 2, S=1, act="f32")),
    # several k-chunks, the last one shorter
    ("chunks", _cfg(767, 40, 128, 8192, 2, 1)),
    ("ragged_chunks", _cfg(768, 150, 192, 12352, 2, 2)),
]


# The body and the token rows that a tile loads go by its token count: 32, 64 and
# 128 tokens are the last of each (one expert holds every token; 129 leave a
# second tile of one).
CASES += [(f"tokens_{t}", _cfg(770 + i, t, 192, 320, 1, 1)) for i, t in enumerate((32, 33, 64, 65, 128, 129))]
CASES += [
    ("tokens_48_f32", _cfg(780, 48, 320, 128, 1, 1, act="f32")),
    # more narrow tiles than CUs (18 row tiles of 17 experts), and more workgroups
    # than tiles (most experts without a token)
    ("two_per_cu", _cfg(781, 43, 2304, 128, 17, 5)),
    ("few_of_many", _cfg(782, 17, 128, 64, 120, 1)),
]


@pytest.mark.parametrize("cfg", [pytest.param(c, id=i) for i, c in CASES])
def test_narrow_down(mira, cfg):
    run_and_check(Layer(cfg))
