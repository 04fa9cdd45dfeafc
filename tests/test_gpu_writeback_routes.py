"""The decode step's write-backs by grid size (one lane per clip factor, four
lanes per group of factors, a block per head) are one function: the step on the
workspace, whose route depends on B H, against kda_step_noalloc, which always
rebuilds the state from the record in a block per head (d_k <= 128), and one
launch of many heads against the same heads in launches of few (d_k = 256).
Head counts lie at the edges of the routes' ranges."""
import pytest
import torch

import paper_2609_30950_amd as K
from tests._gpu import say

pytestmark = pytest.mark.gpu


def _inputs(B, H, d, heavy, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    unit = lambda: torch.nn.functional.normalize(torch.randn(B, H, d, generator=g, device="cuda"), dim=-1)  # noqa: E731
    v = torch.randn(B, H, d, generator=g, device="cuda")
    if heavy:
        v = v * torch.exp(3 * torch.randn(B, H, d, generator=g, device="cuda"))
        v[0, 0] = 0.0        # a head whose state stays zero
    s = torch.exp(-7 * torch.rand(B, H, d, generator=g, device="cuda"))
    return unit(), unit(), v, s, torch.sigmoid(torch.randn(B, H, generator=g, device="cuda"))


def _cfg(B, H, d, **kw):
    return K.Config(B=B, H=H, d_k=d, d_v=d, **{"group_rows": d, **kw})


@pytest.mark.parametrize("B,H,d,kw", [
    (1, 1, 64, {}), (1, 3, 64, dict(b_min=1, mean_bits=1.75)), (8, 32, 64, {}), (8, 33, 64, dict(mean_bits=3.0)),
    (32, 32, 64, {}), (1, 1, 128, dict(b_min=1, mean_bits=2.5)), (2, 32, 128, dict(group_rows=64)), (5, 13, 128, {}),
    (8, 32, 128, dict(mean_bits=3.0)), (2, 2, 128, dict(b_max=16, mean_bits=9.0)), (2, 2, 64, dict(b_max=16, mean_bits=8.5)),
    (2, 6, 128, dict(group_rows=3 * 128, b_min=1)), (3, 5, 128, dict(scope=1, b_min=1, mean_bits=2.0)),
])
def test_routes_write_the_same_records(B, H, d, kw):
    cfg = _cfg(B, H, d, **kw)
    ws = K.new_workspace(cfg)
    ra, rb = K.new_records(cfg), K.new_records(cfg)
    oa, ob = (torch.empty(B, H, d, device="cuda") for _ in range(2))
    for t in range(5):
        x = _inputs(B, H, d, t % 2 == 1, 100 * t + d)
        K.kda_step(cfg, ra, *x, oa, ws)
        K.kda_step_noalloc(cfg, rb, *x, ob)
        say(f"routes B={B} H={H} d={d} t={t}")
        assert torch.equal(ra, rb) and torch.equal(oa, ob)


@pytest.mark.parametrize("B", [2, 3, 6, 7])
def test_routes_at_256(B):
    # heads per launch: 32 (one round, widths selected inside), 48 and 96, 112 (a block per head)
    H, d = 16, 256
    cfg, one = _cfg(B, H, d, b_min=1, mean_bits=2.5), _cfg(1, H, d, b_min=1, mean_bits=2.5)
    ws, ws1 = K.new_workspace(cfg), K.new_workspace(one)
    ra, rb = K.new_records(cfg), K.new_records(cfg).view(B, -1)
    oa, ob = (torch.empty(B, H, d, device="cuda") for _ in range(2))
    for t in range(3):
        x = _inputs(B, H, d, t == 1, t)
        K.kda_step(cfg, ra, *x, oa, ws)
        for b in range(B):
            K.kda_step(one, rb[b], *(a[b].contiguous() for a in x), ob[b], ws1)
        say(f"routes d=256 B={B} t={t}")
        assert torch.equal(ra.view(B, -1), rb) and torch.equal(oa, ob)
