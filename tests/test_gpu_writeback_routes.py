"""The decode step's write-backs by grid size (one lane per clip factor, four
lanes per group of factors, a block per head) are one function: the step on the
workspace, whose route depends on B H, against kda_step_noalloc, which always
rebuilds the state from the record in a block per head (d_k <= 128), and one
launch of many heads against the same heads in launches of few (d_k = 256, the
prefill's intervals, the codec).  Head counts lie at the edges of the routes'
ranges."""
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
    (32, 32, 64, {}), (33, 32, 64, dict(b_min=1, mean_bits=2.5)), (33, 32, 64, dict(b_max=12, mean_bits=7.0)), (1, 1, 128, dict(b_min=1, mean_bits=2.5)), (2, 32, 128, dict(group_rows=64)), (5, 13, 128, {}),
    (8, 32, 128, dict(mean_bits=3.0)), (9, 29, 128, {}), (2, 2, 128, dict(b_max=16, mean_bits=9.0)), (2, 2, 64, dict(b_max=16, mean_bits=8.5)),
    (2, 6, 128, dict(group_rows=3 * 128, b_min=1)), (3, 5, 128, dict(scope=1, b_min=1, mean_bits=2.0)),
    # four lanes with int16 codes
    (5, 13, 128, dict(b_max=12, mean_bits=7.0)), (9, 32, 64, dict(b_max=16, mean_bits=8.5)),
    # rows of two bits only: the fit's ternary form, with four lanes against one and two
    (5, 13, 128, dict(mean_bits=2.0)), (8, 32, 128, dict(mean_bits=2.25)), (9, 32, 64, dict(mean_bits=2.0)),
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


@pytest.mark.parametrize("B", [2, 3, 6, 7, 17])
def test_routes_at_256(B):
    # heads per launch: 32 (one round, widths selected inside), 48 and 96, 112 (a block per head),
    # 272 (the same with two segments per thread)
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


PREFILLS = [
    # 128: more than 64 heads (four lanes, two blocks per head; chunked: each selects its widths)
    (5, 13, 128, {}), (5, 13, 128, dict(b_max=12, mean_bits=7.0, group_rows=64)),
    (5, 13, 128, dict(scope=1, b_min=1, mean_bits=2.5, group_rows=64)), (5, 13, 128, dict(scope=1, b_max=16, mean_bits=9.0)),
    (3, 24, 128, dict(group_rows=12 * 128, b_min=1)),
    # 64: more than 256 heads; 256: more than 32 (a block per head)
    (9, 29, 64, {}), (9, 29, 64, dict(b_max=16, mean_bits=8.5)), (3, 11, 256, dict(b_min=1, mean_bits=2.5)),
]


@pytest.mark.parametrize("B,H,d,kw,chunked",
                         [(*p, c) for p in PREFILLS for c in ((0, 1) if p[2] <= 128 else (0,))])
def test_prefill_routes_write_the_same_records(B, H, d, kw, chunked):
    # all sequences in one call against calls of one sequence (one lane per clip factor)
    C, T = 16, 40
    cfg, one = (_cfg(n, H, d, chunked=chunked, **kw) for n in (B, 1))
    g = torch.Generator(device="cuda").manual_seed(d + H)
    unit = lambda: torch.nn.functional.normalize(torch.randn(B, T, H, d, generator=g, device="cuda"), dim=-1).bfloat16()  # noqa: E731
    q, k = unit(), unit()
    v = torch.randn(B, T, H, d, generator=g, device="cuda")
    v[-1] *= torch.exp(3 * torch.randn(T, H, d, generator=g, device="cuda"))   # heavy tails in the last sequence
    v[0, :, 0] = 0.0                                                           # a head whose state stays zero
    x = (q, k, v.bfloat16(), torch.exp(-7 * torch.rand(B, T, H, d, generator=g, device="cuda")),
         torch.sigmoid(torch.randn(B, T, H, generator=g, device="cuda")))
    ra, rb = K.new_records(cfg), K.new_records(cfg).view(B, -1)
    oa, ob = (torch.empty(B, T, H, d, device="cuda") for _ in range(2))
    K.kda_prefill(cfg, T, C, ra, *x, oa, K.new_workspace(cfg))
    ws = K.new_workspace(one)
    for b in range(B):
        K.kda_prefill(one, T, C, rb[b], *(a[b] for a in x), ob[b], ws)
    assert torch.equal(ra.view(B, -1), rb) and torch.equal(oa, ob)


@pytest.mark.parametrize("d,B,H,bmin,bmax", [
    (64, 33, 32, 1, 8), (64, 33, 32, 1, 16), (128, 9, 29, 1, 8), (128, 9, 29, 1, 16), (128, 23, 28, 1, 8),
    (256, 17, 16, 1, 8),   # 272 heads: two segments per thread instead of one
    # rows of two bits only: the ternary form with one, two and four lanes
    (64, 33, 32, 2, 2), (128, 9, 29, 2, 2), (128, 23, 28, 2, 2),
])
def test_pack_routes_write_the_same_records(d, B, H, bmin, bmax):
    # more than 256 and 640 (d = 128), 1024 (d = 64) or 256 (d = 256) heads in one call against the
    # same heads in calls of few (whose route the codec tests pin to the oracle)
    g = torch.Generator(device="cuda").manual_seed(d + B)
    S = torch.randn(B, H, d, d, generator=g, device="cuda") * torch.exp(4 * torch.randn(B, H, d, 1, generator=g, device="cuda"))
    S[0, 0, 1] = 0.0
    S[1, :, 2, ::3] = -0.0
    bits = torch.randint(bmin, bmax + 1, (B, H, d), generator=g, device="cuda").to(torch.uint8)
    s_hat = torch.rand(B, H, d, generator=g, device="cuda").double() + 1e-4
    r = torch.rand(B, H, d, generator=g, device="cuda").double() / d
    cfg, one = (_cfg(n, H, d, b_min=bmin, b_max=bmax, mean_bits=(bmin + bmax) / 2) for n in (B, 1))
    # outside a record's meaningful bytes nothing is written, inside everything:
    # start from ones
    ra = torch.full_like(K.new_records(cfg), 255)
    rb = torch.full_like(ra, 255).view(B, -1)
    K.kda_pack_state(cfg, S, bits, s_hat, r, 7, ra)
    for b in range(B):
        K.kda_pack_state(one, S[b].contiguous(), bits[b].contiguous(), s_hat[b].contiguous(), r[b].contiguous(), 7, rb[b])
    assert torch.equal(ra.view(B, -1), rb)
