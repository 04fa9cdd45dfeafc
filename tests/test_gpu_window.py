"""kda_weights at the edges of its token tiles (16 tokens: one, a remainder,
a whole tile, several) and of the windows that its rows take in turn, against
the oracle's float64 recursion and of one form against the other."""
import numpy as np
import pytest
import torch

import paper_2609_30950_amd as K
import workloads as W
from oracle import stats
from tests._gpu import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Wn,C", [(1, 1), (2, 1), (4, 1), (5, 2), (16, 3), (17, 1), (18, 64), (33, 16), (50, 7)])
@pytest.mark.parametrize("d,per_head,erase", [(64, False, True), (128, True, False), (256, True, True),
                                              (128, False, False)])
def test_window_weights_at_tile_edges(Wn, C, d, per_head, erase):
    B, H = 2, 3
    w = W.sized(W.WORKLOADS["gdn2" if per_head else "tiny"], B=B, H=H, dk=d, dv=d)
    x = W.tokens(w, 0, Wn)
    cfg = K.Config(B=B, H=H, d_k=d, d_v=d, group_rows=d, decay_per_head=int(per_head), no_erase=int(not erase))
    g = torch.full((B * H * d,), -1.0, dtype=torch.float64, device="cuda")
    s_arg = x["s"][..., 0] if per_head else x["s"]
    K.kda_weights(cfg, Wn, C, dev(x["q"]), dev(s_arg), dev(x["beta"]), dev(x["k"]), g)
    s_full = np.broadcast_to(x["s"], x["k"].shape)
    want = stats.window_gamma(*(np.moveaxis(a, 1, 0) for a in (x["q"], s_full, x["k"], x["beta"])), C, erase=erase)
    # sums of non-negative terms in the same order; exp arguments of magnitude
    # below 10, so each factor agrees within some 20 ulp and 50 of them within 2e-13
    np.testing.assert_allclose(host(g).reshape(B, H, d), want, rtol=1e-12)


@pytest.mark.parametrize("Wn,C", [(7, 3), (16, 1), (17, 5), (32, 7)])
@pytest.mark.parametrize("per_head,erase", [(False, True), (True, True), (False, False), (True, False)])
def test_windows_of_many_rows_equal_those_of_few(Wn, C, per_head, erase):
    """131072 rows take windows of up to 16 or 32 tokens in turn, 4096 rows only up to four:
    the same operations per row in the same order, so the same bits."""
    B, H, d = 32, 32, 128
    gen = torch.Generator(device="cuda").manual_seed(Wn)
    q, k = (torch.randn(B, Wn, H, d, generator=gen, device="cuda") for _ in range(2))
    s = torch.rand(*((B, Wn, H) if per_head else (B, Wn, H, d)), generator=gen, device="cuda")
    beta = torch.rand(B, Wn, H, generator=gen, device="cuda")
    many, few = (torch.full((B, H, d), -1.0, dtype=torch.float64, device="cuda") for _ in range(2))
    cfg, one = (K.Config(B=n, H=H, d_k=d, d_v=d, group_rows=d, decay_per_head=int(per_head), no_erase=int(not erase))
                for n in (B, 1))
    K.kda_weights(cfg, Wn, C, q, s, beta, k, many)
    for b in range(B):
        K.kda_weights(one, Wn, C, q[b], s[b], beta[b], k[b], few[b])
    assert torch.equal(many, few)


def test_window_weights_of_more_rows_than_one_grid():
    """2^30 + 4096 rows (more blocks than a launch takes, so two launches): all
    rows of a two-token window, in closed form."""
    B, H, d = 2**18 + 1, 64, 64
    n = B * H
    cfg = K.Config(B=B, H=H, d_k=d, d_v=d, group_rows=d, decay_per_head=1, no_erase=0)
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k = (torch.rand(B, 2, H, d, generator=gen, device="cuda") for _ in range(2))
    s, beta = (torch.rand(B, 2, H, generator=gen, device="cuda") for _ in range(2))
    g = torch.full((B, H, d), -1.0, dtype=torch.float64, device="cuda")
    assert n * d == 2**30 + 4096
    K.kda_weights(cfg, 2, 1, q, s, beta, k, g)
    for b0 in range(0, B, 2**14):
        sl = slice(b0, b0 + 2**14)
        q1, k1, s1, b1 = (x[sl, 1].double() for x in (q, k, s, beta))
        lam = torch.exp(-2 * s1[..., None] - (b1 * (2 - b1))[..., None] * k1 * k1)
        # one product of three float64 factors: a few ulp, as above
        torch.testing.assert_close(g[sl], q1 * q1 * lam / 2, rtol=1e-12, atol=0.0)
