"""Performance cases of the library's public entry points.

A case is a dict of plain values:
  kind   step      one decode token with its write-back (kda_step)
         prefill   a prompt from the empty state (kda_prefill; chunked = 1: the
                   MFMA form, 2: the same with a second stream of the caller's)
         codec     dense states into records and back (kda_alloc_bits,
                   kda_pack_state, kda_unpack_state)
         weights   window Gramian row weights (kda_weights)
  B H d  sequences, heads, head width (d_k = d_v)
  T C    tokens (prefill: of the prompt; weights: of the window) and the
         write-back interval
  mean bmin bmax G   payload budget, width clamp, normalisation group rows
  decay  "channel" (per row and token), "static" (per row, constant in time),
         "head" (one rate per head and token)
  erase  False: no erasure (Mamba-2)
  units  "row", or "head" (one width per head, block scales)
  heavy  True: heavy-tailed values (Student-t, 3 degrees of freedom)
  given  True: row weights given by the caller (from a query window)

Inputs follow the recipes of workloads.py, drawn on the GPU.
"""
import math

import torch

import paper_2609_30950_amd as K

WARM = 32        # tokens in hand: the warm-up from the zero state and the steps cycle through them
PREFILL_MAX = 4 * 32 * 8192 * 128 * 128   # state elements x tokens of the largest prefill


def _case(kind, B, H, d, **kw):
    c = dict(kind=kind, B=B, H=H, d=d, T=1, C=1, mean=4.0, bmin=2, bmax=8, G=d, decay="channel",
             erase=True, units="row", chunked=0, heavy=False, given=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest layer: two heads of 64, one token (launches and latency)
        dict(_case("step", 1, 2, 64, G=64), name="step_tiny"),
        # one request being decoded on a Kimi-Linear-shaped layer
        dict(_case("step", 1, 32, 128), name="step_one_request"),
        # a decode batch on that layer (the benchmark's default workload)
        dict(_case("step", 64, 32, 128, G=64), name="step_batch"),
        # a large long-context batch at three bits with heavy-tailed values, row
        # weights recomputed by the caller from a query window
        dict(_case("step", 128, 32, 128, mean=3.0, G=64, heavy=True, given=True), name="step_long_context"),
        # Gated-DeltaNet-shaped layer, a width per row at two bits
        dict(_case("step", 16, 16, 256, mean=2.0, bmin=1, decay="head"), name="step_gdn_rows"),
        # the same layer with that architecture's unit, a width per head, at six bits
        dict(_case("step", 16, 16, 256, mean=6.0, decay="head", units="head"), name="step_gdn_heads"),
        # Mamba-2-shaped layer: no erasure, normalisation groups of 12 heads
        dict(_case("step", 16, 24, 128, bmin=1, G=12 * 128, decay="head", erase=False), name="step_mamba2"),
        # a ragged batch of prompts in the bit-reproducible token-sequential form
        dict(_case("prefill", 4, 32, 128, T=2000, C=64, bmin=1, decay="static"), name="prefill_sequential"),
        # long prompts in the chunked form with a second stream (the prefill workload)
        dict(_case("prefill", 4, 32, 128, T=8192, C=64, bmin=1, decay="static", chunked=2), name="prefill_chunked"),
        # one ragged prompt in the chunked form on one stream
        dict(_case("prefill", 1, 32, 128, T=1000, C=64, bmin=1, decay="static", chunked=1), name="prefill_one_prompt"),
        # states of a batch encoded into records and decoded (saving, moving, inspecting)
        dict(_case("codec", 16, 32, 128), name="codec"),
        # row weights of a long-context layer from a 1024-token query window
        dict(_case("weights", 32, 32, 128, T=1024, G=64), name="window_weights"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step"] * 7 + ["prefill"] * 3 + ["codec", "weights"])
    d = rng.choice([64, 128, 128, 128, 256])
    H = rng.choice([h for h in (1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64) if h * d <= 4096])
    bmin = rng.choice([1, 2])
    mean = rng.choice([2.0, 2.5, 3.0, 3.75, 4.0, 4.0, 5.0, 6.0])
    bmax = rng.choice([8, 8, 8, 7, 6])
    decay = rng.choice(["channel", "channel", "head"])
    G = rng.choice([d, d, 64])
    if kind == "step":
        B = _log_int(rng, 1, 128)
        while B * H * d * d > 128 * 32 * 128 * 128:
            B = max(1, B // 2)
        units = rng.choice(["row", "row", "row", "row", "head"])
        if units == "head":
            return _case(kind, B, H, d, mean=mean, bmin=2, bmax=bmax, decay="head", units="head")
        erase = rng.random() > 0.2
        if not erase and H % 2 == 0:
            G = d * (H // 2)
        return _case(kind, B, H, d, mean=mean, bmin=bmin, bmax=bmax, G=G, decay=decay, erase=erase,
                     heavy=rng.random() < 0.25, given=rng.random() < 0.2)
    if kind == "prefill":
        chunked = rng.choice([0, 1, 2]) if d <= 128 else 0
        C = rng.choice([16, 32, 48, 64, 64, 64])
        B = _log_int(rng, 1, 8)
        T = _log_int(rng, 1, 64 * C)
        while B * H * d * d * T > PREFILL_MAX:
            T = max(1, T // 2)
        return _case(kind, B, H, d, T=T, C=C, mean=mean, bmin=bmin, bmax=bmax, G=G,
                     decay=rng.choice(["static", "static", "head"]), chunked=chunked)
    if kind == "codec":
        B = _log_int(rng, 1, 32)
        while B * H * d * d > 32 * 32 * 128 * 128:
            B = max(1, B // 2)
        return _case(kind, B, H, d, mean=mean, bmin=bmin, bmax=bmax, G=G)
    B = _log_int(rng, 1, 32)
    T = _log_int(rng, 16, 1024)
    while B * H * d * T > 32 * 32 * 128 * 1024:
        B = max(1, B // 2)
    return _case(kind, B, H, d, T=T, C=rng.choice([1, 1, 16, 64]), G=d, decay=decay)


# ------------------------------------------------------------- inputs ---

def _config(c):
    return K.Config(B=c["B"], H=c["H"], d_k=c["d"], d_v=c["d"], group_rows=c["G"], mean_bits=c["mean"],
                    b_min=c["bmin"], b_max=c["bmax"], decay_per_head=int(c["decay"] == "head"),
                    no_erase=int(not c["erase"]), chunked=int(c["chunked"] > 0),
                    head_units=int(c["units"] == "head"))


def _unit(g, *shape):
    x = torch.randn(*shape, generator=g, device="cuda")
    return x / x.norm(dim=-1, keepdim=True)


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device="cuda")


def _log_uniform(g, lo, hi, *shape):
    return torch.exp(_uniform(g, math.log(lo), math.log(hi), *shape))


def _values(c, g, *shape):
    v = torch.randn(*shape, generator=g, device="cuda")
    if c["heavy"]:
        v = v / (sum(torch.randn(*shape, generator=g, device="cuda").square() for _ in range(3)) / 3).sqrt()
    return v


def _base(c, g):
    """Per-row base rates [B, H, d]."""
    shape = (c["B"], c["H"], c["d"])
    if c["decay"] == "static":
        slow = torch.rand(*shape, generator=g, device="cuda") < 0.1
        return torch.where(slow, _log_uniform(g, 1e-4, 1e-3, *shape), _log_uniform(g, 1e-3, 2.0, *shape))
    return _log_uniform(g, 1e-3, 1.0, *shape)


def _rates(c, g, *lead):
    """Rates s of tokens with leading axes `lead` = (T,) (steps) or (B, T)."""
    B, H, d = c["B"], c["H"], c["d"]
    steps = len(lead) == 1
    if c["decay"] == "head":
        return _log_uniform(g, 1e-4, 1.0, *((lead[0], B, H) if steps else (*lead, H)))
    base = _base(c, g)
    shape = (lead[0], B, H, d) if steps else (*lead, H, d)
    base = base if steps else base[:, None]
    if c["decay"] == "static":
        return base.expand(shape).contiguous()
    return (base + 0.05 * torch.randn(*shape, generator=g, device="cuda")).clamp_(min=1e-4)


def prepare(case, seed):
    c, B, H, d, T = case, case["B"], case["H"], case["d"], case["T"]
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    cfg = _config(c)
    if c["kind"] == "weights":
        return dict(case=c, cfg=cfg, q=_unit(g, B, T, H, d), k=_unit(g, B, T, H, d), s=_rates(c, g, B, T),
                    beta=torch.sigmoid(torch.randn(B, T, H, generator=g, device="cuda")),
                    gamma=torch.empty(B, H, d, dtype=torch.float64, device="cuda"))
    if c["kind"] == "codec":
        # rows whose scales differ as the decay rates make them differ
        s_hat = _log_uniform(g, 1e-3, 1.0, B, H, d).double()
        r = 0.5 * torch.rand(B, H, d, generator=g, device="cuda").double() / d
        S = torch.randn(B, H, d, d, generator=g, device="cuda") / s_hat.float().mul(2 * d).sqrt()[..., None]
        gamma = 1.0 / torch.expm1(2.0 * (s_hat + r))
        return dict(case=c, cfg=cfg, S=S, R=S.abs().amax(-1), gamma=gamma, s_hat=s_hat, r=r,
                    bits=torch.empty(B, H, d, dtype=torch.uint8, device="cuda"), recs=K.new_records(cfg),
                    ws=K.new_workspace(cfg), S_out=torch.empty_like(S), s_out=torch.empty_like(s_hat),
                    r_out=torch.empty_like(r))
    if c["kind"] == "prefill":
        bf = torch.bfloat16
        return dict(case=c, cfg=cfg, q=_unit(g, B, T, H, d).to(bf), k=_unit(g, B, T, H, d).to(bf),
                    v=_values(c, g, B, T, H, d).to(bf), s=_rates(c, g, B, T),
                    beta=torch.sigmoid(torch.randn(B, T, H, generator=g, device="cuda")),
                    recs=K.new_records(cfg), ws=K.new_workspace(cfg),
                    o=torch.empty(B, T, H, d, device="cuda"), S=torch.empty(B, H, d, d, device="cuda"),
                    aux=torch.cuda.Stream() if c["chunked"] == 2 else None)
    # decode: the records of a layer after WARM tokens from the zero state, and
    # the tokens to come (the same ones again)
    st = dict(case=c, cfg=cfg, q=_unit(g, WARM, B, H, d), k=_unit(g, WARM, B, H, d),
              v=_values(c, g, WARM, B, H, d), s=_rates(c, g, WARM),
              beta=torch.sigmoid(torch.randn(WARM, B, H, generator=g, device="cuda")),
              gamma=_log_uniform(g, 1e-2, 1e3, B, H, d).double() if c["given"] else None,
              recs=K.new_records(cfg), ws=K.new_workspace(cfg), o=torch.empty(B, H, d, device="cuda"), t=0)
    for _ in range(WARM):
        _step(st)
    return st


# --------------------------------------------------------------- runs ---

def _step(st):
    t = st["t"]
    st["t"] = (t + 1) % WARM
    K.kda_step(st["cfg"], st["recs"], st["q"][t], st["k"][t], st["v"][t], st["s"][t], st["beta"][t], st["o"],
               st["ws"], gamma=st["gamma"])


def run(state):
    st, c, cfg = state, state["case"], state["cfg"]
    if c["kind"] == "step":
        _step(st)
        return dict(o=st["o"], records=st["recs"])
    if c["kind"] == "prefill":
        st["recs"].zero_()   # a new prompt starts from the zero state
        K.kda_prefill(cfg, c["T"], c["C"], st["recs"], st["q"], st["k"], st["v"], st["s"], st["beta"], st["o"],
                      st["ws"], aux_stream=st["aux"])
        # outputs of the first write-back interval and of the later ones
        out = dict(o_first=st["o"][:, :c["C"]], o_later=st["o"][:, c["C"]:])
        if c["chunked"]:
            # the chunked form's state agrees to rounding, so its codes may fall
            # on the other side of a tie: the state as values
            K.kda_unpack_state(cfg, st["recs"], S=st["S"])
            out["state"] = st["S"]
        else:
            out["records"] = st["recs"]
        return out
    if c["kind"] == "codec":
        K.kda_alloc_bits(cfg, st["gamma"], st["R"], st["bits"], st["ws"])
        K.kda_pack_state(cfg, st["S"], st["bits"], st["s_hat"], st["r"], 1, st["recs"])
        K.kda_unpack_state(cfg, st["recs"], S=st["S_out"], s_hat=st["s_out"], r=st["r_out"])
        return dict(bits=st["bits"], state=st["S_out"], s_hat=st["s_out"], r=st["r_out"])
    K.kda_weights(cfg, c["T"], c["C"], st["q"], st["s"], st["beta"], st["k"], st["gamma"])
    return dict(gamma=st["gamma"])


def work(case):
    """Bytes: every input once, records at the budgeted payload with their
    metadata in and out (prefill: one write-back's record, the state stays on
    the chip in between), outputs once.  Flops: decay, erase, write and read
    of eq. rule (7 per state element and token; with the products of the
    chunked form these are its flops to leading order as well), and per
    write-back a decode, a scale, a rounding and a clamp of every element."""
    c = case
    n, d = c["B"] * c["H"], c["d"]
    meta = 16 + d // 2 + 6 * d if c["units"] == "row" else 16 + 4 * d + d * d // 16
    rec = n * (meta + c["mean"] * d * d / 8)
    rate = 4 * (1 if c["decay"] == "head" else d)
    if c["kind"] == "step":
        return dict(bytes=2 * rec + n * (12 * d + rate + 4 + 4 * d + (8 * d if c["given"] else 0)),
                    flops=n * d * d * (7 + 4))
    if c["kind"] == "prefill":
        nwb = -(-c["T"] // c["C"])
        return dict(bytes=rec + n * c["T"] * (6 * d + rate + 4 + 4 * d) + (4 * n * d * d if c["chunked"] else 0),
                    flops=n * d * d * (7 * c["T"] + 4 * nwb))
    if c["kind"] == "codec":
        return dict(bytes=2 * rec + n * d * (8 * d + 37), flops=n * d * d * 5)
    return dict(bytes=n * c["T"] * (8 * d + rate + 4) + 8 * n * d, flops=n * c["T"] * d * 12)


def tolerance(case):
    # The float32 contract fixes every sum's order, so codes and records are the
    # same bytes and outputs differ by the last bits of a transcendental at most.
    if case["kind"] == "step" or (case["kind"] == "prefill" and not case["chunked"]):
        return {"rel": 1e-6, "differ": 1e-5}
    # Chunked: products of split bf16 operands (7e-6 on the first interval).  At
    # each write-back a rounding falls on the other side of ties between codes,
    # clip factors and widths, and the quantised state carries that on: against
    # the token-sequential form, 0.2% of the state after one write-back, 1 to 2.5%
    # of the outputs and 3 to 5% of the state after 8 to 128 of them.
    if case["kind"] == "prefill":
        return {"rel": 1e-2, "max": 0.99} if case["T"] <= case["C"] else {"rel": 3e-2, "max": 0.99}
    if case["kind"] == "codec":
        return "exact"
    return {"rel": 1e-12}   # float64 sums


# ------------------------------------------- the same in plain float64 ---

def _decode_records(c, recs):
    """Dequantised states [n, d, d] (float64) of records in the layout of kda.h."""
    n, d = c["B"] * c["H"], c["d"]
    raw = recs.view(n, -1)
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    f16 = lambda a, b: raw[:, a:b].contiguous().view(torch.float16).double()  # noqa: E731
    if c["units"] == "row":
        wb = raw[:, 16:16 + d // 2].long()
        w = torch.stack([wb & 15, wb >> 4], -1).view(n, d) + 1
        a = 16 + d // 2
        scale = f16(a, a + 2 * d)[:, :, None]
        off = up(a + 6 * d)
    else:
        w = raw[:, 4:8].contiguous().view(torch.int32).long().expand(n, d)
        a = 16 + 4 * d
        scale = f16(a, a + d * d // 16).view(n, d // 32, d).repeat_interleave(32, dim=1)
        off = up(a + d * d // 16)
    P = w.cumsum(1) - w
    nw = (d * c["bmax"] + 31) // 32
    words = raw[:, off:off + nw * d * 4].contiguous().view(torch.int32).view(n, nw, d).long() & 0xFFFFFFFF
    at = (P >> 5)[:, :, None].expand(n, d, d)
    lo, hi = words.gather(1, at), words.gather(1, (at + 1).clamp(max=nw - 1))
    w, sh = w[:, :, None], (P & 31)[:, :, None]
    code = ((lo | (hi << 32)) >> sh) & ((1 << w) - 1)
    signed = code - ((code >> (w - 1)) << w)
    return torch.where(w == 1, 1 - 2 * code, signed).double() * scale


def _recur(c, S, q, k, v, s, beta):
    """One token of eq. rule on S [n, d, d]; returns the state and o [n, d]."""
    n, d = S.shape[0], S.shape[1]
    q, k, v = (x.reshape(n, d).double() for x in (q, k, v))
    s = s.reshape(n, -1).double()
    bk = beta.reshape(n, 1).double() * k
    S = S * torch.exp(-s)[:, :, None]
    w = v - (S * k[:, :, None]).sum(1) if c["erase"] else v
    S = S + bk[:, :, None] * w[:, None, :]
    return S, (S * q[:, :, None]).sum(1)


def exact(case, seed):
    c, B, H, d = case, case["B"], case["H"], case["d"]
    st = prepare(case, seed)
    if c["kind"] == "step":
        S = _decode_records(c, st["recs"])
        _, o = _recur(c, S, st["q"][0], st["k"][0], st["v"][0], st["s"][0], st["beta"][0])
        return dict(o=o.view(B, H, d), records=None)
    if c["kind"] == "prefill":
        S, o = torch.zeros(B * H, d, d, dtype=torch.float64, device="cuda"), []
        for t in range(min(c["T"], c["C"])):
            S, ot = _recur(c, S, *(st[n][:, t] for n in ("q", "k", "v", "s", "beta")))
            o.append(ot.view(B, H, d))
        last = "state" if c["chunked"] else "records"
        # later intervals start from a quantised state
        return {"o_first": torch.stack(o, 1), "o_later": None, last: None}
    if c["kind"] == "codec":
        return _exact_codec(c, st)
    A = torch.zeros(B, H, d, dtype=torch.float64, device="cuda")
    acc = torch.zeros_like(A)
    for t in range(1, c["T"]):
        s, b, k, q = (st[n][:, t].double() for n in ("s", "beta", "k", "q"))
        s = s[..., None] if c["decay"] == "head" else s
        lam = torch.exp(-2 * s - (b * (2 - b))[..., None] * k * k)
        A = lam * ((1.0 if t % c["C"] == 0 else 0.0) + A)
        acc += q * q * A
    return dict(gamma=acc / c["T"])


def _exact_codec(c, st):
    n, d = c["B"] * c["H"], c["d"]
    # widths: the budget's slots in the order of c_i 4^-l over a sequence's rows
    R = st["R"].double()
    Rt = R / R.view(n, -1, c["G"]).square().mean(-1, keepdim=True).sqrt().expand(-1, -1, c["G"]).reshape(R.shape)
    N = c["H"] * d
    lev = torch.arange(c["bmin"] + 1, c["bmax"] + 1, device="cuda")
    val = ((st["gamma"] * Rt * Rt).view(c["B"], N, 1) * 4.0 ** -lev.double()).view(c["B"], -1)
    need = int(math.floor(c["mean"] * N + 0.5)) - N * c["bmin"]
    got = torch.zeros_like(val).scatter_(1, val.topk(need, 1).indices, 1.0) if need else torch.zeros_like(val)
    b = (c["bmin"] + got.view(c["B"], N, -1).sum(-1)).long().view(n * d, 1)
    # the clip factor of least squared error for every row, scales in FP16
    x, R = st["S"].view(n * d, d).double(), R.view(-1, 1)
    lv = (2.0 ** (b - 1) - 1).clamp(min=1)
    mu = x.abs().mean(1, keepdim=True).half().double()
    one = torch.where(x < 0, -mu, mu)
    best, y = torch.full_like(R, math.inf), torch.zeros_like(x)
    for m in range(16):
        D = (R * (5 + m) / 20 / lv).half().double()
        z = torch.minimum(torch.maximum((x / D.clamp(min=1e-30)).round(), -lv), lv) * D
        err = (x - z).square().sum(1, keepdim=True)
        y, best = torch.where(err < best, z, y), torch.minimum(err, best)
    y = torch.where(b == 1, one, y)
    step = 25.0 / 65535.0
    zc = ((torch.log2(st["s_hat"]) + 20.0) / step).round().clamp(0, 65535)
    return dict(bits=None, state=y.view(st["S"].shape), s_hat=torch.exp2(zc * step - 20.0),
                r=st["r"].half().double())
