"""The work that users of the library have it do, as measurable cases.

Each case is a dict of plain values; `prepare` makes what a program holds
before the call (device tensors drawn from a seed, operands quantized once),
`run` is one pass through the public Python binding, `work` the bytes and
operations the pass cannot do without, `exact` the same result from plain
torch in 64 bits.

Calls (`op`):

* forward       self-attention of bf16 Q, K, V (a video transformer's block);
* cross         bf16 Q over bf16 K, V of another length (text context, or the
                text segment's queries over a video);
* step          one denoising step's cross-attention on a prompt whose K^, V^
                were quantized once: quantize Q, then attend;
* quantize      MXFP4 operands of Q, K (head-dim blocks) and V (token blocks);
* sweep         squared error over scale boundaries, K along d and V along N;
* diag          row-sum statistics of every attention row, P not materialized;
* rows          a tile of query rows of P materialized, then its statistics.
"""
from __future__ import annotations

import math

import torch

from paper_2607_24377_amd import mxattn

D = 128
MODES = ("ocp_vanilla", "uos", "uos_pnq", "uos_pnq_rot")
SWEEP = [6.0 + 0.05 * i for i in range(41)]  # the boundaries of the paper's sweep


def _case(name, op, H, Nq, Nkv, mode, kind, B=1, **more):
    c = dict(op=op, B=B, H=H, Nq=Nq, Nkv=Nkv, mode=mode, kind=kind, **more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest self-attention of the tests and the smoke run: launches and latency
        _case("fwd_tiny", "forward", 2, 512, 512, "uos_pnq", "iid"),
        # short clips / image tokens with outlier channels, in the baseline mode
        _case("fwd_4k", "forward", 40, 4096, 4096, "ocp_vanilla", "outlier"),
        # one GPU's heads (5 of 40) of the same call sharded by heads over 8 GPUs
        _case("fwd_4k_shard", "forward", 5, 4096, 4096, "uos_pnq", "outlier"),
        # a 480p video block with the full method (rotation, UOS, PNQ)
        _case("fwd_480p", "forward", 40, 32760, 32760, "uos_pnq_rot", "video"),
        # the 720p headline workload
        _case("fwd_720p", "forward", 40, 75600, 75600, "uos_pnq", "video"),
        # 720p video queries over a 512-token text context
        _case("cross_720p_text", "cross", 40, 75600, 512, "uos_pnq", "cross"),
        # the 256 text queries of a joint block over its whole video (ragged last tile)
        _case("text_over_video", "cross", 24, 256, 118800, "uos", "video"),
        # one denoising step at 480p over a ragged prompt quantized beforehand
        _case("step_480p_prompt", "step", 40, 32760, 333, "uos", "cross"),
        # the operands of a 480p block
        _case("quant_480p", "quantize", 40, 32760, 32760, "uos_pnq", "video"),
        # the paper's boundary sweep on a 480p block's K and V
        _case("sweep_480p", "sweep", 40, 32760, 32760, "uos", "video"),
        # row-sum statistics of a whole 4096-token call
        _case("diag_4k", "diag", 40, 4096, 4096, "uos", "outlier", gamma=1.0),
        # a 128-row tile of P at 480p, materialized and diagnosed
        _case("rows_480p", "rows", 40, 32760, 32760, "uos", "video", rows=128, gamma=1.0),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["forward", "forward", "forward", "cross", "cross", "step", "quantize", "sweep", "diag", "rows"])
    B = rng.choice([1, 1, 1, 2])
    H = rng.choice([1, 2, 3, 5, 10, 24, 40])
    mode = rng.choice(MODES)
    Nq = _log_int(rng, 1, 75600)
    Nkv = Nq
    more = {}
    # head-query-key triples of a pass: at most those of the largest listed case of the kind
    most = {"forward": 40 * 75600 ** 2, "diag": 40 * 4096 ** 2, "rows": 40 * 128 * 32760}
    if op in ("cross", "step"):
        Nkv = _log_int(rng, 1, 118800) if rng.random() < 0.5 else _log_int(rng, 1, 512)
    if op in ("diag", "rows"):
        more["gamma"] = rng.choice([1.0, 1.0, 1.37])
        mode = rng.choice(["ocp_vanilla", "uos"])
    if op == "rows":
        Nkv = _log_int(rng, 1, 32760)
        Nq = Nkv
        more["rows"] = min(Nq, rng.choice([1, 64, 100, 128]))
    if op == "sweep":
        mode = "uos"
    if op in ("quantize", "sweep"):
        Nq = Nkv = _log_int(rng, 1, 32760)
    else:
        cap = most.get(op, 40 * 75600 ** 2 // 4)
        while B * H * more.get("rows", Nq) * Nkv > cap:
            if B > 1:
                B = 1
            elif H > 5:
                H = 5
            else:
                Nkv = max(1, Nkv // 2)
                if op in ("forward", "diag", "rows"):
                    Nq = Nkv
                    if op == "rows":
                        more["rows"] = min(Nq, more["rows"])
    kind = rng.choice(["iid", "outlier", "video"]) if Nq == Nkv else "cross"
    if op in ("diag", "rows") and mode == "ocp_vanilla":
        kind = "iid"  # the floor rule jumps at a probability of 1, which only flat rows keep away from
    return _case(None, op, H, Nq, Nkv, mode, kind, B, **more)


# ---------------------------------------------------------------------------
# Inputs: the distributions of the synthetic workloads, drawn on the device.


def _student_t4(shape, g):
    z = torch.randn(shape, generator=g, device="cuda")
    u = torch.rand((2,) + tuple(shape), generator=g, device="cuda").clamp_(min=1e-30)
    return z * torch.rsqrt(-0.5 * (u[0].log_() + u[1].log_()))  # chi2_4 = -2 ln(u0 u1)


def _inputs(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    B, H, Nq, Nkv, kind = c["B"], c["H"], c["Nq"], c["Nkv"], c["kind"]
    q = torch.empty((B, H, Nq, D), dtype=torch.bfloat16, device="cuda")
    k = torch.empty((B, H, Nkv, D), dtype=torch.bfloat16, device="cuda")
    v = torch.empty((B, H, Nkv, D), dtype=torch.bfloat16, device="cuda")
    for b in range(B):
        for h in range(H):
            if kind in ("video", "cross"):
                q[b, h] = _student_t4((Nq, D), g)
                x = _student_t4((Nkv, D), g)
                if kind == "cross":
                    x *= 2.0
                k[b, h] = x + math.sqrt(2.0) * torch.randn((1, D), generator=g, device="cuda")
            else:
                x = torch.randn((Nq, D), generator=g, device="cuda")
                y = torch.randn((Nkv, D), generator=g, device="cuda")
                if kind == "outlier":
                    ch = torch.randperm(D, generator=g, device="cuda")[:4]
                    x[:, ch] *= 20.0
                    y[:, ch] *= 20.0
                q[b, h], k[b, h] = x, y
            v[b, h] = torch.randn((Nkv, D), generator=g, device="cuda")
    return q, k, v


def prepare(case, seed):
    q, k, v = _inputs(case, seed)
    st = dict(case=case, q=q, k=k, v=v)
    if case["op"] == "step":
        st["kq"] = mxattn.quantize(k, mxattn.AXIS_HEAD_DIM, case["mode"])
        st["vq"] = mxattn.quantize(v, mxattn.AXIS_TOKENS, case["mode"])
    return st


def run(state):
    c = state["case"]
    op, mode = c["op"], c["mode"]
    q, k, v = state["q"], state["k"], state["v"]
    if op == "forward":
        return mxattn.forward(q, k, v, mode)
    if op == "cross":
        return mxattn.cross_forward(q, k, v, mode)
    if op == "step":
        qc, qs = mxattn.quantize(q, mxattn.AXIS_HEAD_DIM, mode)
        return mxattn.cross_attend(qc, qs, *state["kq"], *state["vq"], c["Nq"], c["Nkv"], mode)
    if op == "quantize":
        return (mxattn.quantize(q, mxattn.AXIS_HEAD_DIM, mode), mxattn.quantize(k, mxattn.AXIS_HEAD_DIM, mode),
                mxattn.quantize(v, mxattn.AXIS_TOKENS, mode))
    if op == "sweep":
        return mxattn.qmax_sse(k, mxattn.AXIS_HEAD_DIM, SWEEP), mxattn.qmax_sse(v, mxattn.AXIS_TOKENS, SWEEP)
    if op == "diag":
        return mxattn.attention_rowsum_diag(q, k, mode, c["gamma"])
    row0 = c["Nq"] - c["rows"]
    ld = (c["Nkv"] + 3) // 4 * 4
    p = mxattn.softmax_rows(q, k, row0, c["rows"], ld)
    return p, mxattn.rowsum_diag(p, c["Nkv"], mode, c["gamma"])


def work(case):
    B, H, Nq, Nkv, op = case["B"], case["H"], case["Nq"], case["Nkv"], case["op"]
    BH, nb = B * H, (Nkv + 31) // 32
    bq, bk = 2 * BH * Nq * D, 2 * BH * Nkv * D  # bf16 tensors
    qq, kq, vq = BH * Nq * (D // 2 + 4), BH * Nkv * (D // 2 + 4), BH * D * nb * 17  # codes and scales
    pairs = BH * Nq * Nkv
    if op in ("forward", "cross"):
        return dict(bytes=2 * bq + 2 * bk, flops=4 * pairs * D)
    if op == "step":
        return dict(bytes=2 * bq + kq + vq, flops=4 * pairs * D)
    if op == "quantize":
        return dict(bytes=bq + 2 * bk + qq + kq + vq, flops=0)
    if op == "sweep":
        return dict(bytes=2 * bk + 2 * 8 * BH * len(SWEEP), flops=0)
    if op == "diag":  # the scores once
        return dict(bytes=bq + bk + 64 * BH * Nq, flops=2 * pairs * D)
    rows = case["rows"]
    return dict(bytes=2 * BH * rows * D + bk + 2 * 4 * BH * rows * Nkv + 64 * BH * rows, flops=2 * BH * rows * Nkv * D)


def tolerance(case):
    op = case["op"]
    if op == "quantize":  # codes and scales are fixed bit for bit
        return "exact"
    if op in ("forward", "cross", "step"):
        # bf16 outputs: half an ulp is 2^-9 of a value (1.7e-3 in the 2-norm),
        # and sums in another order round some to the other neighbour
        return {"rel": 7e-3, "max": 1.6e-2}
    if op == "sweep":  # 32-bit squares and sums of 8, then 64 bits: 1e-9 to 6e-9 from exact
        return {"rel": 3e-8}
    # statistics of 32-bit probabilities (scores accumulated in 32 bits, whose
    # error grows with the scores: 4e-5 from exact on the video draws, 5.5e-4
    # with outlier channels): an entry next to a threshold may fall either way
    return {"rel": 2e-3 if case["kind"] == "outlier" else 2e-4}


# ---------------------------------------------------------------------------
# The same results in 64 bits from plain torch.


def _hadamard():
    h = torch.ones((1, 1), dtype=torch.float64, device="cuda")
    while h.shape[0] < D:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    return h / math.sqrt(D)


def _e2m1(y):
    """Nearest E2M1 magnitude of y >= 0, ties to the even code, saturating at 6."""
    step = torch.where(y < 2, 0.5, torch.where(y < 4, 1.0, 2.0)).to(y.dtype)
    return torch.round(y / step).mul_(step).clamp_(max=6.0)


def _exponent(M, rule):
    """Scale exponent of block maxima M: OCP floor or UOS ceil(log2(M / 7.25))."""
    f, e = torch.frexp(M)
    e = e - 3 + ((f > 0.90625) if rule == "uos" else torch.zeros_like(f, dtype=torch.bool)).to(e.dtype)
    return torch.where(M == 0, torch.zeros_like(e), e.clamp(-127, 127))


def _rule(mode):
    return "ocp" if mode == "ocp_vanilla" else "uos"


def _deq(x, rule):
    """MXFP4 value of x in blocks of 32 along the last axis (a multiple of 32 long)."""
    y = x.reshape(*x.shape[:-1], -1, 32)
    s = torch.exp2(_exponent(y.abs().amax(-1, keepdim=True), rule).double())
    return (torch.sign(y) * _e2m1(y.abs() / s) * s).reshape(x.shape)


def _pad_to(x, dim, multiple):
    short = -x.shape[dim] % multiple
    if not short:
        return x
    shape = list(x.shape)
    shape[dim] = short
    return torch.cat([x, x.new_zeros(shape)], dim)


def _exact_head(q, k, v, mode, Nkv):
    """One head's attention on bf16 q, k, v: keys in tiles of 128 under a running maximum."""
    rule = _rule(mode)
    q, k, v = q.double(), k.double(), v.double()
    if mode == "uos_pnq_rot":
        R = _hadamard()
        q, k = q @ R, k @ R
    q, k = _deq(q, rule), _pad_to(_deq(k, rule), 0, 128)
    v = _deq(_pad_to(v, 0, 128).t().contiguous(), rule).t().contiguous()
    T = k.shape[0] // 128
    out = torch.empty_like(q)
    step = max(1, (1 << 26) // k.shape[0])
    for r in range(0, q.shape[0], step):
        t = (q[r:r + step] @ k.t()).mul_(math.log2(math.e) / math.sqrt(D))
        t[:, Nkv:] = -math.inf
        n = t.shape[0]
        t = t.view(n, T, 128)
        m = torch.cummax(t.amax(-1), 1).values
        p = t.sub_(m[:, :, None]).exp2_()
        beta = torch.exp2(m - m[:, -1:])
        direct = (p.sum(-1) * beta).sum(-1)
        blocks = p.view(n, 4 * T, 32)
        s = torch.exp2(_exponent(blocks.amax(-1, keepdim=True), rule).double())
        ph = (_e2m1(blocks / s) * s).view(n, T, 128).mul_(beta[:, :, None])
        l = ph.sum((1, 2)) if "pnq" in mode else direct
        out[r:r + step] = (ph.view(n, T * 128) @ v) / l[:, None]
    return out


def _exact_stats(p, mode, gamma):
    """Row statistics [rows, 8] of fp64 p [rows, N]."""
    n, N = p.shape
    x = _pad_to(p * gamma, 1, 32)
    pp = _pad_to(p, 1, 32).view(n, -1, 32)
    y = x.view(n, -1, 32)
    s = torch.exp2(_exponent(y.amax(-1, keepdim=True), _rule(mode)).double())
    xs = y / s
    r = _e2m1(xs)
    c = r * s / gamma - pp
    zer = (pp > 0) & (r == 0)
    sat = ~zer & (xs > 6)
    dn = ~zer & ~sat & (r < xs)
    up = ~zer & ~sat & (r > xs)
    ex = ~(zer | sat | dn | up)
    ent = torch.where(pp > 0, pp * torch.log(pp.clamp(min=1e-300)), 0.0)
    part = [(r * s / gamma), pp] + [torch.where(w, c, 0.0) for w in (zer, sat, dn, up, ex)] + [-ent]
    return torch.stack([a.sum((1, 2)) for a in part], 1)


def _exact_sse(x, axis):
    """[BH, 41] squared error sums of bf16 x [B, H, N, d]: a block takes one of three exponents."""
    rows = []
    thr = torch.tensor(SWEEP, dtype=torch.float64, device="cuda")
    for h in x.reshape(-1, x.shape[2], D):
        h = h.double()
        y = (h if axis == mxattn.AXIS_HEAD_DIM else _pad_to(h, 0, 32).t()).reshape(-1, 32)
        f, e = torch.frexp(y.abs().amax(-1))
        sse = []
        for k in (2, 3, 4):
            s = torch.exp2((e - k).clamp(-127, 127).double())[:, None]
            sse.append((y - torch.sign(y) * _e2m1(y.abs() / s) * s).square().sum(-1))
        f = f * 8  # block maximum over 2^(e - 3), in [4, 8)
        out = []
        for q in thr:
            pick = torch.where(f > q, sse[0], torch.where(2 * f <= q, sse[2], sse[1]))
            out.append(pick.sum())
        rows.append(torch.stack(out))
    return torch.stack(rows)


def exact(case, seed):
    op, mode = case["op"], case["mode"]
    if op == "quantize":
        return None  # codes, compared bit for bit
    B, H, Nq, Nkv = case["B"], case["H"], case["Nq"], case["Nkv"]
    if B * H * case.get("rows", Nq) * Nkv > 45e9:
        return None  # over 20 seconds
    q, k, v = _inputs(case, seed)
    if op == "sweep":
        return _exact_sse(k, mxattn.AXIS_HEAD_DIM), _exact_sse(v, mxattn.AXIS_TOKENS)
    flat = lambda t: t.reshape(-1, t.shape[-2], D)  # noqa: E731
    if op in ("forward", "cross", "step"):
        o = [_exact_head(a, b, c, mode, Nkv) for a, b, c in zip(flat(q), flat(k), flat(v))]
        return torch.stack(o).view(B, H, Nq, D)
    row0 = Nq - case["rows"] if op == "rows" else 0
    ps, sts = [], []
    for a, b in zip(flat(q), flat(k)):
        kd = b.double().t().contiguous()
        step = max(1, (1 << 25) // Nkv)
        for r in range(row0, Nq, step):
            p = torch.softmax(a[r:min(Nq, r + step)].double() @ kd / math.sqrt(D), -1)
            # the statistics are those of 32-bit probabilities (a row's peak may be 1)
            sts.append(_exact_stats(p.float().double(), mode, case["gamma"]))
            if op == "rows":
                ps.append(_pad_to(p, 1, 4))
    st = torch.cat(sts)
    if op == "diag":
        return st.view(B, H, Nq, 8)
    return torch.cat(ps).view(B, H, case["rows"], -1), st
