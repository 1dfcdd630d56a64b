"""What a training or scoring program has this library do, as cases that can be timed and checked.

A case is one pass of one attention layer (or of the layout kernels around it) through the public entry points, the way
``runner.layer_step`` issues them:

* ``layer``    forward of Call 1 and Call 2, then both backward calls: a policy-update micro-batch;
* ``forward``  both forward calls only: scoring log-probabilities under the old or the reference policy;
* ``groups``   the same layer for several prompt groups in one call (the ``*_groups`` entry points);
* ``pack``     the layout kernels: standard packing <-> single-prompt packing of token ids and hidden rows, label map.

Sizes are those of this repository's configurations (``workloads.CONFIGS``) and of the paper's tables, plus generic ones.
"""
import math

import numpy as np
import torch

from paper_2605_15422_amd import accounting, binding as B, runner


def _case(name, kind, N, P, lo, hi, H, Hk, d, window=0, joint=True, packed=True, groups=1, lens_seed=1):
    return dict(name=name, kind=kind, N=N, P=P, lo=lo, hi=hi, H=H, Hk=Hk, d=d, window=window, joint=joint, packed=packed,
                groups=groups, lens_seed=lens_seed)


def listed():
    return [
        # the smallest configuration of the repository: a smoke-sized layer, where latency and launches count
        _case("tiny_d64", "layer", 4, 256, 128, 128, 4, 2, 64, packed=False),
        # short prompts and short answers (grade-school arithmetic: P about 1K, R up to 256, N = 8), gradients of the two
        # calls left as two bf16 terms, as the paper's interface returns them
        _case("short_d128", "layer", 8, 1021, 65, 256, 32, 8, 128, joint=False, lens_seed=2),
        # a micro-batch of eight such groups of unequal size in one call
        _case("groups_d128", "groups", 8, 517, 17, 256, 32, 8, 128, groups=8, lens_seed=3),
        # head dim 64: a mid-size policy-update micro-batch with ragged responses
        _case("layer_d64", "layer", 8, 4096, 131, 2048, 32, 8, 64, lens_seed=4),
        # head dim 96, odd prompt length
        _case("layer_d96", "layer", 8, 4111, 131, 2048, 16, 4, 96, lens_seed=5),
        # the headline configuration: Qwen3-8B attention dimensions, equal responses, full tiles
        _case("layer_d128", "layer", 16, 8192, 1024, 1024, 32, 8, 128, packed=False),
        # the same dimensions with few, short, ragged responses behind a prompt of odd length (the smallest point of the
        # paper's single-layer grid): too few row blocks to fill the chip evenly
        _case("ragged_d128", "layer", 4, 5059, 131, 2048, 32, 8, 128, lens_seed=6),
        # forward only over a long prompt, eight query heads per KV head: scoring a batch of long-context answers
        _case("score_d128", "forward", 16, 32768, 1024, 2048, 32, 4, 128, lens_seed=7),
        # head dim 192
        _case("layer_d192", "layer", 8, 4096, 131, 2048, 12, 4, 192, lens_seed=8),
        # one rank's share of a long-context sliding-window layer, head dim 256
        _case("swa_d256", "layer", 8, 57344, 8192, 8192, 8, 2, 256, window=1024, packed=False),
        # one rank's share of a global layer, head dim 512 (the repository's configuration at a quarter of its lengths)
        _case("global_d512", "layer", 8, 14336, 1025, 2048, 8, 2, 512, lens_seed=9),
        # layout kernels on the headline packing: 4-byte token ids and 8 KB hidden rows, both directions, label map
        _case("pack_rows", "pack", 16, 8192, 1024, 1024, 32, 8, 128, packed=False),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


#: the most algorithmic work of a drawn case (the headline layer's); the slowest head dims of it stay under 40 ms
DRAW_FLOPS = 1.0e13


def draw(rng):
    kind = rng.choice(["layer"] * 6 + ["forward"] * 2 + ["groups"] * 2 + ["pack"])
    d = rng.choice([64, 96, 128, 128, 128, 192, 256, 512])
    H, Hk = rng.choice([(4, 2), (8, 2), (8, 8), (12, 4), (16, 4), (32, 8), (32, 4)])
    window = _log_int(rng, 64, 4096) if d <= 256 and rng.random() < 0.25 else 0
    N = _log_int(rng, 1, 32)
    P = 0 if kind in ("layer", "forward") and rng.random() < 0.1 else _log_int(rng, 16, 65536)
    hi = _log_int(rng, 16, 8192)
    lo = rng.randint(1, hi)
    groups = 1
    if kind == "groups":
        groups = rng.randint(2, 8)
        P, hi = min(P, 2048), min(hi, 512)
        lo = min(lo, hi)
    c = dict(kind=kind, N=N, P=P, lo=lo, hi=hi, H=H, Hk=Hk, d=d, window=window, joint=rng.random() < 0.7,
             packed=rng.random() < 0.6, groups=groups, lens_seed=rng.randint(1, 10**6))
    while work(c)["flops"] > DRAW_FLOPS or (kind == "pack" and work(c)["bytes"] > 2.5e9):
        c["P"] = c["P"] * 7 // 10
        c["hi"] = max(c["lo"], c["hi"] * 8 // 10)
        c["lo"] = max(1, c["lo"] * 8 // 10)
    return c


# ---- lengths: a function of the case alone ------------------------------------------------------------------------
def _lens(c):
    """Per group (P_g, response lengths).  The first group has the case's own prompt length, later ones shorter ones."""
    r = np.random.default_rng(c["lens_seed"])
    out = []
    for g in range(c["groups"]):
        P = c["P"] if g == 0 else int(r.integers(max(1, c["P"] // 4), c["P"], endpoint=True))
        N = c["N"] if g == 0 else int(r.integers(max(1, c["N"] // 2), c["N"], endpoint=True))
        out.append((P, r.integers(c["lo"], c["hi"], endpoint=True, size=N).astype(np.int64)))
    return out


def work(c):
    groups, d, H, Hk = _lens(c), c["d"], c["H"], c["Hk"]
    P, T = sum(g[0] for g in groups), sum(int(g[1].sum()) for g in groups)
    rows = P + T
    if c["kind"] == "pack":
        N = c["N"]
        long_rows, row = N * P + T, 4 + 2 * H * d
        # standard -> packed: the packed rows read and written; packed -> standard: read once, written N times; positions
        # of both layouts and the label map written
        return dict(bytes=rows * row * 2 + (rows + long_rows) * row + 4 * (rows + long_rows) + 4 * (rows + N), flops=0)
    pairs = sum(accounting.pairs_call1(p, c["window"]) + accounting.pairs_call2(p, lens, c["window"]) for p, lens in groups)
    q, kv, lse = 2 * H * d * rows, 2 * Hk * d * rows, 4 * H * rows
    if c["kind"] == "forward":
        return dict(bytes=2 * q + 2 * kv + lse, flops=4 * d * pairs * H)
    # q, k, v, dO read; O, LSE, dQ, dK, dV written (the backward's re-reads of O are of the pass's own making)
    bytes_ = 4 * q + 4 * kv + lse
    if not c["joint"]:
        bytes_ += 2 * 2 * Hk * d * P   # the prompt's dK and dV as two terms
    return dict(bytes=bytes_, flops=14 * d * pairs * H)


def tolerance(c):
    if c["kind"] == "pack":
        return "exact"
    # bf16 operands and results: every output is 1.7e-3 to 3.1e-3 (2-norm) from 64-bit arithmetic.  The largest single
    # difference, up to 0.2 of a tensor's root mean square, sits in the first prompt rows, whose few keys give values far
    # above that mean (dQ there carries the rounding of O in D = rowsum(dO * O)).
    return {"rel": 0.01, "max": 0.8}


# ---- inputs -------------------------------------------------------------------------------------------------------
def _normal(gen, *shape):
    """N(0, 1) in bf16, drawn in row chunks so that the fp32 staging copy stays small."""
    out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    flat = out.view(-1)
    step = 1 << 26
    for s in range(0, flat.numel(), step):
        n = min(step, flat.numel() - s)
        flat[s:s + n].copy_(torch.randn(n, generator=gen, device="cuda"))
    return out


def _inputs(c, seed):
    """Packed (P + T)-row tensors q, k, v, dO: prompts of all groups first, then all responses.  `packed`: q, k and v are
    views of one fused projection output (rows, H + 2 H_k, d)."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    groups, d, H, Hk = _lens(c), c["d"], c["H"], c["Hk"]
    rows = sum(g[0] for g in groups) + sum(int(g[1].sum()) for g in groups)
    qkv = _normal(gen, rows, H + 2 * Hk, d)
    q, k, v = qkv[:, :H], qkv[:, H:H + Hk], qkv[:, H + Hk:]
    if not c["packed"]:
        q, k, v = q.contiguous(), k.contiguous(), v.contiguous()
    return q, k, v, _normal(gen, rows, H, d)


def _cu(lens):
    cu = np.zeros(len(lens) + 1, dtype=np.int32)
    cu[1:] = np.cumsum(lens)
    return cu


class _State:
    pass


def prepare(c, seed):
    s = _State()
    s.case = c
    groups, d, H, Hk = _lens(c), c["d"], c["H"], c["Hk"]
    P = sum(g[0] for g in groups)
    lens = np.concatenate([g[1] for g in groups])
    cu = _cu(lens)
    T = int(cu[-1])
    if c["kind"] == "pack":
        gen = torch.Generator(device="cuda").manual_seed(int(seed))
        N = c["N"]
        s.P, s.T, s.N, s.cu = P, T, N, torch.from_numpy(cu).cuda()
        s.ids = torch.randint(0, 150000, (N * P + T,), generator=gen, device="cuda", dtype=torch.int32)
        s.hidden = _normal(gen, P + T, H * d)
        s.ids_packed = torch.empty(P + T, dtype=torch.int32, device="cuda")
        s.hidden_long = torch.empty((N * P + T, H * d), dtype=torch.bfloat16, device="cuda")
        s.hidden_back = torch.empty_like(s.hidden)
        s.pos = torch.empty(P + T, dtype=torch.int32, device="cuda")
        s.pos_long = torch.empty(N * P + T, dtype=torch.int32, device="cuda")
        s.next = torch.empty(P + T, dtype=torch.int32, device="cuda")
        s.first = torch.empty(N, dtype=torch.int32, device="cuda")
        s.ids_long = torch.empty(N * P + T, dtype=torch.int32, device="cuda")
        return s
    q, k, v, do = _inputs(c, seed)
    flags = B.FLAG_ACCUM_CTX_F32 if c["joint"] else 0
    s.shape = B.make_shape(len(lens), max(g[0] for g in groups), T, int(lens.max()), H, Hk, d, c["window"], 0.0, flags)
    s.dg = B.DeviceGroup(s.shape, q[:P], k[:P], v[:P], q[P:], k[P:], v[P:], do[:P], do[P:], torch.from_numpy(cu).cuda(), cu)
    if c["kind"] != "groups":
        s.b = runner.alloc(s.dg, poison=False)
        return s
    table, off, seq = [], 0, 0
    for p, ls in groups:
        table.append((off, p, seq, seq + len(ls)))
        off += p
        seq += len(ls)
    s.P, s.table = P, np.asarray(table, dtype=np.int32)
    s.table_dev = torch.from_numpy(s.table).cuda()
    s.shape_all = B.make_shape(1, P, 0, 0, H, Hk, d, c["window"], 0.0, flags)
    s.ws = {op: torch.empty(max(16, B.dualkv_groups_workspace_bytes(s.shape, len(groups), P, op)), dtype=torch.uint8, device="cuda")
            for op in (B.OP_CTX_FWD, B.OP_FWD, B.OP_CTX_BWD, B.OP_BWD)}

    def like(x, dtype=torch.bfloat16):
        return torch.empty(x.shape, dtype=dtype, device="cuda")

    g = s.dg
    s.o_c, s.o_d, s.dq_c, s.dq_d = like(g.q_c), like(g.q_d), like(g.q_c), like(g.q_d)
    s.dk_d, s.dv_d, s.dk_c, s.dv_c, s.dk_c1, s.dv_c1 = (like(x) for x in (g.k_d, g.v_d, g.k_c, g.v_c, g.k_c, g.v_c))
    s.acc_k, s.acc_v = (like(g.k_c, torch.float32) for _ in range(2)) if c["joint"] else (None, None)
    s.lse_c = torch.empty((H, P), dtype=torch.float32, device="cuda")
    s.lse_d = torch.empty((H, T), dtype=torch.float32, device="cuda")
    return s


def run(s):
    c = s.case
    if c["kind"] == "pack":
        n, row = 2 * c["H"] * c["d"], (s.N, s.P, s.T, s.cu)
        B.dualkv_repack(*row, 4, s.ids, s.ids_packed, s.pos)
        B.dualkv_replicate(*row, 4, s.ids_packed, s.ids_long, s.pos_long)
        B.dualkv_replicate(*row, n, s.hidden, s.hidden_long)
        B.dualkv_repack(*row, n, s.hidden_long, s.hidden_back)
        B.dualkv_label_map(s.N, s.P, s.T, s.cu, s.next, s.first)
        return dict(ids=s.ids_packed, ids_long=s.ids_long, hidden=s.hidden_back, hidden_long=s.hidden_long, pos=s.pos, pos_long=s.pos_long,
                    next=s.next, first=s.first)
    if c["kind"] == "forward":
        runner.forward(s.dg, s.b)
        return dict(o_c=s.b.o_c, lse_c=s.b.lse_c, o_d=s.b.o_d, lse_d=s.b.lse_d)
    if c["kind"] == "layer":
        runner.layer_step(s.dg, s.b)
        b = s.b
        out = dict(o_c=b.o_c, lse_c=b.lse_c, o_d=b.o_d, lse_d=b.lse_d, dq_c=b.dq_c, dq_d=b.dq_d, dk_d=b.dk_d, dv_d=b.dv_d)
        if c["joint"]:
            out.update(dk_c=b.dk_c, dv_c=b.dv_c)
        else:
            out.update(dk_c1=b.dk_c1, dv_c1=b.dv_c1, dk_c2=b.dk_c2, dv_c2=b.dv_c2)
        return out
    g, joint, tab = s.dg, c["joint"], (s.shape, s.table_dev, s.table, s.P)
    B.dualkv_ctx_fwd_groups(*tab, g.q_c, g.k_c, g.v_c, s.o_c, s.lse_c, s.ws[B.OP_CTX_FWD])
    B.dualkv_fwd_groups(*tab, g.q_d, g.k_c, g.v_c, g.k_d, g.v_d, g.cu_dev, g.cu_host, s.o_d, s.lse_d, s.ws[B.OP_FWD])
    if joint:
        B.dualkv_zero_ctx_grads(s.shape_all, s.acc_k, s.acc_v)
    B.dualkv_bwd_groups(*tab, g.do_d, s.o_d, s.lse_d, g.q_d, g.k_c, g.v_c, g.k_d, g.v_d, g.cu_dev, g.cu_host, s.dq_d,
                        None if joint else s.dk_c, None if joint else s.dv_c, s.dk_d, s.dv_d, s.acc_k, s.acc_v, s.ws[B.OP_BWD])
    B.dualkv_ctx_bwd_groups(*tab, g.do_c, s.o_c, s.lse_c, g.q_c, g.k_c, g.v_c, s.dq_c, None if joint else s.dk_c1,
                            None if joint else s.dv_c1, s.acc_k, s.acc_v, s.ws[B.OP_CTX_BWD])
    out = dict(o_c=s.o_c, lse_c=s.lse_c, o_d=s.o_d, lse_d=s.lse_d, dq_c=s.dq_c, dq_d=s.dq_d, dk_d=s.dk_d, dv_d=s.dv_d)
    if joint:
        B.dualkv_finalize_ctx_grads(s.shape_all, s.acc_k, s.acc_v, s.dk_c, s.dv_c)
        out.update(dk_c=s.dk_c, dv_c=s.dv_c)
    else:
        out.update(dk_c1=s.dk_c1, dv_c1=s.dv_c1, dk_c2=s.dk_c, dv_c2=s.dv_c)
    return out


# ---- 64-bit evaluation --------------------------------------------------------------------------------------------
def _attend(q, k, v, do, first, window, out, rows, dk, dv):
    """Causal attention of the rows of q (n, G, d), at positions first, first + 1, ..., over the keys k, v (m, d) at
    positions 0 ... m - 1, in 64 bits.  Writes O, LSE and dQ at `rows` of `out`; adds to dk, dv (m, d)."""
    n, G, d = q.shape
    scale = 1.0 / math.sqrt(d)
    chunk = max(32, min(2048, (1 << 26) // max(1, G * k.shape[0])))
    for r0 in range(0, n, chunk):
        r1 = min(n, r0 + chunk)
        k0 = max(0, first + r0 - window + 1) if window else 0
        k1 = first + r1
        qq, kk, vv = q[r0:r1].reshape(-1, d), k[k0:k1], v[k0:k1]
        pos = (first + torch.arange(r0, r1, device="cuda")).repeat_interleave(G)[:, None]
        key = torch.arange(k0, k1, device="cuda")[None, :]
        s = (qq @ kk.t()).mul_(scale)
        hidden = key > pos
        if window:
            hidden |= key <= pos - window
        s.masked_fill_(hidden, -math.inf)
        del hidden
        lse = torch.logsumexp(s, dim=1)
        p = s.sub_(lse[:, None]).exp_()
        o = p @ vv
        at = slice(rows + r0, rows + r1)
        out["o"][at] = o.view(r1 - r0, G, d)
        out["lse"][:, at] = lse.view(r1 - r0, G).t()
        if do is None:
            continue
        g = do[r0:r1].reshape(-1, d)
        dv[k0:k1] += p.t() @ g
        ds = (g @ vv.t()).sub_((g * o).sum(dim=1, keepdim=True)).mul_(p).mul_(scale)
        out["dq"][at] = (ds @ kk).view(r1 - r0, G, d)
        dk[k0:k1] += ds.t() @ qq


def exact(c, seed):
    if c["kind"] == "pack":
        return None   # copies
    q, k, v, do = _inputs(c, seed)
    groups, d, H, Hk, W = _lens(c), c["d"], c["H"], c["Hk"], c["window"]
    G, back = H // Hk, c["kind"] != "forward"
    total_P = sum(g[0] for g in groups)
    n = q.shape[0]
    empty = lambda *shape: torch.empty(shape, dtype=torch.float64, device="cuda")   # noqa: E731
    o, lse = empty(n, H, d), empty(H, n)
    dq = empty(n, H, d) if back else None
    dk, dv = (torch.zeros((n, Hk, d), dtype=torch.float64, device="cuda") for _ in range(2))
    dk2, dv2 = (torch.zeros((total_P, Hk, d), dtype=torch.float64, device="cuda") for _ in range(2))   # Call 2's prompt terms
    for hk in range(Hk):
        hs = slice(hk * G, (hk + 1) * G)
        out = dict(o=o[:, hs], lse=lse[hs], dq=dq[:, hs] if back else None)
        Q, K, V = q[:, hs].double(), k[:, hk].double(), v[:, hk].double()
        DO = do[:, hs].double() if back else None
        at_p, at_r = 0, total_P
        for P, lens in groups:
            p = slice(at_p, at_p + P)
            if P:
                _attend(Q[p], K[p], V[p], DO[p] if back else None, 0, W, out, at_p, dk[p, hk], dv[p, hk])
            for R in (int(x) for x in lens):
                r = slice(at_r, at_r + R)
                keys, values = torch.cat([K[p], K[r]]), torch.cat([V[p], V[r]])
                gk, gv = torch.zeros_like(keys), torch.zeros_like(values)
                _attend(Q[r], keys, values, DO[r] if back else None, P, W, out, at_r, gk, gv)
                dk2[p, hk] += gk[:P]
                dv2[p, hk] += gv[:P]
                dk[r, hk] += gk[P:]
                dv[r, hk] += gv[P:]
                at_r += R
            at_p += P
    P = total_P
    got = dict(o_c=o[:P], lse_c=lse[:, :P], o_d=o[P:], lse_d=lse[:, P:])
    if back:
        got.update(dq_c=dq[:P], dq_d=dq[P:], dk_d=dk[P:], dv_d=dv[P:])
        if c["joint"]:
            got.update(dk_c=dk[:P] + dk2, dv_c=dv[:P] + dv2)
        else:
            got.update(dk_c1=dk[:P], dv_c1=dv[:P], dk_c2=dk2, dv_c2=dv2)
    return got
