"""Performance cases of the framework: what a serving program has it do, through its public entry points.

A verification layer calls ssv_nsa_verify once per layer and step: in refresh mode it builds the selected-block indices,
in reuse mode it takes those of an earlier layer or step, and SSV_REFRESH_SHARED is the approximate variant in between.
Around it, ssv_nsa_compress builds the compressed cache after a prefill and extends it after a verification round.  The
sizes are the benchmark's configurations (NSA-27B-style layer: 64 query / 4 KV heads, d_k = 192, d_v = 128; l = 32,
d = 16, l' = 64, n = 16, w = 512), the paper's kernel workload (32 / 8 heads of dimension 64) and shapes between them.

Each case is measured on inputs made here on the GPU from a seed: K, V ~ N(0, 1) (a share of the key positions scaled
where the case says so), verifier queries with correlation rho to a direction shared by the sequence, gates ~ U(0, 1),
compressed rows = means over complete windows of committed tokens.
"""
import math

import torch

from paper_2605_19893_amd import binding as B

L_CMP, STRIDE, L_SEL, N_SEL, WINDOW, N_INIT, N_LOCAL = 32, 16, 64, 16, 512, 1, 2
MODES = {"refresh": B.SSV_REFRESH, "reuse": B.SSV_REUSE, "shared": B.SSV_REFRESH_SHARED}
FANOUTS = {"tree40": (4, 3, 2), "tree21": (3, 2, 2), "tree6": (2, 2)}


def _verify(name, *, batch, queries, ctx, mode, ctx_min=0, heads=64, kv_heads=4, d_k=192, d_v=128, dtype="bf16",
            drafts="chain", rho=0.7, heavy=0.0, grain=64, ragged=False, n_sel=N_SEL, window=WINDOW):
    """ctx: committed tokens of the longest sequence; ctx_min > 0: lengths log-uniform in [ctx_min, ctx], multiples of
    grain; ragged: some sequences bring fewer queries than the batch's capacity."""
    case = {"op": "verify", "batch": batch, "queries": queries, "ctx_min": ctx_min or ctx, "ctx": ctx, "mode": mode, "heads": heads,
            "kv_heads": kv_heads, "d_k": d_k, "d_v": d_v, "dtype": dtype, "drafts": drafts, "rho": rho, "heavy": heavy,
            "grain": grain, "ragged": ragged, "n_sel": n_sel, "window": window}
    return {"name": name, **case} if name else case


def _compress(name, *, batch, ctx, new, ctx_min=0, kv_heads=4, d_k=192, d_v=128, dtype="bf16", grain=64):
    """new: tokens committed per sequence since the last update, at most; 0: the cache is built from scratch."""
    case = {"op": "compress", "batch": batch, "ctx_min": ctx_min or ctx, "ctx": ctx, "new": new, "kv_heads": kv_heads, "d_k": d_k,
            "d_v": d_v, "dtype": dtype, "grain": grain}
    return {"name": name, **case} if name else case


def listed():
    return [
        # the smallest call: a draft chain of four over a 2K context of a small fp32 model; launches and latency
        _verify("tiny_f32", batch=1, queries=4, ctx=2048, mode="refresh", heads=4, kv_heads=1, d_k=64, d_v=64, dtype="f32",
                rho=0.0, n_sel=4, window=128),
        # one user at a 32K context, a chain of eight: the interactive case, bound by latency
        _verify("chain8_32k", batch=1, queries=8, ctx=32768, mode="refresh", rho=0.5),
        # the same on the indices of an earlier layer
        _verify("chain8_32k_reuse", batch=1, queries=8, ctx=32768, mode="reuse", rho=0.5),
        # a batch of sixteen at 64K with short chains and concentrated importance: bound by memory bandwidth
        _verify("batch16_64k", batch=16, queries=4, ctx=65536, mode="refresh", heavy=0.05),
        _verify("batch16_64k_reuse", batch=16, queries=4, ctx=65536, mode="reuse", heavy=0.05),
        # draft trees of forty nodes over 128K contexts: bound by arithmetic
        _verify("tree40_128k", batch=4, queries=40, ctx=131072, mode="refresh", drafts="tree40"),
        # a serving batch of mixed lengths with chains of sixteen, refreshing and reusing
        _verify("mixed32", batch=32, queries=16, ctx_min=4096, ctx=131072, mode="refresh"),
        _verify("mixed32_reuse", batch=32, queries=16, ctx_min=4096, ctx=131072, mode="reuse"),
        # the paper's kernel workload: 32 / 8 heads of dimension 64, a long chain, batch 1
        _verify("heads64_chain64", batch=1, queries=64, ctx=65536, mode="refresh", heads=32, kv_heads=8, d_k=64, d_v=64, rho=0.0),
        # odd lengths, sequences that bring fewer queries, eight heads per group of dimension 128
        _verify("ragged_d128", batch=5, queries=7, ctx_min=3001, ctx=40009, mode="refresh", heads=32, kv_heads=4, d_k=128, d_v=128,
                grain=1, ragged=True),
        # the compressed cache of a batch after its prefill
        _compress("compress_build", batch=16, ctx=65536, new=0),
        # the compressed cache after a verification round that accepted up to sixteen tokens per sequence
        _compress("compress_update", batch=32, ctx_min=4096, ctx=131072, new=16),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _seconds(case):
    """A rough time of one pass, to keep drawn cases within the listed ones."""
    w = work(case)
    return w["bytes"] / 4e12 + w["flops"] / (0.5e15 if case["dtype"] == "bf16" else 0.03e15)


def draw(rng):
    """One more case of the same ranges: every supported head shape, chains of 1 to 64 and the draft trees, contexts
    of 1K to 128K of equal and of mixed lengths, all modes, and both uses of the compression kernel."""
    limit = 0.9 * max(_seconds(c) for c in listed() if c["op"] == "verify")
    bytes_limit = 11e9
    ctx = _log_uniform(rng, 1024, 131072)
    batch = _log_uniform(rng, 1, 32)
    mixed = batch > 1 and rng.random() < 0.5
    ctx_min = max(256, ctx // rng.choice([2, 8, 32])) if mixed else 0
    grain = rng.choice([1, 64])
    ctx = max(64, ctx // grain * grain)
    shape = rng.choices([("bf16", 192, 128, 64, 4), ("bf16", 192, 128, 16, 1), ("bf16", 128, 128, 32, 4), ("bf16", 128, 128, 16, 8),
                         ("bf16", 64, 64, 32, 8), ("f32", 64, 64, 8, 2)], [6, 2, 3, 1, 3, 2])[0]
    dtype, d_k, d_v, heads, kv_heads = shape
    if rng.random() < 0.2:
        make = lambda b: _compress(None, batch=b, ctx_min=ctx_min, ctx=ctx, new=rng.choice([0, 16, 512]), kv_heads=kv_heads, d_k=d_k,
                                   d_v=d_v, dtype=dtype, grain=grain)
    else:
        drafts, queries = "chain", _log_uniform(rng, 1, 64)
        if rng.random() < 0.3:
            drafts = rng.choice(sorted(FANOUTS))
            queries = len(_tree(drafts)[0])
        mode = rng.choices(["refresh", "reuse", "shared"], [6, 3, 1])[0]
        rho, heavy, ragged = rng.choice([0.0, 0.5, 0.7, 0.9]), rng.choice([0.0, 0.0, 0.05]), rng.random() < 0.3
        make = lambda b: _verify(None, batch=b, queries=queries, ctx_min=ctx_min, ctx=ctx, mode=mode, heads=heads, kv_heads=kv_heads,
                                 d_k=d_k, d_v=d_v, dtype=dtype, drafts=drafts, rho=rho, heavy=heavy, grain=grain, ragged=ragged)
    case = make(batch)
    while case["batch"] > 1 and (_seconds(case) > limit or _cache_bytes(case) > bytes_limit):
        case = {**case, "batch": case["batch"] - 1}
    while _seconds(case) > limit:
        case = {**case, "queries": max(1, case["queries"] // 2), "drafts": "chain"}
    return case


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _elem(case):
    return 2 if case["dtype"] == "bf16" else 4


def _cache_bytes(case):
    return case["batch"] * case["kv_heads"] * case["ctx"] * (case["d_k"] + case["d_v"]) * _elem(case)


def _tree(kind):
    """(parents, depths) of a uniform draft tree, breadth first."""
    parents, depths, level = [], [], [-1]
    for depth, fan in enumerate(FANOUTS[kind]):
        nxt = []
        for p in level:
            for _ in range(fan):
                parents.append(p)
                depths.append(depth)
                nxt.append(len(parents) - 1)
        level = nxt
    return parents, depths


def _lengths(case):
    """Committed lengths: equal, or one of every quantile of the log-uniform range (the order is the seed's)."""
    n, lo, hi, grain = case["batch"], case["ctx_min"], case["ctx"], case["grain"]
    if lo >= hi:
        return [hi] * n
    out = []
    for b in range(n):
        x = lo * (hi / lo) ** ((b + 0.5) / n)
        out.append(min(hi, max(1, int(x / grain + 0.5)) * grain))
    return out


def _cmp_rows(length):
    return 0 if length < L_CMP else (length - L_CMP) // STRIDE + 1


def _pooled(x, lens, rows_cap):
    """Means over windows of L_CMP rows every STRIDE rows, over the committed rows of every sequence."""
    out = torch.zeros((x.shape[0], x.shape[1], rows_cap, x.shape[3]), dtype=x.dtype, device=x.device)
    per = L_CMP // STRIDE
    for b, length in enumerate(lens):
        nc = _cmp_rows(length)
        if nc <= 0:
            continue
        chunks = nc + per - 1
        s = x[b, :, :chunks * STRIDE].reshape(x.shape[1], chunks, STRIDE, x.shape[3]).sum(2, dtype=torch.float32)
        acc = s[:, :nc].clone()
        for m in range(1, per):
            acc += s[:, m:m + nc]
        out[b, :, :nc] = acc / L_CMP
    return out


def _index_sets(case, lens, g):
    """Valid index sets as an earlier refresh call leaves them: forced blocks, then the best by a score that is correlated
    between the queries of a sequence as its queries are; ascending, -1 padded."""
    n, t, hk, ns = case["batch"], case["queries"], case["kv_heads"], case["n_sel"]
    dev = torch.device("cuda")
    length = torch.tensor(lens, device=dev).view(n, 1, 1, 1)
    own = (length + torch.arange(t, device=dev).view(1, t, 1, 1)) // L_SEL
    nblk = (max(lens) + t) // L_SEL + 1
    blk = torch.arange(nblk, device=dev).view(1, 1, 1, nblk)
    rho = case["rho"]
    score = math.sqrt(rho) * torch.randn((n, 1, hk, nblk), generator=g, device=dev) + \
        math.sqrt(1.0 - rho) * torch.randn((n, t, hk, nblk), generator=g, device=dev)
    score = torch.where((blk < N_INIT) | (blk > own - N_LOCAL), torch.full_like(score, 1e9), score)
    score = torch.where(blk > own, torch.full_like(score, -math.inf), score)
    top, idx = score.topk(min(ns, nblk), dim=-1)
    idx = torch.where(torch.isinf(top), torch.full_like(idx, 1 << 30), idx).sort(dim=-1).values
    idx = torch.where(idx == 1 << 30, torch.full_like(idx, -1), idx).int()
    if nblk < ns:
        idx = torch.cat([idx, torch.full((n, t, hk, ns - nblk), -1, dtype=torch.int32, device=dev)], dim=-1)
    return idx.contiguous()


def prepare(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    host = torch.Generator()
    host.manual_seed(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    n, hk, d_k, d_v = case["batch"], case["kv_heads"], case["d_k"], case["d_v"]
    order = torch.randperm(n, generator=host).tolist()
    lens = _lengths(case)
    lens = [lens[i] for i in order]
    t = case.get("queries", 0)
    rows = -(-(max(lens) + t) // L_SEL) * L_SEL
    k = torch.randn((n, hk, rows, d_k), generator=g, device=dev, dtype=dt)
    v = torch.randn((n, hk, rows, d_v), generator=g, device=dev, dtype=dt)
    cap = max(1, _cmp_rows(max(lens) + t))
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=dev)

    if case["op"] == "compress":
        new = case["new"]
        before = None
        max_new = cap
        if new:
            took = torch.randint(0, new + 1, (n,), generator=host).tolist()
            before = [max(0, length - a) for length, a in zip(lens, took)]
            max_new = max(1, max(_cmp_rows(length) - _cmp_rows(b) for length, b in zip(lens, before)))
        kc = torch.zeros((n, hk, cap, d_k), dtype=dt, device=dev)
        vc = torch.zeros((n, hk, cap, d_v), dtype=dt, device=dev)
        p = B.make_cmp_params(B=n, H_kv=hk, d_k=d_k, d_v=d_v, l=L_CMP, d=STRIDE, dtype=B.SSV_BF16 if dt == torch.bfloat16 else B.SSV_F32,
                              max_new_rows=max_new, kv_capacity=rows, cmp_capacity=cap, k_stride=k.stride()[:3], v_stride=v.stride()[:3],
                              kc_stride=kc.stride()[:3], vc_stride=vc.stride()[:3])
        return {"op": "compress", "k": k, "v": v, "k_cmp": kc, "v_cmp": vc, "before": None if before is None else i32(before),
                "after": i32(lens), "n_cmp": torch.zeros(n, dtype=torch.int32, device=dev), "params": p}

    if case["heavy"]:
        scale = torch.where(torch.rand((n, 1, rows, 1), generator=g, device=dev) < case["heavy"], 4.0, 1.0).to(dt)
        k.mul_(scale)
    k_cmp, v_cmp = _pooled(k, lens, cap), _pooled(v, lens, cap)
    h, rho = case["heads"], case["rho"]
    q = math.sqrt(rho) * torch.randn((n, 1, h, d_k), generator=g, device=dev) + \
        math.sqrt(1.0 - rho) * torch.randn((n, t, h, d_k), generator=g, device=dev)
    q = q.to(dt).contiguous()
    gates = torch.rand((n, t, h, 3), generator=g, device=dev)
    n_query = [t] * n
    if case["ragged"]:
        n_query = [max(1, t - int(x)) for x in torch.randint(0, max(1, t // 2) + 1, (n,), generator=host)]
    parents = None
    if case["drafts"] != "chain":
        parents = i32([_tree(case["drafts"])[0]] * n)
    out = torch.zeros((n, t, h, d_v), dtype=dt, device=dev)
    mode = MODES[case["mode"]]
    sel = _index_sets(case, lens, g) if mode == B.SSV_REUSE else torch.full((n, t, hk, case["n_sel"]), -1, dtype=torch.int32, device=dev)
    p = B.make_params(B=n, T=t, H=h, H_kv=hk, d_k=d_k, d_v=d_v, l=L_CMP, d=STRIDE, l_sel=L_SEL, n_sel=case["n_sel"], w=case["window"],
                      n_init=N_INIT, n_local=N_LOCAL, dtype=B.SSV_BF16 if dt == torch.bfloat16 else B.SSV_F32, mode=mode,
                      max_seq_len=max(lens), max_n_cmp=max(1, _cmp_rows(max(lens))), avg_seq_len=sum(lens) // n,
                      k_stride=k.stride()[:3], v_stride=v.stride()[:3], kc_stride=k_cmp.stride()[:3], vc_stride=v_cmp.stride()[:3])
    nbytes = B.ssv_nsa_workspace_bytes(p)
    return {"op": "verify", "q": q, "k": k, "v": v, "k_cmp": k_cmp, "v_cmp": v_cmp, "gates": gates, "seq_lens": i32(lens),
            "n_cmp": i32([_cmp_rows(x) for x in lens]), "n_query": i32(n_query), "parents": parents, "params": p, "out": out, "sel_idx": sel,
            "workspace": torch.empty(nbytes, dtype=torch.uint8, device=dev), "workspace_bytes": nbytes}


def run(state):
    s = state
    stream = torch.cuda.current_stream().cuda_stream
    if s["op"] == "compress":
        B.ssv_nsa_compress(s["k"], s["v"], s["k_cmp"], s["v_cmp"], s["before"], s["after"], s["n_cmp"], s["params"], stream)
        return s["k_cmp"], s["v_cmp"], s["n_cmp"]
    B.ssv_nsa_verify(s["q"], s["k"], s["v"], s["k_cmp"], s["v_cmp"], s["gates"], s["seq_lens"], s["n_cmp"], s["n_query"], s["parents"],
                     s["params"], s["out"], s["sel_idx"], s["workspace"], s["workspace_bytes"], stream)
    return s["out"], s["sel_idx"]


def work(case):
    """Bytes: compressed rows once per KV head; the window and the distinct selected blocks of a sequence once per KV head
    (expected number: queries correlated by rho share about 0.6 rho^2 of their free blocks with those before them, the
    others fall on any block);
    queries, gates, indices and output once.  Flops: 2 (d_k + d_v) per query head and visible key of each branch.
    Compression: raw rows under a new compressed row once, new compressed rows once."""
    es, hk, row = _elem(case), case["kv_heads"], (case["d_k"] + case["d_v"]) * _elem(case)
    lens = _lengths(case)
    if case["op"] == "compress":
        total = flops = 0
        for length in lens:
            nc = _cmp_rows(length)
            rows = nc if not case["new"] else min(nc, max(1, case["new"] // 2 // STRIDE))
            raw = (rows - 1) * STRIDE + L_CMP if rows else 0
            total += hk * row * (raw + rows)
            flops += hk * (case["d_k"] + case["d_v"]) * raw
        return {"bytes": total, "flops": flops}
    h, t, w, ns = case["heads"], case["queries"], case["window"], case["n_sel"]
    t_avg = t - (t // 2) / 2 if case["ragged"] else t
    forced = N_INIT + N_LOCAL
    free = max(0, ns - forced)
    fresh = free * (1 + (t_avg - 1) * (1 - 0.6 * case["rho"] ** 2))
    nbytes = flops = 0
    for length in lens:
        nc, raw = _cmp_rows(length), length + t_avg
        blocks = max(1.0, raw / L_SEL - forced)
        distinct = N_INIT + blocks * (1 - math.exp(-fresh / blocks))
        nbytes += hk * row * (nc + min(raw, distinct * L_SEL + min(raw, w + t_avg)))
        flops += 2 * h * t_avg * (case["d_k"] + case["d_v"]) * (nc + min(raw, ns * L_SEL) + min(raw, w))
    nbytes += case["batch"] * t_avg * (h * (case["d_k"] + case["d_v"]) * es + h * 12 + hk * ns * 4)
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    """About four times what other groupings, slicings, kernels and the per-query execution of the same calls differ by
    (bf16: 2.3e-3, largest 1.4e-2; fp32: 1.9e-7, 1.1e-6), and the compressed rows from means in 64 bits (3e-7 and single
    units in the last place; fp32 9e-8).  Indices: the same calls agree in every entry; a tie in block importance within
    the rounding of fp32 sums may fall the other way, which moves up to 13 entries of one sorted set."""
    bf16 = case["dtype"] == "bf16"
    if case["op"] == "compress":
        return {"rel": 1e-5, "max": 1e-2} if bf16 else {"rel": 1e-6, "max": 1e-5}
    return {"rel": 9e-3, "max": 0.06, "differ": 0.005} if bf16 else {"rel": 2e-6, "max": 1e-5, "differ": 0.005}


# ---- the same outputs in 64 bits ------------------------------------------------------------------------------------
def _attend(q, k, v, visible, scale):
    """q [.., R, d_k], k [.., N, d_k], v [.., N, d_v], visible [.., R or 1, N]: (output, probabilities); a row that sees nothing is 0."""
    s = (q @ k.transpose(-1, -2).contiguous() * scale).masked_fill(~visible, -math.inf)
    m = s.amax(-1, keepdim=True)
    p = torch.exp(s - torch.where(torch.isinf(m), torch.zeros_like(m), m))
    z = p.sum(-1, keepdim=True)
    p = p / torch.where(z == 0, torch.ones_like(z), z)
    return p @ v, p


def _select(imp, own, n_sel):
    """imp [t, hk, nblk], own [t]: per query and KV head the forced blocks, then the best; -1 padded."""
    t, hk, nblk = imp.shape
    blk, own = torch.arange(nblk, device=imp.device).view(1, 1, nblk), own.view(t, 1, 1)
    score = torch.where((blk < N_INIT) | (blk > own - N_LOCAL), torch.full_like(imp, 1e9), imp)
    score = torch.where(blk > own, torch.full_like(score, -1.0), score)
    top, idx = score.sort(dim=-1, descending=True, stable=True)
    return torch.where(top < 0, torch.full_like(idx, -1), idx)[..., :n_sel]


def _exact_compress(s):
    out = []
    for x, c in ((s["k"], s["k_cmp"]), (s["v"], s["v_cmp"])):
        y = c.double()
        for b, after in enumerate(s["after"].tolist()):
            lo, hi = _cmp_rows(int(s["before"][b])) if s["before"] is not None else 0, _cmp_rows(after)
            if hi > lo:
                y[b, :, lo:hi] = x[b, :, lo * STRIDE:(hi - 1) * STRIDE + L_CMP].double().unfold(1, L_CMP, STRIDE).mean(-1)
        out.append(y)
    return out[0], out[1], None


def exact(case, seed):
    """The definition, query by query, in 64 bits.  The indices have no such value (a tie may fall either way)."""
    s = prepare(case, seed)
    if case["op"] == "compress":
        return _exact_compress(s)
    dev, t, h, hk = s["q"].device, case["queries"], case["heads"], case["kv_heads"]
    hg, scale = h // hk, 1.0 / math.sqrt(case["d_k"])
    parents = list(range(-1, t - 1)) if case["drafts"] == "chain" else _tree(case["drafts"])[0]
    depth, seen = [], torch.zeros((t, t), dtype=torch.bool)
    for i, p in enumerate(parents):
        depth.append(0 if p < 0 else depth[p] + 1)
        if p >= 0:
            seen[i] = seen[p]
        seen[i, i] = True
    seen, depth = seen.to(dev), torch.tensor(depth, device=dev)
    out = torch.zeros(s["out"].shape, dtype=torch.float64, device=dev)
    by_group = lambda x: x.view(-1, hk, hg, x.shape[-1])                       # [t, hk, hg, d]
    for b, (length, nq) in enumerate(zip(s["seq_lens"].tolist(), s["n_query"].tolist())):
        nc, rows = int(s["n_cmp"][b]), length + nq
        q = by_group(s["q"][b, :nq].double())
        gates = s["gates"][b, :nq].double().view(nq, hk, hg, 3)
        slot = torch.arange(rows, device=dev)
        draft = (slot - length).clamp(min=0)
        sees = (slot < length) | seen[:nq][:, draft]                           # [nq, rows]
        pos = torch.where(slot < length, slot, length + depth[draft])
        own_pos = length + depth[:nq]
        # compressed branch (its rows hold committed tokens only) and the importance of every block
        nblk = rows // L_SEL + 1
        imp = torch.zeros((nq, hk, nblk), dtype=torch.float64, device=dev)
        if nc:
            flat = q.permute(1, 0, 2, 3).reshape(hk, nq * hg, -1)
            o, p = _attend(flat, s["k_cmp"][b, :, :nc].double(), s["v_cmp"][b, :, :nc].double(),
                           torch.ones((1, 1, nc), dtype=torch.bool, device=dev), scale)
            o = o.view(hk, nq, hg, -1).permute(1, 0, 2, 3)
            p = p.view(hk, nq, hg, nc).sum(2).permute(1, 0, 2)
            per = L_SEL // STRIDE
            for m in range(per):
                for n in range(L_CMP // STRIDE):
                    c = torch.arange(nblk, device=dev) * per + m - n
                    ok = (c >= 0) & (c < nc)
                    imp += torch.where(ok, p[..., c.clamp(0, nc - 1)], torch.zeros_like(imp))
            acc = gates[..., 0:1] * o
        else:
            acc = torch.zeros((nq, hk, hg, case["d_v"]), dtype=torch.float64, device=dev)
        if case["mode"] == "reuse":
            sel = s["sel_idx"][b, :nq].long()
        else:
            sel = _select(imp, (length + torch.arange(nq, device=dev)) // L_SEL, case["n_sel"])
            if case["mode"] == "shared":                                       # the deepest (last) member's set for the whole run
                run_len = max(1, min(t, 64 // hg))
                for lo in range(0, nq, run_len):
                    d = depth[lo:min(lo + run_len, nq)].tolist()
                    sel[lo:lo + len(d)] = sel[lo + max(range(len(d)), key=lambda i: (d[i], i))].clone()
        k, v = s["k"][b], s["v"][b]                                            # [hk, rows, d]
        head = torch.arange(hk, device=dev).view(1, hk, 1)
        for lo in range(0, nq, 16):                                            # queries at a time
            qs = slice(lo, min(lo + 16, nq))
            x = sel[qs]
            tok = (x.clamp(min=0).unsqueeze(-1) * L_SEL + torch.arange(L_SEL, device=dev)).flatten(2)
            ok = (x >= 0).repeat_interleave(L_SEL, -1) & (tok < rows)
            tok = tok.clamp(max=rows - 1)
            ok = ok & torch.gather(sees[qs].unsqueeze(1).expand(-1, hk, -1), 2, tok)
            acc[qs] += gates[qs, ..., 1:2] * _attend(q[qs], k[head, tok].double(), v[head, tok].double(), ok.unsqueeze(2), scale)[0]
        lo = max(0, length - case["window"])
        near = (sees & (pos > own_pos.view(-1, 1) - case["window"]) & (pos <= own_pos.view(-1, 1)))[:, lo:].view(nq, 1, 1, -1)
        acc += gates[..., 2:3] * _attend(q, k[:, lo:rows].double(), v[:, lo:rows].double(), near, scale)[0]
        out[b, :nq] = acc.reshape(nq, h, -1)
    return out, None
