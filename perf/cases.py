"""The work that is timed: the calls of a Multi-Block Editing decoder's loop.

Each case is one pass through the package's public entry points, with what a
serving program holds in hand before the call: the paged KV pool and its page
table, the lengths on the device and their host copies (the scheduler's), the
output buffers, and for graphs the captured pool.  Kinds of case:

  window   window_attention, the editing pass over a paged prefix
  block    block_diffusion_attention, the ordinary one-block decoding step
  refresh  refresh_blocks, flagged kv_write, flagged block-causal attention:
           what restores the cache after an editing pass changed some blocks
  edit     edit_select over vocabulary logits
  update   threshold_update with entropies, then tail_entropy_scores and
           select_start_block: a whole decision step and the next window's
           start
  graph    EditPassGraphs.replay: attention and update of one pass, captured

Inputs are N(0, 1) queries, keys and values in bf16, pages in a random order,
and N(0, 3) logits of which every second row has a planted peak (a confident
prediction), as a decoder's rows are part sure and part unsure.
"""
import math

import torch

import paper_2607_22663_amd as mbe
from paper_2607_22663_amd.graphs import EditPassGraphs

PAGE = 16
DEV = "cuda"
OMEGA_MASK, OMEGA_EDIT = 0.5, 0.0     # the defaults of the graph pool
RHO, K_MAX = 0.25, 4                  # tail share and widest window, in blocks


def _attn(name, kind, batch, lo, hi, klo, khi, *, step=1, hq=16, hkv=4, d=128, block=32, v_major=False):
    """Prefixes are drawn from lo..hi in multiples of `step`, windows from
    klo..khi blocks."""
    c = {"kind": kind, "batch": batch, "prefix_lo": lo, "prefix_hi": hi, "prefix_step": step, "k_lo": klo, "k_hi": khi,
         "hq": hq, "hkv": hkv, "d": d, "block": block, "v_major": v_major}
    return dict(c, name=name) if name else c


def _rows(name, kind, rows, vocab, *, pad=0, block=32, theta=0.9):
    """`pad`: columns of the logits buffer past the vocabulary."""
    c = {"kind": kind, "rows": rows, "vocab": vocab, "pad": pad, "block": block}
    if kind == "edit":
        c["theta"] = theta
    return dict(c, name=name) if name else c


def _graph(name, batch, k, hi, vocab):
    c = {"kind": "graph", "batch": batch, "k_lo": k, "k_hi": k, "prefix_lo": hi // 4, "prefix_hi": hi, "prefix_step": 1,
         "hq": 16, "hkv": 4, "d": 128, "block": 32, "v_major": False, "vocab": vocab}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a small model's first window: nothing but latency and launches
        _attn("window_b1_p64_d64", "window", 1, 64, 64, 2, 2, hq=4, hkv=4, d=64),
        # one user, medium prompt, two-block window
        _attn("window_b1_p2048", "window", 1, 2048, 2048, 2, 2),
        # the ordinary decoding step on long prompts, a block per sequence
        _attn("block_b8_p16384", "block", 8, 16384, 16384, 1, 1),
        # a serving batch of mixed lengths, two-block windows
        _attn("window_b32_ragged", "window", 32, 512, 8192, 2, 2, step=32),
        # large batch on long contexts, four-block windows
        _attn("window_b64_long", "window", 64, 4096, 32768, 4, 4, step=32),
        # the cache layout most engines have (V like K), lengths that end
        # anywhere in a page, windows of one to eight blocks side by side
        _attn("window_b12_vmajor_odd", "window", 12, 1000, 12000, 1, 8, v_major=True),
        # cache refresh of the blocks an editing pass changed
        _attn("refresh_b16", "refresh", 16, 1000, 8192, 4, 4),
        # two blocks of one user against the vocabulary
        _rows("edit_r64", "edit", 64, 131072),
        # the rows of the large batch above
        _rows("edit_r8192", "edit", 8192, 131072, theta=0.95),
        # the rows of the serving batch: decision, entropies, next window
        _rows("update_r2048", "update", 2048, 131072),
        # a vocabulary that is no multiple of anything, rows packed behind each other
        _rows("update_r992_odd_vocab", "update", 992, 100003),
        # a whole captured pass of a small batch
        _graph("graph_b8_w64", 8, 2, 4096, 131072),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(["window", "window", "window", "block", "refresh", "edit", "update", "update", "graph"])
    block = rng.choice([16, 32])
    if kind in ("edit", "update"):
        vocab = _log_int(rng, 1000, 160000)
        if rng.random() < 0.5:
            vocab = max(1024, vocab // 128 * 128)         # most vocabularies are padded
        blocks = _log_int(rng, 1, max(1, min(8192, (1 << 30) // vocab) // block))
        pad = rng.choice([0, 0, rng.randrange(1, 64)])
        return _rows(None, kind, blocks * block, vocab, pad=pad, block=block, theta=rng.choice([0.5, 0.9, 0.95]))
    if kind == "graph":
        return _graph(None, _log_int(rng, 1, 16), rng.randint(1, 4), _log_int(rng, 256, 8192), _log_int(rng, 8192, 131072))
    d = rng.choice([64, 128, 128])
    hkv = rng.choice([2, 4, 8])
    hq = hkv * rng.choice([1, 4, 4, 8])
    k_hi = 1 if kind == "block" else rng.choice([1, 2, 4, 8])
    k_lo = rng.choice([1, k_hi])
    batch = _log_int(rng, 1, 64)
    # the bytes of all keys and the work on them stay below the largest listed case's
    most = min(32768, int(2.4e9 / (4 * hkv * d * batch)), int(1.2e12 / (4 * d * hq * k_hi * block * batch)))
    hi = _log_int(rng, 64, max(64, most - k_hi * block))
    lo = hi if rng.random() < 0.3 else max(0, int(hi * rng.uniform(0.05, 1.0)))
    return _attn(None, kind, batch, lo, hi, k_lo, k_hi, step=rng.choice([1, 32]), hq=hq, hkv=hkv, d=d, block=block,
                 v_major=rng.random() < 0.4)


# ------------------------------------------------------------------- inputs
def _windows(case):
    """Window lengths of the batch, every size from the widest down in turn."""
    sizes = range(case["k_hi"], case["k_lo"] - 1, -1)
    return [sizes[b % len(sizes)] * case["block"] for b in range(case["batch"])]


def _lengths(case, gen):
    """Host prefix and window lengths, int32."""
    n, st = case["batch"], case["prefix_step"]
    lo, hi = case["prefix_lo"] // st, case["prefix_hi"] // st
    p = torch.randint(lo, hi + 1, (n,), generator=gen, dtype=torch.int32) * st
    return p, torch.tensor(_windows(case), dtype=torch.int32)[torch.randperm(n, generator=gen)]


def _mean_lengths(case):
    """(sum of prefixes, sum of windows, sum of window * keys) as drawn on average."""
    p, ws = (case["prefix_lo"] + case["prefix_hi"]) / 2, _windows(case)
    return p * len(ws), sum(ws), sum(w * (p + w) for w in ws)


def _cache(case, seed):
    """Lengths, page table, pools and queries of one layer."""
    gen = torch.Generator().manual_seed(seed)
    g = torch.Generator(DEV).manual_seed(seed)
    hp, hw = _lengths(case, gen)
    pages = (hp + hw + PAGE - 1) // PAGE
    widest = int(pages.max())
    # the pool holds a batch of the longest sequences of the range
    total = case["batch"] * -(-(case["prefix_hi"] + case["k_hi"] * case["block"]) // PAGE)
    perm = torch.randperm(total, generator=gen).to(torch.int32)
    table = torch.zeros(case["batch"], widest, dtype=torch.int32)
    at = 0
    for b, n in enumerate(pages.tolist()):
        table[b, :n] = perm[at:at + n]
        at += n
    hkv, d = case["hkv"], case["d"]

    def normal(*shape):
        return torch.randn(*shape, generator=g, dtype=torch.bfloat16, device=DEV)

    s = {"hp": hp, "hw": hw, "max_p": int(hp.max()), "max_w": int(hw.max()), "block": case["block"],
         "prefix": hp.to(DEV), "window": hw.to(DEV), "table": table.to(DEV), "q": normal(int(hw.sum()), case["hq"], d),
         "k": normal(total, hkv, PAGE, d), "v": normal(total, hkv, PAGE, d) if case["v_major"] else normal(total, hkv, d, PAGE)}
    s["out"] = torch.zeros_like(s["q"])
    return s, gen, g


def _logits(rows, vocab, pad, g):
    """N(0, 3) rows with a peak of max + 8 in every second one, and the current tokens."""
    x = torch.empty(rows, vocab + pad, dtype=torch.bfloat16, device=DEV).normal_(0.0, 3.0, generator=g)
    n = rows // 2
    col = torch.randint(0, vocab, (n,), generator=g, device=DEV)
    peak = x[1:2 * n:2, :vocab].amax(dim=1) + 8
    x[torch.arange(1, 2 * n, 2, device=DEV), col] = peak
    cur = torch.randint(0, vocab - 1, (rows,), generator=g, device=DEV, dtype=torch.int32)
    return x, cur


def _update_inputs(case, rows, g):
    vocab, block = case["vocab"], case["block"]
    x, cur = _logits(rows, vocab, case.get("pad", 0), g)
    masked = torch.rand(rows, generator=g, device=DEV) < 0.4
    return x, torch.where(masked, torch.full_like(cur, vocab - 1), cur), vocab - 1, block


def _update_out(rows, block):
    return {"new_tokens": torch.empty(rows, dtype=torch.int32, device=DEV),
            "conf": torch.empty(rows, dtype=torch.float32, device=DEV),
            "action": torch.empty(rows, dtype=torch.uint8, device=DEV),
            "block_changed": torch.empty(rows // block, dtype=torch.uint8, device=DEV),
            "changed_count": torch.empty(1, dtype=torch.int32, device=DEV),
            "entropy": torch.empty(rows, dtype=torch.float32, device=DEV)}


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("window", "block"):
        s, _, _ = _cache(case, seed)
    elif kind == "refresh":
        s, gen, g = _cache(case, seed)
        n = case["k_hi"]
        s["max_w"] = n * case["block"]          # one flag per block of the widest window
        s["changed"] = (torch.rand(case["batch"], n, generator=gen) < 0.5).to(torch.uint8).to(DEV)
        s["flags"] = torch.empty_like(s["changed"])
        shape = (s["q"].shape[0], case["hkv"], case["d"])
        s["k_new"] = torch.randn(*shape, generator=g, dtype=torch.bfloat16, device=DEV)
        s["v_new"] = torch.randn(*shape, generator=g, dtype=torch.bfloat16, device=DEV)
    elif kind == "edit":
        g = torch.Generator(DEV).manual_seed(seed)
        rows = case["rows"]
        s = {"theta": case["theta"], "vocab": case["vocab"]}
        s["logits"], s["cur"] = _logits(rows, case["vocab"], case["pad"], g)
        s["out"] = tuple(torch.empty(rows, dtype=t, device=DEV) for t in (torch.int32, torch.float32, torch.uint8))
    elif kind == "update":
        g = torch.Generator(DEV).manual_seed(seed)
        rows, block = case["rows"], case["block"]
        s = {"vocab": case["vocab"], "block": block, "blocks": rows // block}
        s["logits"], s["cur"], s["mask_id"], _ = _update_inputs(case, rows, g)
        s["out"] = _update_out(rows, block)
        s["scores"] = torch.empty(rows // block, dtype=torch.float32, device=DEV)
        # the rows are the history of sequences of up to four blocks
        per = max(n for n in range(1, K_MAX + 1) if s["blocks"] % n == 0)
        s["per_seq"] = per
        s["current"] = torch.full((s["blocks"] // per,), per, dtype=torch.int32, device=DEV)
        s["start"] = torch.empty_like(s["current"])
    else:
        s, _, g = _cache(case, seed)
        batch, window = case["batch"], case["k_hi"] * case["block"]
        pool = EditPassGraphs(k_pages=s["k"], v_pages=s["v"], max_batch=batch, max_window=window, block_size=case["block"],
                              num_q_heads=case["hq"], max_pages_per_seq=s["table"].shape[1], max_prefix_len=case["prefix_hi"],
                              vocab=case["vocab"], mask_id=case["vocab"] - 1)
        x, cur, _, _ = _update_inputs(case, batch * window, g)
        put = pool.inputs(batch, window)
        for name, t in (("q", s["q"]), ("page_table", s["table"]), ("prefix_lens", s["prefix"]), ("logits", x), ("cur_tokens", cur)):
            put[name].copy_(t)
        pool.capture(batch, window)
        s = {"pool": pool, "shape": (batch, window)}
    s["kind"] = kind
    return s


# --------------------------------------------------------------------- a pass
def run(s):
    kind = s["kind"]
    if kind == "window":
        return mbe.window_attention(s["q"], s["k"], s["v"], s["table"], s["prefix"], s["window"], s["block"], out=s["out"],
                                    max_prefix_len=s["max_p"], max_window_len=s["max_w"], host_prefix_lens=s["hp"],
                                    host_window_lens=s["hw"])
    if kind == "block":
        return mbe.block_diffusion_attention(s["q"], s["k"], s["v"], s["table"], s["prefix"], s["block"], out=s["out"],
                                             max_prefix_len=s["max_p"], host_prefix_lens=s["hp"])
    if kind == "refresh":
        mbe.refresh_blocks(s["changed"], "changed_and_later", out=s["flags"])
        mbe.kv_write(s["k"], s["v"], s["table"], s["prefix"], s["window"], s["k_new"], s["v_new"], max_len=s["max_w"],
                     block_flags=s["flags"], block_size=s["block"])
        mbe.window_attention(s["q"], s["k"], s["v"], s["table"], s["prefix"], s["window"], s["block"], out=s["out"],
                             mask_mode="block_causal", max_prefix_len=s["max_p"], max_window_len=s["max_w"],
                             host_prefix_lens=s["hp"], host_window_lens=s["hw"], block_flags=s["flags"])
        return {"flags": s["flags"], "out": s["out"], "k_pages": s["k"], "v_pages": s["v"]}
    if kind == "edit":
        new, conf, changed = mbe.edit_select(s["logits"], s["cur"], s["theta"], vocab=s["vocab"], out=s["out"])
        return {"new_tokens": new, "conf": conf, "changed": changed}
    if kind == "update":
        got = mbe.threshold_update(s["logits"], s["cur"], s["mask_id"], s["block"], OMEGA_MASK, OMEGA_EDIT, vocab=s["vocab"],
                                   with_entropy=True, out=s["out"])
        scores = mbe.tail_entropy_scores(got["entropy"], s["block"], RHO, out=s["scores"])
        start = mbe.select_start_block(scores.view(-1, s["per_seq"]), s["current"], K_MAX, out=s["start"])
        return dict(got, scores=scores, start=start)
    s["pool"].replay(*s["shape"])
    return s["pool"].outputs(*s["shape"])


def work(case):
    kind = case["kind"]
    nbytes = flops = 0.0
    if kind in ("edit", "update"):
        rows, vocab = case["rows"], case["vocab"]
    elif kind == "graph":
        rows, vocab = case["batch"] * case["k_hi"] * case["block"], case["vocab"]
    if kind in ("edit", "update", "graph"):
        nbytes += rows * vocab * 2 + rows * (13 if kind == "edit" else 17)
        flops += 4.0 * rows * vocab                    # compare, subtract, exponentiate, add
    if kind not in ("edit", "update"):
        p, w, pairs = _mean_lengths(case)
        kv, share = case["hkv"] * case["d"] * 4, 1.0
        if kind == "refresh":
            share = (case["k_hi"] - 1 + 0.5 ** case["k_hi"]) / case["k_hi"]     # blocks after the first changed one
            nbytes += 2 * share * w * kv               # new K/V read and written
        nbytes += (p + w) * kv + share * w * case["hq"] * case["d"] * 4
        flops += 4.0 * case["d"] * case["hq"] * pairs * share
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Attention: bf16 outputs and bf16 probabilities.  Confidences, entropies
    and scores: fp32 sums.  Tokens, actions and flags are the same unless a
    confidence lies within rounding of a threshold."""
    if case["kind"] in ("edit", "update"):
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-3}
    return {"rel": 1e-2, "max": 5e-2, "differ": 1e-3}


# ------------------------------------------------------------- 64-bit results
def _exact_attention(s, causal, flags=None, out=None):
    """Attention of every sequence over its gathered pages, in float64."""
    q, k, v, block = s["q"], s["k"], s["v"], s["block"]
    hq, d = q.shape[1], q.shape[2]
    hkv = k.shape[1]
    group = hq // hkv
    if tuple(v.shape) != tuple(k.shape):
        v = v.transpose(2, 3)
    res = torch.zeros(q.shape, dtype=torch.float64, device=DEV) if out is None else out.double()
    row = 0
    for b, (p, w) in enumerate(zip(s["hp"].tolist(), s["hw"].tolist())):
        n = p + w
        ids = s["table"][b, :(n + PAGE - 1) // PAGE].long()
        i = torch.arange(w, device=DEV)
        seen = torch.arange(n, device=DEV)[None, :] < (p + (i // block + 1) * block)[:, None] if causal else None
        for g in range(hkv):
            kk = k[ids, g].reshape(-1, d)[:n].double()
            vv = v[ids, g].reshape(-1, d)[:n].double()
            for h in range(g * group, (g + 1) * group):
                sc = q[row:row + w, h].double() @ kk.t().contiguous() / math.sqrt(d)
                if seen is not None:
                    sc = sc.masked_fill(~seen, -math.inf)
                o = torch.softmax(sc, dim=1) @ vv
                if flags is None:
                    res[row:row + w, h] = o
                else:
                    keep = flags[b, i // block] != 0
                    res[row:row + w, h] = torch.where(keep[:, None], o, res[row:row + w, h])
        row += w
    return res


def _exact_rows(x, vocab):
    """(argmax, confidence, entropy) of every row in float64, lowest index on ties."""
    idx, conf, ent = [], [], []
    step = max(1, (1 << 27) // vocab)
    cols = torch.arange(vocab, device=DEV)
    for r in range(0, x.shape[0], step):
        y = x[r:r + step, :vocab].double()
        m = y.amax(dim=1, keepdim=True)
        idx.append(torch.where(y == m, cols, vocab).amin(dim=1))
        e = torch.exp(y - m)
        z = e.sum(dim=1)
        conf.append(1 / z)
        ent.append(torch.log(z) - (e * (y - m)).sum(dim=1) / z)
    return torch.cat(idx), torch.cat(conf), torch.cat(ent)


def _exact_update(x, cur, vocab, mask_id, block):
    idx, conf, ent = _exact_rows(x, vocab)
    masked = (cur == mask_id).view(-1, block)
    c = conf.view(-1, block)
    unmask = masked & (c > OMEGA_MASK)
    best = torch.where(masked, c, -1.0).argmax(dim=1, keepdim=True)
    force = torch.zeros_like(masked).scatter_(1, best, True) & masked & ~unmask.any(dim=1, keepdim=True)
    edit = ~masked & (idx != cur).view(-1, block) & (c >= OMEGA_EDIT)
    action = (unmask.int() + 2 * force.int() + 3 * edit.int()).to(torch.uint8)
    act = action.view(-1) != 0
    return {"new_tokens": torch.where(act, idx, cur.long()).to(torch.int32), "conf": conf, "action": action.view(-1),
            "block_changed": act.view(-1, block).any(dim=1).to(torch.uint8),
            "changed_count": act.sum().view(1).to(torch.int32), "entropy": ent}


def exact(case, seed):
    kind = case["kind"]
    if kind != "graph":
        s = prepare(case, seed)
    if kind in ("window", "block"):
        return _exact_attention(s, False)
    if kind == "refresh":
        n = case["k_hi"]
        flags = (torch.cummax(s["changed"].int(), dim=1).values != 0).to(torch.uint8)
        start, row, block = s["hp"].tolist(), 0, s["block"]
        major = tuple(s["v"].shape) == tuple(s["k"].shape)
        for b, w in enumerate(s["hw"].tolist()):
            for i in range(min(n, w // block)):
                if flags[b, i]:
                    pos = torch.arange(start[b] + i * block, start[b] + (i + 1) * block, device=DEV)
                    page, slot = s["table"][b, pos // PAGE].long(), pos % PAGE
                    rows = slice(row + i * block, row + (i + 1) * block)
                    s["k"][page, :, slot] = s["k_new"][rows]
                    if major:
                        s["v"][page, :, slot] = s["v_new"][rows]
                    else:
                        s["v"][page, :, :, slot] = s["v_new"][rows]
            row += w
        return {"flags": flags, "out": _exact_attention(s, True, flags, s["out"]), "k_pages": s["k"], "v_pages": s["v"]}
    if kind == "edit":
        idx, conf, _ = _exact_rows(s["logits"], s["vocab"])
        change = (idx != s["cur"]) & (conf >= s["theta"])
        return {"new_tokens": torch.where(change, idx, s["cur"].long()).to(torch.int32), "conf": conf,
                "changed": change.to(torch.uint8)}
    if kind == "update":
        got = _exact_update(s["logits"], s["cur"], s["vocab"], s["mask_id"], s["block"])
        k = math.ceil(RHO * s["block"])
        scores = got["entropy"].view(-1, s["block"]).sort(dim=1, descending=True).values[:, :k].mean(dim=1)
        sc = scores.view(-1, s["per_seq"])
        lo = max(0, s["per_seq"] - K_MAX + 1)
        start = sc[:, lo:].argmax(dim=1).to(torch.int32) + lo
        return dict(got, scores=scores, start=start)
    s, _, g = _cache(case, seed)
    batch, window = case["batch"], case["k_hi"] * case["block"]
    x, cur, mask_id, block = _update_inputs(case, batch * window, g)
    return dict(_exact_update(x, cur, case["vocab"], mask_id, block), attention=_exact_attention(s, False))
