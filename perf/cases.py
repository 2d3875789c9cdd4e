"""Performance cases: what a user of the library has it do, sized by use.

Each case is one call (or one step of calls) through the public binding:

* ``fwd``: ``libra_attn_fwd`` of a tile list;
* ``bwd``: ``libra_attn_bwd`` of a tile list, bf16 dK / dV (the default mode);
* ``step``: forward and backward of one worker's tile set, dK / dV summed into
  zeroed fp32 buffers (how a pool's workers run);
* ``plan``: the host side of an optimizer step, ``libra_vrsp`` over a window
  of packs and ``libra_plan`` of the first pool that it forms.

Sample lengths are long-tailed (lognormal, median 644 tokens, with an optional
Pareto tail and one forced long sample at the end of a pack), drawn from the
case's own ``len_seed``; tensors are standard normal in bf16, drawn from the
seed that is passed in.  Buffers, workspace and the device copy of the tile
list are made once, as a training program keeps them over its layers.
"""
import math

import numpy as np
import torch

import paper_2607_23250_amd as pl

DEV = "cuda:0"


def _case(name, op, **kw):
    c = dict(op=op, packs=1, tokens=4096, forced=0, sigma=1.5, tail=0, len_seed=1, h_q=32, h_kv=8,
             d=128, B=2048, H=2, cp=1, share=False, worker=-1, tile=-1, window=0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one short prompt: nothing but launches and latency
        _case("fwd_512_d64", "fwd", tokens=512, h_q=8, h_kv=2, d=64, B=256, sigma=1.0),
        # the smallest workload of the repository: a 4K pack, two heads
        _case("fwd_4K_d64", "fwd", tokens=4096, h_q=2, h_kv=1, d=64, B=256, cp=4, sigma=1.0),
        # the backward of a small model's 4K pack
        _case("bwd_4K_d64", "bwd", tokens=4096, h_q=8, h_kv=2, d=64, B=512, sigma=1.0),
        # a whole 32K pack with the attention shapes of Qwen3-8B, each direction
        _case("fwd_32K", "fwd", tokens=32768, forced=16384, cp=8, len_seed=2),
        _case("bwd_32K", "bwd", tokens=32768, forced=16384, cp=8, len_seed=2),
        # a ragged pack: sizes that are multiples of nothing, three query heads
        # per KV head, blocks that end inside every kernel tile
        _case("step_ragged_d64", "step", tokens=20010, h_q=12, h_kv=4, d=64, B=1237, H=4,
              len_seed=3),
        # one worker of a pool of 8 packs of 64K (Qwen3-30B-A3B shapes)
        _case("step_pool_worker", "step", packs=8, tokens=65536, tail=8192, h_kv=4, B=4096,
              len_seed=3, worker=2),
        # one tile per call: 2048 rows x 4 heads deep inside a 256K pack's long sample
        _case("step_one_tile", "step", tokens=262144, forced=240000, h_kv=4, B=2048, H=8, cp=16,
              len_seed=4, tile=100),
        # a context-parallel rank's share of a 256K pack (Qwen3-235B-A22B shapes)
        _case("bwd_256K_share", "bwd", tokens=262144, forced=200000, h_q=64, h_kv=4, B=4096, cp=16,
              share=True, len_seed=4),
        # a context-parallel rank's share of a 1M pack, each direction: the largest calls
        _case("fwd_1M_share", "fwd", tokens=1048576, forced=900000, sigma=2.0, tail=32768, h_kv=4,
              B=8192, cp=16, share=True, len_seed=5),
        _case("bwd_1M_share", "bwd", tokens=1048576, forced=900000, sigma=2.0, tail=32768, h_kv=4,
              B=8192, cp=16, share=True, len_seed=5),
        # the planner of one optimizer step: a window of 64 packs of 256K, a
        # pool of 8 packs on 64 workers
        _case("plan_256K_pool8", "plan", packs=8, tokens=262144, tail=8192, h_kv=4, B=4096, cp=8,
              window=64),
    ]


_HEADS = ((1, 1), (2, 1), (4, 1), (4, 4), (6, 3), (8, 2), (8, 8), (12, 4), (16, 2), (32, 4),
          (32, 8), (64, 4))


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    op = rng.choice(("fwd", "fwd", "bwd", "bwd", "step", "step", "plan"))
    seed = rng.randrange(1 << 20)
    sigma = rng.choice((1.0, 1.5, 2.0))
    h_q, h_kv = rng.choice(_HEADS)
    d = rng.choice((64, 128, 128))
    H = rng.choice([h for h in (1, 2, 4, 8) if h_q % h == 0 and (h_kv % h == 0 or h % h_kv == 0)])
    c = _case(None, op, sigma=sigma, h_q=h_q, h_kv=h_kv, d=d, H=H, len_seed=seed)
    if op == "plan":
        c.update(packs=rng.choice((1, 2, 4, 8)), cp=rng.choice((1, 2, 4, 8)), tail=8192,
                 tokens=_log_uniform(rng, 512, 8192) * 32, B=_log_uniform(rng, 1024, 8192))
        c["window"] = c["packs"] * rng.choice((4, 8, 16))
        return c
    form = rng.choice(("pack", "pack", "pool", "share", "tile"))
    if form in ("pack", "pool"):
        c["packs"] = rng.choice((2, 3, 4)) if form == "pool" else 1
        c["tokens"] = 2 * _log_uniform(rng, 128, 32768 // c["packs"])
        c["B"] = min(_log_uniform(rng, 128, 8192), c["tokens"])
        if form == "pool":
            c["worker"] = rng.randrange(c["packs"])
        elif rng.random() < 0.5:
            c["forced"] = rng.randint(1, c["tokens"] // 2)
        return c
    cp = rng.choice((4, 8, 16))
    B = _log_uniform(rng, 256, 4096)
    c.update(cp=cp, B=B)
    c["tokens"] = 2 * cp * B * rng.randint(1, max(1, 131072 // (2 * cp * B)))
    c["forced"] = rng.randint(1, int(0.95 * c["tokens"]))
    if form == "share":
        c["share"] = True
    else:
        c["tile"] = rng.randrange(c["tokens"] // B)
    return c


def draw(rng):
    while True:
        c = _draw_once(rng)
        if c["op"] == "plan" or (len(_tiles(c)[1]) > 0 and work(c)["flops"] < 1.5e14):
            return c


# ---------------------------------------------------------------------------
# sample lengths and tiles

def _fill(rng, case, room):
    """Sample lengths of one pack: draws until `room` tokens are full, the last one cut."""
    out = []
    while room > 0:
        if case["tail"] and rng.random() < 0.05:
            n = int(case["tail"] / (1.0 - rng.random()) ** (1 / 1.1))
        else:
            n = int(round(644 * math.exp(case["sigma"] * rng.standard_normal())))
        n = min(max(n, 1), room)
        out.append(n)
        room -= n
    return out


def _pack_list(case, seed, packs):
    rng = np.random.default_rng(seed)
    forced = [case["forced"]] if case["forced"] else []
    return [_fill(rng, case, case["tokens"] - case["forced"]) + forced for _ in range(packs)]


def _lengths(case):
    return [n for p in _pack_list(case, case["len_seed"], case["packs"]) for n in p]


def _plan(case, lengths, **kw):
    return pl.libra_plan(lengths, [case["tokens"]] * case["packs"], block_tokens=case["B"],
                         head_shards=case["H"], cp=case["cp"], num_q_heads=case["h_q"],
                         num_kv_heads=case["h_kv"], head_dim=case["d"], **kw)


def _tiles(case):
    """(sample lengths, the call's tiles, query rows of its buffers)."""
    lengths, q_ranges = _lengths(case), None
    if case["share"]:
        c = case["tokens"] // (2 * case["cp"])
        q_ranges = [(0, c), (case["tokens"] - c, case["tokens"])]
    elif case["tile"] >= 0:
        b = case["tile"] * case["B"]
        q_ranges = [(b, min(b + case["B"], case["tokens"]))]
    tiles, _ = _plan(case, lengths, q_ranges=q_ranges)
    rows = sum(lengths) if q_ranges is None else sum(e - b for b, e in q_ranges)
    if case["worker"] >= 0:
        tiles = tiles[tiles["worker"] == case["worker"]]
    elif case["tile"] >= 0:
        tiles = tiles[:1]
    return lengths, tiles, rows


# ---------------------------------------------------------------------------

def prepare(case, seed):
    if case["op"] == "plan":
        return {"case": case, "packs": _pack_list(case, seed, case["window"])}
    lengths, tiles, rows = _tiles(case)
    h_q, h_kv, d = case["h_q"], case["h_kv"], case["d"]
    keys = sum(lengths)
    g = torch.Generator(device=DEV).manual_seed(int(seed))

    def randn(n, h):
        out = torch.empty((n, h, d), dtype=torch.bfloat16, device=DEV)
        step = max(1, (1 << 28) // (h * d))
        for a in range(0, n, step):
            m = min(step, n - a)
            out[a:a + m] = torch.randn((m, h, d), generator=g, device=DEV)
        return out

    cu = np.zeros(len(lengths) + 1, dtype=np.int64)
    cu[1:] = np.cumsum(lengths)
    s = {"case": case, "q": randn(rows, h_q), "k": randn(keys, h_kv), "v": randn(keys, h_kv),
         "cu": torch.from_numpy(cu).to(DEV), "tiles": pl.tiles_to_device(tiles, DEV)}
    s["o"] = torch.zeros_like(s["q"])
    s["lse"] = torch.zeros((h_q, rows), dtype=torch.float32, device=DEV)
    size = [pl.libra_attn_workspace_size(len(tiles), len(lengths), rows, keys, h_q, h_kv, d, b)
            for b in (False, True)]
    s["ws"] = pl.alloc_workspace(size[0] if case["op"] == "fwd" else max(size), DEV)
    if case["op"] != "fwd":
        s["do"] = randn(rows, h_q)
        s["dq"] = torch.zeros_like(s["q"])
        kv_type = torch.float32 if case["op"] == "step" else torch.bfloat16
        s["dk"] = torch.zeros(s["k"].shape, dtype=kv_type, device=DEV)
        s["dv"] = torch.zeros_like(s["dk"])
    if case["op"] == "bwd":
        _fwd(s)
    return s


def _fwd(s):
    pl.libra_attn_fwd(s["q"], s["k"], s["v"], s["cu"], s["tiles"], o=s["o"], lse=s["lse"],
                      workspace=s["ws"])


def run(s):
    case = s["case"]
    if case["op"] == "plan":
        order, pool_load, seq_work = pl.libra_vrsp(s["packs"], case["packs"])
        pool = [n for i in order[:case["packs"]] for n in s["packs"][i]]
        tiles, loads, received = _plan(case, pool, with_bytes=True)
        return {"order": order, "pool_load": pool_load, "seq_work": seq_work,
                "tiles": tiles.view(np.int32).reshape(len(tiles), -1), "loads": loads,
                "received": received}
    if case["op"] == "fwd":
        _fwd(s)
        return {"o": s["o"], "lse": s["lse"]}
    acc = case["op"] == "step"
    if acc:
        s["dk"].zero_()
        s["dv"].zero_()
        _fwd(s)
    pl.libra_attn_bwd(s["q"], s["k"], s["v"], s["o"], s["lse"], s["do"], s["cu"], s["tiles"],
                      dq=s["dq"], dk=s["dk"], dv=s["dv"], accumulate=acc, workspace=s["ws"])
    out = {"dq": s["dq"], "dk": s["dk"], "dv": s["dv"]}
    if acc:
        out.update(o=s["o"], lse=s["lse"])
    return out


def _fragments(lengths, tiles):
    """(sample start, first row of the sample, rows, Q row, heads) of every tile x sample."""
    cu = np.concatenate([[0], np.cumsum(lengths)])
    for t in tiles:
        b, e = int(t["q_begin"]), int(t["q_end"])
        j = int(np.searchsorted(cu, b, side="right")) - 1
        while j < len(lengths) and cu[j] < e:
            x, y = max(b, int(cu[j])), min(e, int(cu[j + 1]))
            yield (int(cu[j]), x - int(cu[j]), y - x, int(t["q_row"]) + x - b,
                   int(t["head_begin"]), int(t["head_end"]))
            j += 1


def work(case):
    if case["op"] == "plan":
        # the lengths once in, the orders and the tiles once out; a typical window
        n = sum(len(p) for p in _pack_list(case, case["len_seed"], min(case["window"], 8)))
        n = n * case["window"] // min(case["window"], 8)
        blocks = -(-case["tokens"] // case["B"]) * case["packs"]
        return {"bytes": 8 * (n + 2 * case["window"]) + 56 * blocks * case["H"], "flops": 0}
    lengths, tiles, _ = _tiles(case)
    d, G, esz = case["d"], case["h_q"] // case["h_kv"], 2
    pairs = int(tiles["cost"].sum())
    row_heads = int(((tiles["q_end"] - tiles["q_begin"])
                     * (tiles["head_end"] - tiles["head_begin"])).sum())
    reach = {}   # (sample start, KV head): keys that the covered rows attend
    for start, q0, n, _, h0, h1 in _fragments(lengths, tiles):
        for g in range(h0 // G, (h1 - 1) // G + 1):
            reach[start, g] = max(reach.get((start, g), 0), q0 + n)
    key_heads = sum(reach.values())
    fwd = row_heads * (2 * d * esz + 4) + key_heads * 2 * d * esz
    # q, o, dO and lse in, dQ out; K and V in; dK and dV out
    bwd = row_heads * (4 * d * esz + 4) + key_heads * 2 * d * esz
    all_kv = sum(lengths) * case["h_kv"] * d
    if case["op"] == "fwd":
        return {"bytes": fwd, "flops": 4 * d * pairs}
    if case["op"] == "bwd":
        return {"bytes": bwd + 2 * all_kv * esz, "flops": 10 * d * pairs}
    # a step zeroes the fp32 buffers, then adds to the reached keys
    return {"bytes": fwd + bwd + 2 * all_kv * 4 + key_heads * d * 16, "flops": 14 * d * pairs}


def tolerance(case):
    """bf16 outputs carry 2^-9 of rounding each; P, dS and the bf16 O of a
    backward add as much again.  Against 64 bits the outputs are 1.7e-3 (dV) to
    2.7e-3 (dQ) off; four times that."""
    return "exact" if case["op"] == "plan" else {"rel": 1e-2}


def exact(case, seed):
    """Softmax attention and its gradients in float64, sample by sample."""
    if case["op"] == "plan":
        return None
    if work(case)["flops"] > 2e14:
        return None   # over 20 seconds in 64 bits
    lengths, tiles, rows = _tiles(case)
    s = prepare(case, seed)
    h_q, h_kv, d = case["h_q"], case["h_kv"], case["d"]
    G, scale = h_q // h_kv, 1.0 / math.sqrt(d)
    f64 = dict(dtype=torch.float64, device=DEV)
    o, lse = torch.zeros((rows, h_q, d), **f64), torch.zeros((h_q, rows), **f64)
    back = case["op"] != "fwd"
    if back:
        dq = torch.zeros((rows, h_q, d), **f64)
        dk = torch.zeros((sum(lengths), h_kv, d), **f64)
        dv = torch.zeros_like(dk)
    for start, q0, n, row, h0, h1 in _fragments(lengths, tiles):
        for g in range(h0 // G, (h1 - 1) // G + 1):
            heads = slice(max(h0, g * G), min(h1, (g + 1) * G))
            nh = heads.stop - heads.start
            step = max(1, (1 << 26) // (nh * (q0 + n)))
            for a in range(0, n, step):
                m = min(step, n - a)
                rs, nk = slice(row + a, row + a + m), q0 + a + m
                ks = s["k"][start:start + nk, g].double()
                vs = s["v"][start:start + nk, g].double()
                qs = s["q"][rs, heads].double().reshape(m * nh, d)
                x = (qs @ ks.T).mul_(scale)
                late = (torch.arange(nk, device=DEV)[None, :]
                        > torch.arange(q0 + a, nk, device=DEV)[:, None])
                x.view(m, nh, nk).masked_fill_(late[:, None, :], -math.inf)
                l = torch.logsumexp(x, dim=1, keepdim=True)
                p = x.sub_(l).exp_()
                ov = p @ vs
                o[rs, heads] = ov.view(m, nh, d)
                lse[heads, rs] = l.view(m, nh).T
                if back:
                    dos = s["do"][rs, heads].double().reshape(m * nh, d)
                    dv[start:start + nk, g] += p.T @ dos
                    ds = (dos @ vs.T).sub_((dos * ov).sum(1, keepdim=True)).mul_(p)
                    dq[rs, heads] = (ds @ ks).mul_(scale).view(m, nh, d)
                    dk[start:start + nk, g] += (ds.T @ qs).mul_(scale)
    if case["op"] == "fwd":
        return {"o": o, "lse": lse}
    out = {"dq": dq, "dk": dk, "dv": dv}
    if case["op"] == "step":
        out.update(o=o, lse=lse)
    return out
