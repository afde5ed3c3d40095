"""Cases that the stage's speed is measured on, each through the public entry points of
paper_2503_08461_amd.fastcache.

A case is one batch in a paged pool: a compression call (SnapKV-style, key-norm, streaming or mixed, with or without
scores, with the row log-sum-exp handed over, or with the chunk MLP), or one decode step (append + attention).  A pass
rewinds the pool's metadata (free list, tables, lengths) and issues the call, so that it can be repeated on one state:
compaction writes only into blocks that were free, so the data needs no rewind.
"""

import math

import numpy as np
import torch

from paper_2503_08461_amd import fastcache as fc
from paper_2503_08461_amd import synth

_METHODS = {"snapkv": fc.FC_METHOD_SNAPKV, "knorm": fc.FC_METHOD_KNORM, "streaming": fc.FC_METHOD_STREAMING}


def _case(name, kind, layers, heads, dim, n_req, len_lo, len_hi, grain=1, method="snapkv", window=32, pool_kernel=7,
          keep_lo=20, keep_hi=20, entry="plain", in_place=False, chunk=5, hidden=256, act="erf", shape_seed=1):
    """One batch: n_req requests of len_lo + grain * i tokens (i drawn from shape_seed, up to len_hi), keep_lo..keep_hi
    per cent of the tokens kept; window 0: every request has its own window and pooling width."""
    c = dict(kind=kind, layers=layers, heads=heads, dim=dim, n_req=n_req, len_lo=len_lo, len_hi=len_hi, grain=grain,
             method=method, window=window, pool_kernel=pool_kernel, keep_lo=keep_lo, keep_hi=keep_hi, entry=entry,
             in_place=in_place, chunk=chunk, hidden=hidden, act=act, shape_seed=shape_seed)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one short prompt of a four-head toy model (benchmark configuration 1); launches and host
        # time are all there is
        _case("tiny_prompt", "compress", 1, 4, 64, 1, 256, 256, window=16, keep_lo=25, keep_hi=25),
        # one single-image prompt as soon as its prefill is done (configuration 2), from a serving loop that must not
        # allocate while it runs
        _case("single_image", "compress", 32, 32, 128, 1, 640, 640, keep_lo=25, keep_hi=25, entry="noalloc"),
        # one long prompt in a pool that holds one layer: the layer-by-layer use, where a call has few heads to offer
        _case("one_layer_long", "compress", 1, 32, 128, 2, 7001, 8000, window=32, keep_lo=15, keep_hi=25),
        # an ordinary batch of short prompts, half of them key-norm, half of the tokens kept (configuration 3)
        _case("mixed_batch", "compress", 8, 32, 128, 32, 600, 1200, method="mixed", keep_lo=50, keep_hi=50),
        # the headline: many multi-image prompts, a fifth of the tokens kept (configuration 4, 4 of its 32 layers)
        _case("multi_image", "compress", 4, 32, 128, 64, 1280, 7040, grain=576, window=64),
        # high concurrency with prompts of up to 16384 tokens, both scoring methods (configuration 5, 40 of 256 requests)
        _case("long_mixed", "compress", 2, 32, 128, 40, 512, 16384, method="mixed", keep_lo=10, keep_hi=50),
        # every request with its own window and pooling width, the scores asked for (a client that logs or reuses them)
        _case("scores_var", "scores", 2, 32, 128, 24, 500, 6000, window=0, keep_lo=10, keep_hi=40),
        # the prefill's row log-sum-exp: computed from the pool, then handed over to the one-pass score
        _case("given_lse", "lse", 4, 32, 128, 16, 1280, 7040, grain=576, window=64),
        # the paper's compressor, a small MLP over chunks of 5 tokens per modality (configuration 4's batch, 2 layers)
        _case("chunk_mlp", "mlp", 2, 32, 128, 24, 1280, 7040, grain=576),
        # the same with the narrow hidden layer, ragged segments and 64-channel heads: a small batch
        _case("chunk_mlp_small", "mlp", 4, 12, 64, 5, 300, 1501, chunk=4, hidden=128, act="tanh"),
        # one decode step of a large batch over uncompressed caches
        _case("decode_full", "decode", 2, 32, 128, 48, 1280, 7040, grain=576),
        # one decode step of a few requests over compressed caches, pool of one layer: what each layer of a model asks for
        _case("decode_small", "decode", 1, 32, 128, 8, 256, 1408),
    ]


_MAX_POOL_BYTES = 16e9
_MAX_COST = 12e9


def _cost(c):
    """Bytes of a pass, with the chunk MLP's arithmetic counted in."""
    w = work(c)
    return max(w["bytes"], w["flops"] / 200)


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["compress", "compress", "compress", "compress", "scores", "lse", "mlp", "decode", "decode"])
    layers = rng.choice([1, 2, 4, 8, 32])
    heads = rng.choice([4, 8, 12, 32, 32, 40])
    dim = rng.choice([64, 128, 128])
    n_req = log_int(1, 64)
    len_lo = log_int(130, 6000)
    len_hi = min(16384, len_lo * rng.choice([1, 2, 3]) + rng.randrange(16))
    method = rng.choice(["snapkv", "snapkv", "snapkv", "mixed", "knorm", "streaming"]) if kind == "compress" else "snapkv"
    window = rng.choice([16, 32, 64, rng.randrange(1, 65)])
    if kind == "scores" and rng.random() < 0.5:
        window = 0
    keep_lo = rng.randrange(5, 50)
    keep_hi = min(60, keep_lo + rng.randrange(20))
    entry = "noalloc" if kind == "compress" and len_hi <= 8192 and rng.random() < 0.25 else "plain"
    in_place = kind == "compress" and rng.random() < 0.15
    c = _case("", kind, layers, heads, dim, n_req, len_lo, len_hi, 1, method, window, rng.choice([1, 5, 7, 7, 13]), keep_lo,
              keep_hi, entry, in_place, rng.choice([2, 3, 4, 5, 8]), rng.choice([128, 256]), rng.choice(["erf", "tanh"]),
              rng.randrange(1 << 20))
    while (_pool_bytes(c) > _MAX_POOL_BYTES or _cost(c) > _MAX_COST) and c["n_req"] > 1:
        c["n_req"] = max(1, c["n_req"] // 2)
    while _pool_bytes(c) > _MAX_POOL_BYTES or _cost(c) > _MAX_COST:
        c["layers"] = max(1, c["layers"] // 2)
    return c


# --- the batch's shape ------------------------------------------------------------------------------------------------


def _shape(c):
    """(lengths, methods, budgets, windows, pooling widths), int32, from the case alone."""
    rng = np.random.Generator(np.random.PCG64(c["shape_seed"]))
    n = c["n_req"]
    lens = (c["len_lo"] + c["grain"] * rng.integers(0, (c["len_hi"] - c["len_lo"]) // c["grain"] + 1, size=n)).astype(np.int32)
    pct = rng.integers(c["keep_lo"], c["keep_hi"] + 1, size=n)
    if c["method"] == "mixed":
        methods = np.where(np.arange(n) % 2 == 0, fc.FC_METHOD_SNAPKV, fc.FC_METHOD_KNORM).astype(np.int32)
    else:
        methods = np.full(n, _METHODS[c["method"]], np.int32)
    if c["window"]:
        windows = np.full(n, c["window"], np.int32)
        widths = np.full(n, c["pool_kernel"], np.int32)
    else:
        windows = rng.integers(1, 65, size=n).astype(np.int32)
        widths = (2 * rng.integers(0, 8, size=n) + 1).astype(np.int32)
    floor = np.where(methods == fc.FC_METHOD_SNAPKV, windows, 1)
    budgets = np.maximum(lens * pct // 100, floor).astype(np.int32)
    return lens, methods, budgets, windows, widths


def _image_span(c, lens):
    """Where each request's image tokens lie: all but a short text prefix and suffix."""
    rng = np.random.Generator(np.random.PCG64(c["shape_seed"] + 1))
    begin = rng.integers(0, 65, size=len(lens)).astype(np.int32)
    end = (lens - rng.integers(0, 65, size=len(lens))).astype(np.int32)
    return begin, end


def _chunks(c, lens):
    """Rows that the chunk MLP makes of each request, per segment (text, image, text)."""
    b, e = _image_span(c, lens)
    k = c["chunk"]
    return (b + k - 1) // k, (e - b + k - 1) // k, (lens - e + k - 1) // k


def _new_tokens(c, lens, budgets):
    return sum(_chunks(c, lens)) if c["kind"] == "mlp" else lens * 0 + 16 if c["kind"] == "decode" else budgets


def _n_blocks(c):
    lens, _, budgets, _, _ = _shape(c)
    new = _new_tokens(c, lens, budgets)
    return int(math.ceil((int(((lens + 15) // 16).sum()) + int(((new + 15) // 16).sum())) / 0.85)) + 1


def _pool_bytes(c):
    return 2 * c["layers"] * _n_blocks(c) * 2 * c["heads"] * 16 * c["dim"]


def work(c):
    lens, methods, budgets, windows, _ = (a.astype(np.int64) for a in _shape(c))
    units, row = c["layers"] * c["heads"], 2 * c["dim"]
    if c["kind"] == "mlp":
        rows = int(sum(_chunks(c, lens)).sum())
        return {"bytes": units * 2 * row * (int(lens.sum()) + rows),
                "flops": units * 2 * rows * 2 * c["dim"] * c["hidden"] * (c["chunk"] + 1)}
    if c["kind"] == "decode":
        # every cached row and the new one, the new row in and out, the query in, the fp32 result out
        return {"bytes": units * (2 * row * int(lens.sum()) + len(lens) * (4 * row + row + 2 * row)),
                "flops": units * 4 * c["dim"] * int(lens.sum() + len(lens))}
    snap, scored = methods == fc.FC_METHOD_SNAPKV, methods != fc.FC_METHOD_STREAMING
    # the keys once, the kept values (and, where nothing was scored, the kept keys), both written
    b = int(lens[scored].sum()) * row + int(budgets[~scored].sum()) * row + int(budgets.sum()) * 3 * row
    b += int(windows[snap].sum()) * row
    f = int((2 * windows * lens * c["dim"])[snap].sum())
    if c["kind"] == "scores":
        b += 4 * int(lens.sum()) + 4 * int(budgets.sum())
    if c["kind"] == "lse":
        b += int(lens.sum()) * row + 8 * int(windows.sum())  # two calls, each reads the keys
        f *= 2
    return {"bytes": units * b, "flops": units * f}


# --- inputs ---------------------------------------------------------------------------------------------------------------


class _State:
    """A pool with a batch resident in it.  The library's side of it goes with the object."""

    def __init__(self, c, seed):
        dev = torch.device("cuda:0")
        self.case = c
        self.lens0, self.methods, self.budgets, self.windows, self.widths = _shape(c)
        n_blocks = _n_blocks(c)
        wl = synth.Workload("case", c["layers"], c["heads"], c["dim"], n_blocks, c["window"], c["pool_kernel"], self.lens0,
                            self.methods, self.budgets, seed, True, True)
        self.kv = torch.empty(wl.pool_shape(), dtype=torch.float16, device=dev)
        synth.fill_pool_device(wl, self.kv)
        self.pool = fc.fc_pool_create(self.kv, n_blocks, c["layers"], c["heads"], c["dim"])
        if c["in_place"]:
            fc.fc_set_compaction_mode(self.pool, fc.FC_COMPACT_IN_PLACE)
        rows = synth.build_block_tables(wl, lambda n: fc.fc_pool_alloc(self.pool, n), lambda ids: fc.fc_pool_free(self.pool, ids),
                                        lambda ids, ix: ids[torch.from_numpy(ix).to(dev)].contiguous())
        # (a decode step may need one block more)
        table = np.full((len(self.lens0), wl.max_blocks + 1), -1, np.int32)
        for r, ids in enumerate(rows):
            table[r, :ids.shape[0]] = ids.cpu().numpy()
        self.table0 = torch.from_numpy(table).to(dev)
        self.table = self.table0.clone()
        self.lens = self.lens0.copy()
        stack, self.top0 = fc.fc_pool_export_state(self.pool)
        self.stack0 = torch.from_numpy(stack).to(dev)

        gen = torch.Generator(device=dev)
        gen.manual_seed(seed + 4000)
        normal = lambda *shape, dtype=torch.float16: torch.empty(shape, dtype=dtype, device=dev).normal_(0.0, 1.0, generator=gen)  # noqa: E731
        n, units, d = len(self.lens0), c["layers"] * c["heads"], c["dim"]
        self.scores = self.kept = None
        if c["kind"] == "decode":
            self.new_kv = normal(n, c["layers"], 2, c["heads"], d)
            self.q = normal(n, c["layers"], c["heads"], d)
            self.out = torch.zeros((n, c["layers"], c["heads"], d), dtype=torch.float32, device=dev)
            return
        if c["kind"] == "mlp":
            self.begin, self.end = _image_span(c, self.lens0)
            k, h = c["chunk"], c["hidden"]
            self.w1 = [(normal(h, k * d, dtype=torch.float32) / math.sqrt(k * d)).half() for _ in range(2)]
            self.b1 = [0.1 * normal(h, dtype=torch.float32) for _ in range(2)]
            self.w2 = [(normal(d, h, dtype=torch.float32) / math.sqrt(h)).half() for _ in range(2)]
            self.b2 = [0.1 * normal(d, dtype=torch.float32) for _ in range(2)]
            fc.fc_mlp_set_weights(self.pool, k, self.w1, self.b1, self.w2, self.b2,
                                  fc.FC_ACT_GELU_ERF if c["act"] == "erf" else fc.FC_ACT_GELU_TANH)
            return
        snap = self.methods == fc.FC_METHOD_SNAPKV
        self.q = None
        if snap.any():
            self.q = (normal(n, c["layers"], c["heads"], c["window"], d) if c["window"]
                      else normal(int(self.windows[snap].sum()) * units * d))
        if c["kind"] == "scores":
            self.scores = torch.zeros(int(self.lens0.sum()) * units, dtype=torch.float32, device=dev)
        if c["kind"] == "lse":
            self.lse = torch.zeros((n, c["layers"], c["heads"], c["window"]), dtype=torch.float32, device=dev)
        if c["kind"] == "scores" or c["entry"] == "noalloc" or n == 1:
            self.kept = torch.zeros(int(self.budgets.sum()) * units, dtype=torch.int32, device=dev)

    def __del__(self):
        if getattr(self, "pool", None) is not None:
            fc.fc_pool_destroy(self.pool)
            self.pool = None


def prepare(case, seed):
    s = _State(case, int(seed))
    torch.cuda.synchronize()
    return s


# --- one pass -------------------------------------------------------------------------------------------------------------


def run(s):
    c = s.case
    fc.fc_pool_import_state_dev(s.pool, s.stack0, s.top0)
    s.table.copy_(s.table0)
    s.lens[:] = s.lens0
    if c["kind"] == "decode":
        fc.fc_append_batch(s.pool, s.table, s.lens, s.new_kv)
        fc.fc_decode_attention(s.pool, s.table, s.lens, s.q, s.out)
        return {"out": s.out, "table": s.table, "lens": s.lens, "kv": s.kv.view(torch.int64)}
    if c["kind"] == "mlp":
        fc.fc_compress_batch_mlp(s.pool, s.table, s.lens, s.begin, s.end)
        return {"kv": s.kv, "table": s.table, "lens": s.lens, "free": fc.fc_pool_num_free(s.pool)}
    if c["kind"] == "lse":
        fc.fc_window_lse(s.pool, s.table, s.lens, s.q, c["window"], s.methods, s.lse)
        fc.fc_compress_batch_lse(s.pool, s.table, s.lens, s.q, s.lse, c["window"], s.methods, s.budgets, c["pool_kernel"])
    elif c["window"] == 0:
        fc.fc_compress_batch_var(s.pool, s.table, s.lens, s.q, s.windows, s.methods, s.budgets, s.widths, 0.0, s.scores, s.kept)
    else:
        call = fc.fc_compress_batch_noalloc if c["entry"] == "noalloc" else fc.fc_compress_batch
        call(s.pool, s.table, s.lens, s.q, c["window"], s.methods, s.budgets, c["pool_kernel"], 0.0, s.scores, s.kept)
    # (copied rows are bytes: compared as whole numbers)
    got = {"kv": s.kv.view(torch.int64), "table": s.table, "lens": s.lens, "free": fc.fc_pool_num_free(s.pool)}
    if s.kept is not None:
        got["kept"] = s.kept
    if s.scores is not None:
        got["scores"] = s.scores
    if c["kind"] == "lse":
        got["lse"] = s.lse
    return got


def tolerance(c):
    # rel: four times the distance from 64 bits measured on these cases (fp32 sums of fp16 products and exponentials:
    # scores and attention 5e-7, log-sum-exp 5e-8; fp16 rounding of hidden layer and result over the whole pool: 9e-5).
    # differ: two tokens whose pooled scores are closer than that rounding may swap at a head's threshold (pooled scores
    # near it are about 5e-4 of their value apart), and the kept entries between the two then move by one place.
    if c["kind"] == "mlp":
        return {"rel": 4e-4}
    if c["kind"] == "decode":
        return {"rel": 2e-6}
    return {"rel": 4e-7 if c["kind"] == "lse" else 2e-6, "differ": 5e-4}


# --- the same in 64 bits ----------------------------------------------------------------------------------------------------


def _keys_values(s, r, n):
    """fp64 [layers][heads][n][dim] of request r's first n tokens: keys, values (before the pass)."""
    ids = s.table0[r, :(n + 15) // 16].long()
    t = s.kv[:, ids].double()  # [layer][block][2][head][16][d]
    t = t.permute(2, 0, 3, 1, 4, 5).flatten(3, 4)[..., :n, :]
    return t[0], t[1]


def _exact_scores(s):
    """(scores, lse) as the entry points lay them out."""
    c = s.case
    scores, lses, at = [], [], 0
    shape = (c["layers"], c["heads"])
    for r, L in enumerate(int(x) for x in s.lens0):
        w, width = int(s.windows[r]), int(s.widths[r])
        if c["window"]:
            q = s.q[r].double()
        else:
            n = c["layers"] * c["heads"] * w * c["dim"]
            q = s.q[at:at + n].view(*shape, w, c["dim"]).double()
            at += n
        k, _ = _keys_values(s, r, L)
        logits = q @ k.transpose(-1, -2).contiguous() / math.sqrt(c["dim"])
        pos = torch.arange(L, device=q.device)
        logits.masked_fill_(pos[None, :] > (L - w + torch.arange(w, device=q.device))[:, None], float("-inf"))
        lses.append(torch.logsumexp(logits, -1))
        a = torch.softmax(logits, -1).sum(-2)
        full = torch.full_like(a, float("inf"))
        if L > w:
            p = a[..., :L - w]
            full[..., :L - w] = torch.nn.functional.max_pool1d(p.reshape(-1, 1, L - w), width, 1, width // 2).view(p.shape)
        scores.append(full.reshape(-1))
    return torch.cat(scores), (torch.stack(lses) if c["window"] else None)


def _exact_mlp(s):
    """The pool after the call, fp64."""
    c = s.case
    k, d = c["chunk"], c["dim"]
    kv = s.kv.double()
    popped = s.stack0[:s.top0].flip(0).long()
    at = 0
    for r, L in enumerate(int(x) for x in s.lens0):
        both = torch.stack(_keys_values(s, r, L))  # [2][layer][head][L][d]
        b, e = int(s.begin[r]), int(s.end[r])
        parts = []
        for m, lo, hi in ((0, 0, b), (1, b, e), (0, e, L)):
            n = (hi - lo + k - 1) // k
            if n == 0:
                continue
            x = torch.zeros(*both.shape[:3], n * k, d, dtype=torch.float64, device=both.device)
            x[..., :hi - lo, :] = both[..., lo:hi, :]
            h = x.reshape(-1, k * d) @ s.w1[m].double().t().contiguous() + s.b1[m].double()
            h = torch.nn.functional.gelu(h, approximate="none" if c["act"] == "erf" else "tanh")
            y = h @ s.w2[m].double().t().contiguous() + s.b2[m].double()
            parts.append(y.view(*both.shape[:3], n, d))
        y = torch.cat(parts, 3)
        n = y.shape[3]
        nb = (n + 15) // 16
        blocks = popped[at:at + nb]
        at += nb
        old = kv[:, blocks].permute(2, 0, 3, 1, 4, 5).flatten(3, 4).contiguous()  # [2][layer][head][nb * 16][d]
        old[..., :n, :] = y
        kv[:, blocks] = old.unflatten(3, (nb, 16)).permute(1, 3, 0, 2, 4, 5).contiguous()
    return kv


def exact(case, seed):
    if case["kind"] == "compress":
        return None  # indices and copied bytes: no computed numbers come back
    s = prepare(case, seed)
    if case["kind"] == "mlp":
        return {"kv": _exact_mlp(s), "table": None, "lens": None, "free": None}
    if case["kind"] == "decode":
        out = torch.zeros(s.out.shape, dtype=torch.float64, device=s.out.device)
        for r, L in enumerate(int(x) for x in s.lens0):
            k, v = _keys_values(s, r, L)
            k = torch.cat([k, s.new_kv[r][:, 0].double()[:, :, None]], 2)
            v = torch.cat([v, s.new_kv[r][:, 1].double()[:, :, None]], 2)
            p = torch.softmax((k * s.q[r].double()[:, :, None]).sum(-1) / math.sqrt(case["dim"]), -1)
            out[r] = (p[..., None] * v).sum(2)
        return {"out": out, "table": None, "lens": None, "kv": None}
    scores, lse = _exact_scores(s)
    got = {"kv": None, "table": None, "lens": None, "free": None, "kept": None}
    if case["kind"] == "scores":
        got["scores"] = scores
    else:
        got["lse"] = lse
    return got
