"""The work that a user of this library has it do, as measurable cases.

A serving program loads its models once, keeps one scheduler with its queues,
and then passes requests through one of four public entry points:

  replay  Sched.sim_run on a trace whose payloads are in device memory
          (marshalled once with prepare_sim_run)
  group   Queue.run_group: one launch group the program formed itself
  static  the same through rb_run_group_static (no allocation)
  serve   host payloads: submit, flush, run_window, sync, collect

A case names the model (its kind, layer widths and type), the entry point, the
requests and the scheduler's options. Models and schedulers are kept for the
life of the process, as a server keeps them. How many rows each request has,
for which servable and when, belongs to the case (so that every seed's outputs
have one shape); every prepare() draws new payloads on the GPU from its seed
alone.
"""
import math
import zlib

import numpy as np
import torch

from paper_1712_06139_amd import rb

DEV = "cuda"
TABLES, TABLE_ROWS, EMB, N_DENSE = 26, 100_000, 64, 13  # the ranking model's tables and dense features
ZIPF = 1.1                                              # popularity of table rows
RANK_LAYERS = "1677-1024-512-256-1"
LARGE_LAYERS = "4096-8192-8192-4096"
SEQ_LAYERS = "256-512-256"
TENANT_LAYERS = "256-1024-1024-32"
SEQ_BUCKETS = (64, 128, 256, 512)
RANK_ALLOWED, LARGE_ALLOWED = "64,128,256,512", "128,256,512,1024"


def _case(name, kind, entry, layers, dtype, requests, rows, allowed, window=64, streams=8, bags=0, tokens=0,
          pack=False):
    """requests of 1..rows rows; allowed: batch sizes, the last the largest ("256+" closes at 256 and does not
    pad); bags: ids per bag 1..bags; tokens: longest sequence; window, streams, pack: the scheduler's options."""
    c = dict(kind=kind, entry=entry, layers=layers, dtype=dtype, requests=requests, rows=rows, allowed=allowed,
             window=window, streams=streams, bags=bags, tokens=tokens, pack=pack)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a small fp32 model's burst of requests: everything in one launch group, so launches and latency count
        _case("small_replay", "mlp", "replay", "64-128-16", "f32", 256, 8, "8,16,32"),
        # one ranking request at an idle server: the shortest chain of the flagship model
        _case("rank_one", "rank", "group", RANK_LAYERS, "bf16", 1, 8, RANK_ALLOWED, bags=20),
        # a lightly loaded ranking server: a few ragged batches in a launch group
        _case("rank_group", "rank", "group", RANK_LAYERS, "bf16", 120, 64, RANK_ALLOWED, bags=20),
        # the flagship: a backlogged ranking server in the benchmark's configuration
        _case("rank_replay", "rank", "replay", RANK_LAYERS, "bf16", 12000, 64, RANK_ALLOWED, bags=20),
        # the same server taking host payloads through the serving calls
        _case("rank_serve", "rank", "serve", RANK_LAYERS, "bf16", 128, 64, RANK_ALLOWED, streams=1, bags=20),
        # a large bf16 MLP with one small batch, in a loop that may not allocate
        _case("large_one", "mlp", "static", LARGE_LAYERS, "bf16", 7, 32, LARGE_ALLOWED),
        # the large MLP at moderate load: odd row counts in a few full batches
        _case("large_group", "mlp", "group", LARGE_LAYERS, "bf16", 250, 32, LARGE_ALLOWED),
        # the large MLP backlogged
        _case("large_replay", "mlp", "replay", LARGE_LAYERS, "bf16", 4000, 32, LARGE_ALLOWED),
        # one batch of ragged sequences in the longest bucket
        _case("seq_group", "seq", "group", SEQ_LAYERS, "f32", 24, 4, "64+", tokens=512),
        # ragged sequences over four length buckets, padded (the default) and with packed tokens
        _case("seq_replay", "seq", "replay", SEQ_LAYERS, "f32", 8000, 4, "64+", tokens=512),
        _case("seq_packed_replay", "seq", "replay", SEQ_LAYERS, "f32", 8000, 4, "64+", tokens=512, pack=True),
        # eight servables (four fp32 MLPs, four ranking models) sharing the device, closing on 2 ms timeouts
        _case("tenants_replay", "tenants", "replay", TENANT_LAYERS, "f32", 8000, 16, "256+", bags=20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: any entry point, from one request to a backlog, odd widths among them."""
    k = rng.randrange(8)
    window, streams = rng.choice([1, 8, 32, 64, 128]), rng.choice([1, 4, 8])
    if k == 0:  # small and medium fp32 MLPs of any width
        layers = "-".join(str(_log_int(rng, a, b)) for a, b in ((16, 512), (32, 1024), (1, 200)))
        entry, allowed = rng.choice(["replay", "group", "static"]), rng.choice(["8,16,32", "64,256", "100+", "256+"])
        return _case("", "mlp", entry, layers, "f32", _log_int(rng, 1, 4000 if entry == "replay" else 400),
                     rng.randint(1, 8), allowed, window, streams)
    if k == 1:  # large bf16 MLPs of any width
        layers = "-".join(str(_log_int(rng, 300, 6000)) for _ in range(rng.choice([3, 4])))
        return _case("", "mlp", rng.choice(["replay", "group"]), layers, "bf16", _log_int(rng, 1, 1500),
                     rng.randint(1, 32), rng.choice([LARGE_ALLOWED, "512+"]), window, streams)
    if k == 2:
        return _case("", "rank", "group", RANK_LAYERS, "bf16", _log_int(rng, 1, 1000), rng.randint(1, 64),
                     rng.choice([RANK_ALLOWED, "256+"]), bags=rng.randint(1, 40))
    if k == 3:
        return _case("", "rank", "replay", RANK_LAYERS, "bf16", _log_int(rng, 50, 10000), rng.randint(1, 64),
                     rng.choice([RANK_ALLOWED, "256+"]), window, streams, bags=rng.randint(2, 20))
    if k == 4:
        return _case("", "rank", "serve", RANK_LAYERS, "bf16", _log_int(rng, 1, 200), rng.randint(1, 64),
                     RANK_ALLOWED, window, 1, bags=rng.randint(1, 20))
    if k == 5:
        return _case("", "seq", "group", SEQ_LAYERS, "f32", _log_int(rng, 1, 200), rng.randint(1, 4), "64+",
                     tokens=_log_int(rng, 3, 512), pack=rng.random() < 0.5)
    if k == 6:
        return _case("", "seq", "replay", SEQ_LAYERS, "f32", _log_int(rng, 20, 8000), rng.randint(1, 4), "64+",
                     window, streams, tokens=_log_int(rng, 16, 512), pack=rng.random() < 0.5)
    return _case("", "tenants", "replay", TENANT_LAYERS, "f32", _log_int(rng, 100, 8000), rng.randint(1, 16), "256+",
                 window, streams, bags=rng.randint(1, 20))


# ---------------------------------------------------------------- models and servers, kept for the process

def _gen(*key):
    return torch.Generator(device=DEV).manual_seed(zlib.crc32(repr(key).encode()))


def _uniform(g, shape, a):
    return (torch.rand(shape, generator=g, device=DEV) * 2 - 1) * a


_weights, _models, _servers, _ctx = {}, {}, {}, []


def _params(kind, layers, seed):
    """fp32 parameters on the GPU: [(W, b, act)], tables, head."""
    key = (kind, layers, seed)
    if key not in _weights:
        g = _gen("weights", *key)
        dims = [int(v) for v in layers.split("-")]
        ls = []
        for i, (fi, fo) in enumerate(zip(dims[:-1], dims[1:])):
            last = i == len(dims) - 2
            act = ("sigmoid" if kind == "rank" else "none") if last else "relu"
            ls.append((_uniform(g, (fo, fi), math.sqrt(6.0 / (fi + fo))), _uniform(g, (fo,), fi ** -0.5), act))
        tables = head = None
        if kind == "rank":
            tables = torch.randn((TABLES, TABLE_ROWS, EMB), generator=g, device=DEV) / 8.0
        if kind == "seq":
            fi = dims[-1]
            head = (_uniform(g, (2, fi), math.sqrt(6.0 / (fi + 2))), _uniform(g, (2,), fi ** -0.5), "softmax")
        _weights[key] = (ls, tables, head)
    return _weights[key]


def _model(kind, layers, dtype, seed):
    key = (kind, layers, dtype, seed)
    if key not in _models:
        ls, tables, head = _params(kind, layers, seed)
        host = [(W.cpu().numpy(), b.cpu().numpy(), act) for W, b, act in ls]
        if not _ctx:
            _ctx.append(rb.Ctx(0))
        _models[key] = rb.Model(_ctx[0], {"rank": "ranking", "seq": "seqpool"}.get(kind, kind), dtype, host,
                                tables=None if tables is None else list(tables.cpu().numpy()),
                                n_dense=N_DENSE if kind == "rank" else 0,
                                head=None if head is None else (head[0].cpu().numpy(), head[1].cpu().numpy(), head[2]))
    return _models[key]


def _servables(case):
    """(kind, layers, dtype, seed) of each model that the server holds."""
    if case["kind"] == "tenants":
        return [("mlp", case["layers"], "f32", i) for i in range(4)] + [("rank", RANK_LAYERS, "bf16", i)
                                                                        for i in range(4)]
    return [(case["kind"], case["layers"], case["dtype"], 0)]


class _Server:
    def __init__(self, case):
        models = [_model(*s) for s in _servables(case)]
        self.sched = rb.Sched(_ctx[0], window_batches=case["window"], n_streams=case["streams"],
                              seq_pack=case["pack"])
        sizes = [int(v) for v in case["allowed"].rstrip("+").split(",")]
        padded = () if case["allowed"].endswith("+") else sizes
        timeout = 2_000_000 if case["kind"] == "tenants" else None
        buckets = (0,) if case["kind"] != "seq" else SEQ_BUCKETS if case["entry"] == "replay" else SEQ_BUCKETS[-1:]
        self.servables = [[rb.Queue(self.sched, m, sizes[-1], padded, timeout, bucket_len=b) for b in buckets]
                          for m in models]
        self.queue = self.servables[0][0]
        self.max_rows, self.padded = sizes[-1], padded
        self.now = 0


def _server(case):
    key = (tuple(_servables(case)), case["entry"], case["window"], case["streams"], case["pack"], case["allowed"])
    if key not in _servers:
        _servers[key] = _Server(case)
    return _servers[key]


# ---------------------------------------------------------------- requests

_cdf, _perm = [], {}


def _zipf_rows(g, table_of):
    """Table rows for ids of the given tables: Zipf-distributed ranks, scattered by a permutation per table."""
    if not _cdf:
        p = torch.arange(1, TABLE_ROWS + 1, dtype=torch.float64, device=DEV) ** -ZIPF
        _cdf.append(torch.cumsum(p / p.sum(), 0))
        gp = _gen("rows")
        _perm["rows"] = torch.stack([torch.randperm(TABLE_ROWS, generator=gp, device=DEV)
                                     for _ in range(TABLES)]).to(torch.int32).reshape(-1)
    ids = torch.empty(table_of.numel(), dtype=torch.int32, device=DEV)
    for a in range(0, ids.numel(), 1 << 24):
        t = table_of[a:a + (1 << 24)]
        u = torch.rand(t.numel(), generator=g, device=DEV, dtype=torch.float64)
        rank = torch.searchsorted(_cdf[0], u).clamp_(max=TABLE_ROWS - 1)
        ids[a:a + (1 << 24)] = _perm["rows"][t.to(torch.int64) * TABLE_ROWS + rank]
    return ids


def _requests(case, seed):
    """The requests of a seed: host metadata, payload arenas on the GPU in request order."""
    n = case["requests"]
    r = np.random.default_rng([n, case["rows"], case["tokens"]])
    rows = r.integers(1, case["rows"] + 1, n).astype(np.int32)
    arrival = np.cumsum(r.exponential(20_000, n)).astype(np.int64)
    models = _servables(case)
    p = 1.0 / np.arange(1, len(models) + 1)
    servable = r.choice(len(models), n, p=p / p.sum()).astype(np.int32)
    is_rank = np.array([m[0] == "rank" for m in models])[servable]
    d_in = np.array([N_DENSE if m[0] == "rank" else int(m[1].split("-")[0]) for m in models])[servable]
    d_out = np.array([2 if m[0] == "seq" else int(m[1].split("-")[-1]) for m in models])[servable]
    q = dict(n=n, rows=rows, arrival=arrival, servable=servable, d_in=d_in, d_out=d_out, lens=None, ids=None,
             lens_off=None, ids_off=None, max_len=None)
    off = lambda counts: np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)  # noqa: E731
    g = torch.Generator(device=DEV).manual_seed(seed)
    units = rows.astype(np.int64)
    if case["kind"] == "seq":
        u = r.random(int(rows.sum()))
        L = np.clip(np.floor(np.exp(u * math.log(case["tokens"] + 1))), 1, case["tokens"]).astype(np.int32)
        first = off(rows)[:-1]
        q["max_len"] = np.maximum.reduceat(L, first)
        units = np.add.reduceat(L.astype(np.int64), first)
        q["lens"], q["lens_off"] = torch.from_numpy(L).to(DEV), off(rows)
    if is_rank.any():
        rank_rows = np.where(is_rank, rows, 0).astype(np.int64)
        lens = torch.randint(1, case["bags"] + 1, (int(rank_rows.sum()), TABLES), generator=g, device=DEV)
        table_of = torch.arange(TABLES, dtype=torch.int32, device=DEV).repeat(lens.shape[0])
        q["ids"] = _zipf_rows(g, torch.repeat_interleave(table_of, lens.reshape(-1)))
        q["lens"], q["lens_off"] = lens.to(torch.int32).reshape(-1), off(rank_rows * TABLES)
        per_row = off(lens.sum(1).cpu().numpy())
        q["ids_off"] = per_row[off(rank_rows)]
    q["dense_off"], q["out_off"] = off(units * d_in), off(rows * d_out)
    q["dense"] = torch.randn(int(q["dense_off"][-1]), generator=g, device=DEV)
    return q


def _group(srv, q):
    """Descriptors of one launch group: the requests merged in order into batches, each padded to an allowed size."""
    batches, begin, s = [], 0, 0
    for i in range(q["n"] + 1):
        if i == q["n"] or s + q["rows"][i] > srv.max_rows:
            batches.append((begin, i - begin, s))
            begin, s = i, 0
        if i < q["n"]:
            s += int(q["rows"][i])
    kb = np.zeros(len(batches), rb.K_BATCH_DTYPE)
    slots = 0
    for b, (begin, count, s) in zip(kb, batches):
        padded = min([a for a in srv.padded if a >= s], default=s)
        b["req_begin"], b["n_req"], b["row_base"], b["padded"], b["real"] = begin, count, slots, padded, s
        b["seq_T"] = srv.queue.bucket_len
        slots += padded
    kr = np.zeros(q["n"], rb.K_REQ_DTYPE)
    kr["dense_off"], kr["dense_end"] = q["dense_off"][:-1], q["dense_off"][1:]
    kr["out_off"], kr["n_rows"] = q["out_off"][:-1], q["rows"]
    tokens = 0
    if q["lens"] is not None:
        kr["lens_off"] = q["lens_off"][:-1]
    if q["ids"] is not None:
        kr["ids_off"], kr["ids_end"] = q["ids_off"][:-1], q["ids_off"][1:]
    elif q["lens"] is not None:
        kr["tok_off"] = q["dense_off"][:-1] // q["d_in"][0]
        tokens = int(q["dense_off"][-1] // q["d_in"][0])
    up = lambda a: torch.from_numpy(a.view(np.uint8)).to(DEV)  # noqa: E731
    return up(kb), len(kb), up(kr), slots, tokens


def prepare(case, seed):
    srv, q = _server(case), _requests(case, seed)
    state = dict(srv=srv, entry=case["entry"], q=q)
    if case["entry"] == "serve":
        dense, lens, ids = (q[k].cpu().numpy() for k in ("dense", "lens", "ids"))
        cut = lambda a, o: [a[o[i]:o[i + 1]] for i in range(q["n"])]  # noqa: E731
        state["payloads"] = list(zip(q["rows"].tolist(), cut(dense, q["dense_off"]), cut(lens, q["lens_off"]),
                                     cut(ids, q["ids_off"])))
        return state
    state["out"] = torch.full((int(q["out_off"][-1]),), math.nan, device=DEV)
    torch.cuda.synchronize()
    if case["entry"] == "replay":
        state["call"] = srv.sched.prepare_sim_run(srv.servables, q["servable"], q["arrival"], q["rows"], q["max_len"],
                                                  q["dense"], q["dense_off"], q["lens"], q["lens_off"], q["ids"],
                                                  q["ids_off"], state["out"], q["out_off"])
    else:
        kb, nb, kr, slots, tokens = _group(srv, q)
        n = lambda t: 0 if t is None else t.numel()  # noqa: E731
        state["args"] = (0, kb, nb, kr, q["n"], slots, tokens, q["dense"], n(q["dense"]), q["lens"], n(q["lens"]),
                         q["ids"], n(q["ids"]), state["out"], n(state["out"]),
                         "rb_run_group" if case["entry"] == "group" else "rb_run_group_static")
    return state


def run(state):
    srv = state["srv"]
    if state["entry"] == "replay":
        log = state["call"]()
        return {"out": state["out"], "padded": log["b_padded"], "queue": log["b_queue"], "reqs": log["b_reqs"],
                "done": log["req_done_ns"]}
    if state["entry"] != "serve":
        srv.queue.run_group(*state["args"])
        return {"out": state["out"]}
    srv.now += 1000
    ids = [srv.sched.submit(srv.queue, n, dense, lens, ids, srv.now) for n, dense, lens, ids in state["payloads"]]
    rb.check(rb.lib().rb_flush(srv.queue.h), "rb_flush")
    while srv.sched.run_window() is not None:
        pass
    srv.sched.sync()
    return {"out": np.concatenate([srv.sched.collect(i, p[0], srv.queue.model.d_out)[:, 0]
                                   for i, p in zip(ids, state["payloads"])])}


# ---------------------------------------------------------------- work, tolerance and the 64-bit result

def _flops_bytes(kind, layers, dtype, rows, units, bags):
    """Of `rows` output rows (and `units` rows of the layers) of one model: weights and distinct table rows once."""
    dims = [int(v) for v in layers.split("-")]
    macs = sum(a * b for a, b in zip(dims[:-1], dims[1:]))
    size = 2 if dtype == "bf16" else 4
    flops, nbytes = 2.0 * units * macs, macs * size + 4.0 * sum(dims[1:])
    if kind == "rank":
        mean = (1 + bags) / 2
        p = np.arange(1, TABLE_ROWS + 1, dtype=np.float64) ** -ZIPF
        distinct = float(-np.expm1(rows * mean * np.log1p(-p / p.sum())).sum())
        flops += rows * TABLES * mean * EMB
        nbytes += rows * (4 * N_DENSE + TABLES * 4 * (1 + mean) + 4) + TABLES * distinct * EMB * 2
    elif kind == "seq":
        flops += 2.0 * rows * 2 * dims[-1] + units * dims[-1]
        nbytes += units * dims[0] * 4 + rows * 12
    else:
        nbytes += rows * (dims[0] + dims[-1]) * 4
    return flops, nbytes


def work(case):
    rows = case["requests"] * (1 + case["rows"]) / 2
    models = _servables(case)
    p = 1.0 / np.arange(1, len(models) + 1)
    flops = nbytes = 0.0
    for (kind, layers, dtype, _), share in zip(models, p / p.sum()):
        units = rows * share
        if case["kind"] == "seq":
            k = np.arange(1, case["tokens"] + 1, dtype=np.float64)
            units *= float((k * np.log1p(1 / k)).sum() / math.log(case["tokens"] + 1))
        f, b = _flops_bytes(kind, layers, dtype, rows * share, units, case["bags"])
        flops, nbytes = flops + f, nbytes + b
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """fp32 models: sums of up to 1024 fp32 products in another order (2e-7 to 4e-7 off 64 bits, measured). bf16
    models: hidden layers rounded to bf16 after sums in another order, so single roundings flip (2.5e-4 off 64 bits
    with the same rounding points for linear outputs, 5e-5 for a sigmoid's); "max" allows for a row with a flip."""
    if case["kind"] == "tenants":
        return {"rel": 4e-5, "max": 1e-2}
    if case["kind"] == "rank":
        return {"rel": 4e-4, "max": 1e-2}
    return {"rel": 1.2e-3, "max": 2e-2} if case["dtype"] == "bf16" else {"rel": 2e-6, "max": 4e-5}


def _stored(x, dtype):
    """x as the model stores it between layers, held in 64 bits."""
    return x.float().to(torch.bfloat16).double() if dtype == "bf16" else x.float().double()


def _exact_rows(params, dtype, x):
    for i, (W, b, act) in enumerate(params):
        x = x @ _stored(W, dtype).T + b.double()
        if act == "relu":
            x = x.clamp_(min=0)
        if i + 1 < len(params):
            x = _stored(x, dtype)
    return torch.sigmoid(x) if params[-1][2] == "sigmoid" else x


def exact(case, seed):
    q = _requests(case, seed)
    out = torch.empty(int(q["out_off"][-1]), dtype=torch.float64, device=DEV)
    row_req = np.repeat(np.arange(q["n"]), q["rows"])
    within = np.arange(len(row_req)) - np.repeat(np.cumsum(q["rows"]) - q["rows"], q["rows"])
    row_out = q["out_off"][:-1][row_req] + within * q["d_out"][row_req]
    if q["ids"] is not None:
        lens = q["lens"].reshape(-1, TABLES).to(torch.int64)
        bag0 = torch.cumsum(lens.reshape(-1), 0) - lens.reshape(-1)
        rank_of = np.cumsum(np.array([m[0] == "rank" for m in _servables(case)])[q["servable"][row_req]]) - 1
    for s, (kind, layers, dtype, wseed) in enumerate(_servables(case)):
        params, tables, head = _params(kind, layers, wseed)
        if kind == "seq":
            tokens = q["dense"].reshape(-1, int(layers.split("-")[0]))
            seq_of = torch.repeat_interleave(torch.arange(len(row_req), device=DEV), q["lens"].to(torch.int64))
            pooled = torch.zeros(len(row_req), params[-1][0].shape[0], dtype=torch.float64, device=DEV)
            for a in range(0, tokens.shape[0], 1 << 18):
                y = _exact_rows(params, dtype, tokens[a:a + (1 << 18)].double())
                pooled.index_add_(0, seq_of[a:a + (1 << 18)], y)
            z = pooled / q["lens"].double()[:, None] @ head[0].double().T + head[1].double()
            out.view(-1, 2)[:] = torch.softmax(z, 1)
            continue
        sel = np.nonzero(q["servable"][row_req] == s)[0]
        width, d_out = (N_DENSE if kind == "rank" else int(layers.split("-")[0])), int(layers.split("-")[-1])
        src = q["dense_off"][:-1][row_req[sel]] + within[sel] * width
        if kind == "rank" and len(sel):
            flat = _stored(tables, dtype).reshape(-1, EMB)
        for a in range(0, len(sel), 1 << 15):
            at = torch.from_numpy(src[a:a + (1 << 15)]).to(DEV)[:, None] + torch.arange(width, device=DEV)
            x = _stored(q["dense"][at], dtype)
            if kind == "rank":
                rr = torch.from_numpy(rank_of[sel[a:a + (1 << 15)]]).to(DEV)
                L = lens[rr].reshape(-1)
                first = bag0.reshape(-1, TABLES)[rr].reshape(-1)
                ends = torch.cumsum(L, 0)
                pos = torch.repeat_interleave(first - (ends - L), L) + torch.arange(int(ends[-1]), device=DEV)
                table_of = torch.repeat_interleave(torch.arange(TABLES, device=DEV).repeat(len(rr)), L)
                bags = torch.nn.functional.embedding_bag(table_of * TABLE_ROWS + q["ids"][pos].to(torch.int64), flat,
                                                         ends - L, mode="sum")
                x = torch.cat([_stored(bags, dtype).reshape(len(rr), -1), x], 1)
            y = _exact_rows(params, dtype, x)
            o = torch.from_numpy(row_out[sel[a:a + (1 << 15)]]).to(DEV)[:, None] + torch.arange(d_out, device=DEV)
            out[o] = y
    return {"out": out, "padded": None, "queue": None, "reqs": None, "done": None} if case["entry"] == "replay" else {
        "out": out.cpu().numpy() if case["entry"] == "serve" else out}
