"""The calls a program of this library spends its time in, for timing.

Four kinds of data, the shapes of the library's workloads: a Gaussian mixture
in fp32, ReLU-like embeddings in bf16, genome reads as sets of 64-bit 20-gram
items, and URL-like strings as sets of 32-bit 3-gram items.  Six operations on
them: batched queries (from device memory, or one call from host memory),
queries given as raw text, queries at a fixed threshold, a burst of served
requests of two families, index builds, and streams of inserts.

Every output is a whole number (point ids, counts, sizes) decided by exact
hashing and counting, so there is no floating result to compare with a more
exact one, and no `exact` here.
"""
import math

import numpy as np
import torch

import paper_2106_11565_amd as flinng

FAMILY = {"gmm": flinng.SRP_F32, "relu": flinng.SRP_BF16, "reads": flinng.MINHASH_U64,
          "urls": flinng.MINHASH_U32}
SEED = 0x5EEDF1A7          # of the hash functions and groups
READ_LEN, READ_GRAM = 100, 20
URL_MIN, URL_MAX, URL_EDITS, URL_ALPHABET, URL_GRAM = 20, 120, 5, 40, 3


def _case(name, op, data, N, K, L, R, B, nq, k=10, d=0, bits=0, **more):
    c = {"op": op, "data": data, "N": N, "d": d, "K": K, "L": L, "R": R, "B": B, "bits": bits,
         "nq": nq, "k": k}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # an interactive lookup: one vector from host memory, the answer back in
        # host memory; nothing but launches, copies and waits
        _case("one_query_host_f32", "host_query", "gmm", 10_000, 8, 4, 3, 100, 1, d=128),
        # a batch of fp32 embeddings of a common width (the fp32 hashing path)
        _case("query_f32_768", "query", "gmm", 100_000, 16, 48, 4, 1024, 4096, d=768),
        # the benchmark's ReLU embeddings: 10,000 queries at the tuned (K, L)
        _case("query_relu_bf16", "query", "relu", 1_000_000, 24, 12, 8, 8192, 10_000, d=4096),
        # a small batch that wants many neighbours of each query (re-ranking),
        # with a width that no vector load divides
        _case("query_bf16_d1000_k100", "query", "relu", 200_003, 16, 64, 4, 4093, 517, k=100, d=1000),
        # the benchmark's genome reads: 10,000 item sets at the tuned (K, L)
        _case("query_reads_u64", "query", "reads", 1_000_000, 1, 12, 4, 4096, 10_000, bits=20),
        # the benchmark's URL strings: 10,000 item sets through the persistent grid
        _case("query_urls_u32", "query", "urls", 5_000_000, 3, 48, 8, 16384, 10_000, bits=22,
              persistent=True),
        # raw reads queried without any host preprocessing, an odd count of them,
        # at the configured (K, L)
        _case("query_reads_text", "text", "reads", 1_000_000, 2, 32, 4, 4096, 7_777, bits=20),
        # the fixed-threshold query (Algorithm 2)
        _case("threshold_reads", "threshold", "reads", 1_000_000, 1, 12, 4, 4096, 10_000, k=64,
              bits=20, t=6),
        # the benchmark's burst of mixed requests of 1..512 queries through one
        # server, inputs and results in device memory
        _case("serve_mixed", "serve", "relu", 1_000_000, 24, 12, 8, 8192, 10_000, d=4096, most=512,
              reads=1_000_000),
        # the one-pass builds: bf16 embeddings, and raw strings
        _case("build_relu_bf16", "build", "relu", 1_000_000, 24, 12, 8, 8192, 1000, d=4096),
        _case("build_urls_text", "build_text", "urls", 5_000_000, 3, 48, 8, 16384, 1000, bits=22),
        # sequencer data arriving: a built index, then batches of new reads
        _case("stream_reads", "stream", "reads", 900_000, 1, 12, 4, 4096, 1000, bits=20, batches=3,
              per=10_000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["query", "query", "query", "host_query", "text", "threshold", "build",
                     "build_text", "stream", "serve"])
    if op in ("text", "build_text"):
        data = rng.choice(["reads", "urls"])
    elif op == "stream":
        data = rng.choice(["reads", "urls", "gmm", "relu"])
    elif op == "serve":
        data = "relu"
    else:
        data = rng.choice(["gmm", "relu", "reads", "urls"])
    dense = data in ("gmm", "relu")
    N = _log(rng, 10_000, 400_000 if dense else 2_000_000)
    R = rng.choice([2, 3, 4, 8])
    B = max(16, min(8192 if R == 8 else 16384, int(N / rng.uniform(100, 300))))
    nq = _log(rng, 1, 500 if op == "host_query" else 12_000)
    k = 10 if rng.random() < 0.7 else _log(rng, 1, 500)
    more = {}
    if dense:
        d = _log(rng, 64, 1536 if data == "gmm" else 4096)
        if rng.random() < 0.5:
            d = (d + 31) // 32 * 32
        K, L, bits = rng.randint(8, min(20, int(math.log2(N)) + 3)), rng.randint(4, 64), 0
    else:
        d, bits = 0, rng.randint(14, 22)
        K = rng.choice([1, 1, 2, 2, 3]) if data == "reads" else rng.choice([2, 3, 3])
        L = rng.randint(8, 48)
    if op == "query":
        more["persistent"] = rng.random() < 0.3
    if op == "threshold":
        more["t"] = rng.randint(max(1, L // 3), max(2, L // 2))
        k = rng.choice([16, 64, 256])
    if op in ("build", "build_text", "stream"):
        nq, k = _log(rng, 200, 2000), 10
    if op == "stream":
        more.update(batches=rng.randint(1, 3), per=_log(rng, 100, 20_000))
    if op == "serve":
        more.update(most=_log(rng, 16, 1024), reads=_log(rng, 20_000, 1_000_000))
        nq, k = _log(rng, 1000, 12_000), 10
    return _case(None, op, data, N, K, L, R, B, nq, k=k, d=d, bits=bits, **more)


# ---------------------------------------------------------------------------
# inputs, made on the GPU from the seed

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _rand_rows(rows, d, g, chunk):
    for s in range(0, rows, chunk):
        n = min(chunk, rows - s)
        yield s, n, torch.randn((n, d), generator=g, device="cuda")


def _dense(data, N, d, nq, g):
    """Points and queries: a Gaussian mixture (fp32), or ReLU embeddings (bf16
    bit patterns) whose coordinates are zero off their centre's support."""
    nc = max(2, N // 100)
    centres = torch.randn((nc, d), generator=g, device="cuda")
    if data == "relu":
        keep = torch.rand((nc, d), generator=g, device="cuda") >= 0.6
        centres = centres.abs_().mul_(keep)
    of = torch.randint(0, nc, (N,), generator=g, device="cuda")
    X = torch.empty((N, d), device="cuda", dtype=torch.float32 if data == "gmm" else torch.bfloat16)
    for s, n, z in _rand_rows(N, d, g, max(1, (1 << 27) // d)):
        c = centres[of[s:s + n]]
        v = z.mul_(0.1).add_(c)
        X[s:s + n] = v if data == "gmm" else v.clamp_(min=0).mul_(c > 0)
    base = torch.randint(0, N, (nq,), generator=g, device="cuda")
    z = torch.randn((nq, d), generator=g, device="cuda").mul_(0.05).add_(X[base].float())
    if data == "relu":
        z = z.clamp_(min=0).mul_(centres[of[base]] > 0)
        return X.view(torch.int16), z.to(torch.bfloat16).view(torch.int16)
    return X, z.contiguous()


def _substitute(A, g):
    """1..5 substitutions per row, each to another base."""
    A = A.clone()
    rows = torch.arange(A.shape[0], device="cuda")
    n = torch.randint(1, 6, (A.shape[0],), generator=g, device="cuda")
    for e in range(5):
        at = torch.randint(0, A.shape[1], (A.shape[0],), generator=g, device="cuda")
        by = torch.randint(1, 4, (A.shape[0],), generator=g, device="cuda", dtype=torch.uint8)
        A[rows, at] = torch.where(n > e, (A[rows, at] + by) % 4, A[rows, at])
    return A


def _mix64(v, key):
    def shift(x):
        return (x >> 33) & 0x7FFFFFFF
    v = v ^ key
    v = (v ^ shift(v)) * (0xFF51AFD7ED558CCD - (1 << 64))
    v = (v ^ shift(v)) * (0xC4CEB9FE1A85EC53 - (1 << 64))
    return v ^ shift(v)


def _mix32(v, key):
    v = (v ^ key).to(torch.int32)
    v = (v ^ ((v >> 16) & 0xFFFF)) * (0x85EBCA6B - (1 << 32))
    v = (v ^ ((v >> 13) & 0x7FFFF)) * (0xC2B2AE35 - (1 << 32))
    return v ^ ((v >> 16) & 0xFFFF)


def _read_text(A):
    offs = torch.arange(0, A.numel() + 1, READ_LEN, device="cuda", dtype=torch.int64)
    return A.reshape(-1).contiguous(), offs


def _read_items(A, key):
    W = READ_LEN - READ_GRAM + 1
    out = torch.empty((A.shape[0], W), device="cuda", dtype=torch.int64)
    for s in range(0, A.shape[0], 1 << 18):
        a = A[s:s + (1 << 18)]
        v = torch.zeros((a.shape[0], W), device="cuda", dtype=torch.int64)
        for j in range(READ_GRAM):
            v = v * 4 + a[:, j:j + W]
        out[s:s + (1 << 18)] = _mix64(v, key)
    return out.reshape(-1), torch.arange(0, out.numel() + 1, W, device="cuda", dtype=torch.int64)


def _reads(N, nq, g):
    """Random reads, a mutated copy of each, and queries mutated afresh."""
    half = (N + 1) // 2
    A = torch.randint(0, 4, (half, READ_LEN), generator=g, device="cuda", dtype=torch.uint8)
    X = torch.cat([A, _substitute(A, g)])[:N].contiguous()
    return X, _substitute(A[torch.randint(0, half, (nq,), generator=g, device="cuda")], g)


def _edit(A, lens, g):
    """1..5 insertions, deletions or substitutions per row of padded symbols."""
    rows, W = A.shape
    cols = torch.arange(W, device="cuda")[None, :]
    r = torch.arange(rows, device="cuda")
    n = torch.randint(1, URL_EDITS + 1, (rows,), generator=g, device="cuda")
    for e in range(URL_EDITS):
        kind = torch.randint(0, 3, (rows,), generator=g, device="cuda")
        kind = torch.where(n > e, kind, 3)
        at = (torch.rand((rows,), generator=g, device="cuda") * lens).long()
        src = cols - ((kind == 0)[:, None] & (cols > at[:, None])).long()
        src += ((kind == 1)[:, None] & (cols >= at[:, None])).long()
        A = torch.gather(A, 1, src.clamp_(0, W - 1))
        new = torch.randint(0, URL_ALPHABET, (rows,), generator=g, device="cuda", dtype=torch.uint8)
        A[r, at] = torch.where((kind == 0) | (kind == 2), new, A[r, at])
        lens = lens + (kind == 0).long() - ((kind == 1) & (lens > URL_GRAM)).long()
    return A, lens


def _url_rows(n, g):
    W = URL_MAX + URL_EDITS + 1
    A = torch.randint(0, URL_ALPHABET, (n, W), generator=g, device="cuda", dtype=torch.uint8)
    return A, torch.randint(URL_MIN, URL_MAX + 1, (n,), generator=g, device="cuda")


def _offsets(lens):
    offs = torch.zeros(lens.numel() + 1, device="cuda", dtype=torch.int64)
    torch.cumsum(lens, 0, out=offs[1:])
    return offs


def _url_text(A, lens):
    keep = torch.arange(A.shape[1], device="cuda")[None, :] < lens[:, None]
    return A[keep]


def _url_items(A, lens, key):
    a = A.int()
    v = (a[:, :-2] * URL_ALPHABET + a[:, 1:-1]) * URL_ALPHABET + a[:, 2:]
    keep = torch.arange(v.shape[1], device="cuda")[None, :] < (lens - 2)[:, None]
    return _mix32(v[keep], key)


def _urls(N, nq, g, key, text):
    """Strings and four edited copies of each; queries edited afresh.  Points
    as text (symbols, offsets) or as item sets; queries as both."""
    parts, lens, qa, ql = [], [], [], []
    nt = (N + 4) // 5
    chunk = 1 << 17
    for s in range(0, nt, chunk):
        n = min(chunk, nt - s)
        A, le = _url_rows(n, g)
        rows, rl = [A], [le]
        for _ in range(4):
            a, b = _edit(A, le, g)
            rows.append(a)
            rl.append(b)
        SA, SL = torch.stack(rows, 1).reshape(5 * n, -1), torch.stack(rl, 1).reshape(-1)
        if s + n == nt:
            SA, SL = SA[:N - 5 * s], SL[:N - 5 * s]
        parts.append(_url_text(SA, SL) if text else _url_items(SA, SL, key))
        lens.append(SL if text else SL - 2)
        pick = torch.randint(0, n, (-(-nq * n // nt) + 1,), generator=g, device="cuda")
        qa.append(A[pick])
        ql.append(le[pick])
    Q, qlen = _edit(torch.cat(qa)[:nq], torch.cat(ql)[:nq], g)
    queries = {"text": (_url_text(Q, qlen), _offsets(qlen)),
               "sets": (_url_items(Q, qlen, key), _offsets(qlen - 2))}
    return (torch.cat(parts), _offsets(torch.cat(lens))), queries


def _tuple_of(case, key):
    if case["data"] == "reads":
        return (READ_GRAM, 4, key)
    return (URL_GRAM, URL_ALPHABET, key)


def _inputs(case, seed, text=False):
    """(points, queries as the index takes them, queries as text, item key)."""
    g = _gen(seed)
    if case["data"] in ("gmm", "relu"):
        X, Q = _dense(case["data"], case["N"], case["d"], case["nq"], g)
        return X, Q, None, 0
    key = int(np.random.default_rng(seed).integers(1, 2**31)) | 1
    if case["data"] == "reads":
        A, QA = _reads(case["N"], case["nq"], g)
        X = _read_text(A) if text else _read_items(A, key)
        return X, _read_items(QA, key), _read_text(QA), key
    X, q = _urls(case["N"], case["nq"], g, key, text)
    return X, q["sets"], q["text"], key


def _params(case):
    return dict(family=FAMILY[case["data"]], K=case["K"], L=case["L"], R=case["R"], B=case["B"],
                seed=SEED, bucket_bits=case["bits"])


def _out(nq, k):
    return (torch.empty((nq, k), device="cuda", dtype=torch.int32),
            torch.empty((nq, k), device="cuda", dtype=torch.int32))


def _slice(q, a, b):
    """Sets a..b of a batch, as device items with host offsets."""
    items, offs = q
    return items[int(offs[a]):int(offs[b])], (offs[a:b + 1] - offs[a])


def _serve_state(case, seed):
    """Two resident indexes and the requests of a burst, the families mixed."""
    rng = np.random.default_rng(seed)
    reads = _case(None, "query", "reads", case["reads"], 1, 12, 4,
                  max(16, min(4096, case["reads"] // 244)), case["nq"], bits=20)
    indexes, reqs, outs = [], [], []
    for slot, c in enumerate((reads, case)):
        X, Q, _, _ = _inputs(c, seed + 7919 * slot)
        indexes.append(flinng.Index(X, **_params(c)))
        del X
        out = _out(case["nq"], case["k"])
        outs.append(out)
        if slot == 0:
            Q = (Q[0], Q[1].cpu().numpy().astype(np.uint64))
        at = 0
        while at < case["nq"]:
            n = int(min(rng.integers(1, case["most"] + 1), case["nq"] - at))
            q = Q[at:at + n] if slot else _slice(Q, at, at + n)
            reqs.append((slot, q, (out[0][at:at + n], out[1][at:at + n])))
            at += n
    order = rng.permutation(len(reqs))
    srv = flinng.Server(indexes, mem_budget=8 << 30, max_inflight=2, max_batch=4096)
    return {"op": "serve", "server": srv, "indexes": indexes, "requests": [reqs[i] for i in order],
            "k": case["k"], "out": outs}


def prepare(case, seed):
    op = case["op"]
    if op == "serve":
        st = _serve_state(case, seed)
        torch.cuda.synchronize()
        return st
    text = op == "build_text"
    X, Q, T, key = _inputs(case, seed, text)
    st = {"op": op, "k": case["k"], "params": _params(case), "q": Q, "out": _out(case["nq"], case["k"])}
    if op in ("build", "build_text"):
        st["data"] = X
        st["text"] = _tuple_of(case, key) if text else None
    elif op == "stream":
        total = case["batches"] * case["per"]
        more = dict(case, N=total, nq=1)
        st["data"] = X
        Y, _, _, _ = _inputs_same_key(more, seed, key)
        st["batches"] = _cut(Y, case["batches"], case["per"])
    else:
        st["index"] = flinng.Index(X, **_params(case))
        st["persistent"] = bool(case.get("persistent", False))
        if op == "text":
            st["q"], st["text"] = T, _tuple_of(case, key)
        if op == "threshold":
            st["t"] = case["t"]
            st["out"] = (st["out"][0], torch.empty(case["nq"], device="cuda", dtype=torch.int32))
        if op == "host_query":
            if case["data"] in ("gmm", "relu"):
                st["q"] = Q.cpu().numpy()
            else:
                st["q"] = (Q[0].cpu().numpy(), Q[1].cpu().numpy().astype(np.uint64))
            if case["data"] != "gmm":
                unsigned = {"relu": np.uint16, "reads": np.uint64, "urls": np.uint32}[case["data"]]
                st["q"] = (st["q"].view(unsigned) if case["data"] == "relu"
                           else (st["q"][0].view(unsigned), st["q"][1]))
    torch.cuda.synchronize()
    return st


def _inputs_same_key(case, seed, key):
    """Later arrivals of the same source: other points, the same item key."""
    g = _gen(seed + 104729)
    if case["data"] in ("gmm", "relu"):
        return _dense(case["data"], case["N"], case["d"], 1, g) + (None, 0)
    if case["data"] == "reads":
        return _read_items(_reads(case["N"], 1, g)[0], key), None, None, key
    return _urls(case["N"], 1, g, key, False)[0], None, None, key


def _cut(Y, batches, per):
    if not isinstance(Y, tuple):
        return [Y[i * per:(i + 1) * per] for i in range(batches)]
    items, offs = Y
    got = []
    for i in range(batches):
        o = offs[i * per:(i + 1) * per + 1]
        got.append((items[int(o[0]):int(o[-1])], (o - o[0]).contiguous()))
    return got


def run(st):
    op, k = st["op"], st["k"]
    if op == "query":
        return st["index"].query(st["q"], k, persistent=st["persistent"], out=st["out"])
    if op == "host_query":
        return st["index"].query(st["q"], k)
    if op == "text":
        return st["index"].query_text(st["q"], st["text"], k, out=st["out"])
    if op == "threshold":
        return st["index"].query_threshold(st["q"], st["t"], k, out=st["out"])
    if op == "serve":
        srv = st["server"]
        tickets = [srv.submit_to(slot, q, k, out)[0] for slot, q, out in st["requests"]]
        for t in tickets:
            srv.wait_done(t)
        return st["out"]
    # a build, its inserts, and the first batch it answers; the index of the
    # pass before makes room for the new one
    if "index" in st:
        st["index"].close()
    ix = flinng.Index(st["data"], text=st.get("text"), **st["params"])
    st["index"] = ix
    for b in st.get("batches", ()):
        ix.insert(b)
    ids, scores = ix.query(st["q"], k, out=st["out"])
    info = ix.info
    return ids, scores, int(info.N), int(info.list_entries)


# ---------------------------------------------------------------------------
def _item_bytes(case, n, text):
    """Bytes of n points or queries."""
    if case["data"] == "gmm":
        return 4.0 * n * case["d"]
    if case["data"] == "relu":
        return 2.0 * n * case["d"]
    if case["data"] == "reads":
        return n * (8.0 + (READ_LEN if text else 8 * (READ_LEN - READ_GRAM + 1)))
    mean = (URL_MIN + URL_MAX) / 2
    return n * (8.0 + (mean if text else 4 * (mean - URL_GRAM + 1)))


def _query_work(case, nq, text=False):
    """Per query: its input, L bucket ranges, the lists of a bucket that holds
    its share of the points, the members of one cell (a word each), and k
    results.  The hyperplanes are read once."""
    N, R, B, L, K = case["N"], case["R"], case["B"], case["L"], case["K"]
    bits = case["bits"] or K
    cell = 2 if R * ((B + 3) // 4 * 4) <= 65536 else 4
    per = L * (8 + cell * R * max(1.0, N / 2.0**bits)) + 4.0 * N / B + 8.0 * case["k"]
    by = _item_bytes(case, nq, text) + nq * per
    dense = case["data"] in ("gmm", "relu")
    return by + (2.0 * K * L * case["d"] if dense else 0), (2.0 * nq * case["d"] * K * L if dense else 0)


def _build_work(case, text=False):
    """The points read once; the lists, offsets, members and their groups
    written once."""
    N, R, B, L, K = case["N"], case["R"], case["B"], case["L"], case["K"]
    rp = 1 << (R - 1).bit_length()
    cell = 2 if R * ((B + 3) // 4 * 4) <= 65536 else 4
    by = (_item_bytes(case, N, text) + float(N) * R * L * cell + 4.0 * L * 2.0**(case["bits"] or K)
          + float(N) * R * (8 + 2 * rp))
    dense = case["data"] in ("gmm", "relu")
    return by, (2.0 * N * case["d"] * K * L if dense else 0)


def work(case):
    op = case["op"]
    by, fl = _query_work(case, case["nq"], op == "text")
    if op == "serve":
        reads = _case(None, "query", "reads", case["reads"], 1, 12, 4,
                      max(16, min(4096, case["reads"] // 244)), case["nq"], bits=20)
        by += _query_work(reads, case["nq"])[0]
    if op in ("build", "build_text", "stream"):
        b, f = _build_work(case, op == "build_text")
        by, fl = by + b, fl + f
    if op == "stream":
        n = case["batches"] * case["per"]
        b, f = _build_work(dict(case, N=n))
        by, fl = by + b, fl + f
    return {"bytes": by, "flops": fl}
