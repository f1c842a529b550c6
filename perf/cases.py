"""What the speed of this framework is judged by: calls that a training program makes, over their real range.

A worker of the word-embedding model spends its life in the training step (its own gradient, then the merged update
with the gradients that arrived), so half of the cases are steps; the others are the calls around it: the gradient
alone, the update alone, the send buffer, a dense model's update, and the two read-outs of a trained model.  Sizes are
those of the five workloads of workload.py where they exist, else odd ones in between.

Inputs are made on the GPU from the seed alone.  A step case walks along its token stream, one mini-batch per pass, and
announces the coming mini-batch as the trainer does; the gradients of its peers are inputs.
"""
import math

import numpy as np
import torch

from paper_2211_10280_amd import binding as B

LR = 0.025
STREAM = 1 << 22          # tokens of the stream that a case holds, at most
DT = {"f32": B.F32, "bf16": B.BF16}


# ---------------------------------------------------------------- cases
def listed():
    def words(name, kind, V, D, dtype, corpus, zipf, w, N, batch, K):
        return {"name": name, "kind": kind, "vocab": V, "dim": D, "dtype": dtype, "corpus": corpus, "zipf": zipf,
                "window": w, "negatives": N, "batch": batch, "peers": K}

    return [
        # the five workloads, one training step each:
        # a small vocabulary and a small mini-batch, one worker: launches and host work are all there is
        words("step_1k", "step", 1_000, 32, "f32", 10_000, 1.0, 2, 5, 64, 0),
        # an ordinary domain vocabulary on four workers
        words("step_50k", "step", 50_000, 128, "f32", 5_000_000, 1.0, 5, 5, 1_024, 3),
        # the headline: a million words, eight workers
        words("step_1m", "step", 1_000_000, 300, "f32", 50_000_000, 1.1, 5, 10, 4_096, 7),
        # few, very unevenly frequent words and a large mini-batch: rows that are hit thousands of times
        words("step_hot", "step", 10_000, 256, "f32", 20_000_000, 1.5, 8, 15, 16_384, 7),
        # the largest: two million words in bfloat16, sixteen workers
        words("step_2m_bf16", "step", 2_000_000, 512, "bf16", 100_000_000, 1.05, 5, 10, 8_192, 15),
        # the headline workload with gradient messages in bfloat16, its own message written too
        words("step_1m_messages", "step_packed", 1_000_000, 300, "f32", 50_000_000, 1.1, 5, 10, 4_096, 7),
        # gradient calculation alone, with the loss, on a mini-batch nobody announced: what a worker with a send
        # buffer (maxGradBuffer > 1) calls; rows of 400 bytes
        words("grad_200k_d100", "grad", 200_000, 100, "f32", 10_000_000, 1.1, 4, 7, 1_500, 0),
        # gradient application alone, few of a large vocabulary's rows touched
        words("apply_4m_bf16", "apply", 4_000_000, 200, "bf16", 100_000_000, 1.05, 5, 5, 4_096, 3),
        # the send buffer: gradients += gradient, then the buffer as a bfloat16 message
        words("buffer_1m", "buffer", 1_000_000, 300, "f32", 50_000_000, 1.1, 5, 10, 4_096, 0),
        # gradient application of a dense model (a convolutional network), eight workers
        {"name": "dense_25m", "kind": "dense", "n": 25_000_003, "dtype": "f32", "peers": 7},
        # predict: the vectors of the words of a batch of short messages
        {"name": "lookup_3k", "kind": "lookup", "vocab": 1_000_000, "dim": 300, "dtype": "f32", "n": 3_000, "zipf": 1.1},
        # how far every word has moved since a snapshot
        {"name": "cosine_1m", "kind": "cosine", "vocab": 1_000_000, "dim": 300, "dtype": "f32"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 8 + ["step_packed", "grad", "grad", "apply", "buffer", "dense", "lookup", "cosine"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    dim = 4 * _log_int(rng, 8, 128)
    if kind == "dense":
        return {"kind": kind, "n": _log_int(rng, 50_000, 100_000_000), "dtype": dtype, "peers": rng.randrange(0, 8)}
    if kind == "lookup":
        return {"kind": kind, "vocab": _log_int(rng, 1_000, 2_000_000), "dim": dim, "dtype": dtype,
                "n": _log_int(rng, 16, 1_000_000), "zipf": round(rng.uniform(1.0, 1.5), 3)}
    if kind == "cosine":
        return {"kind": kind, "vocab": _log_int(rng, 1_000, 2_000_000), "dim": dim, "dtype": dtype}
    c = {"kind": kind, "vocab": _log_int(rng, 1_000, 4_000_000 if kind == "apply" else 2_000_000), "dim": dim,
         "dtype": dtype, "corpus": 0, "zipf": round(rng.uniform(1.0, 1.5), 3), "window": rng.randrange(2, 9),
         "negatives": rng.randrange(3, 16), "batch": _log_int(rng, 48, 8_192),
         "peers": 0 if kind in ("grad", "buffer") else rng.randrange(0, 8)}
    if kind == "apply":
        c["peers"] = max(c["peers"], 1)
    c["corpus"] = 50 * c["vocab"]
    return c


# ---------------------------------------------------------------- inputs
def _zipf_p(V, s):
    p = np.arange(1, V + 1, dtype=np.float64) ** -float(s)
    return p / p.sum()


def _counts(case):
    return np.maximum(np.rint(_zipf_p(case["vocab"], case["zipf"]) * case["corpus"]), 1).astype(np.uint64)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _sample(p, n, g):
    """n draws (int32) from the weights p, by inverse CDF in 64 bits."""
    cdf = torch.cumsum(torch.as_tensor(p, device="cuda", dtype=torch.float64), 0)
    u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
    return torch.searchsorted(cdf, u, right=True).clamp_(max=len(p) - 1).to(torch.int32)


def _tables(case, g, n=2):
    """Trained-looking tables on the row pitch that the trainer uses; padding columns zero."""
    V, D = case["vocab"], case["dim"]
    td = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    stride = B.tensair_aligned_row_stride(D, DT[case["dtype"]])
    out = []
    for _ in range(n):
        w = torch.zeros((V, stride), dtype=td, device="cuda")
        w[:, :D] = torch.randn((V, D), generator=g, device="cuda") * 0.25
        out.append(w)
    return out


def _message(case, counts, g, packed=False):
    """A gradient as it arrives from a peer: the rows a mini-batch of the same distribution touches, every row a sum
    of as many terms as its word was met."""
    V, D, w, N, n = case["vocab"], case["dim"], case["window"], case["negatives"], case["batch"]
    freq = counts.astype(np.float64)
    P = 2 * w * n
    sides = []
    for draws, per in ((_sample(freq, n, g), 2 * w * (N + 1)),
                       (torch.cat([_sample(freq, n + 2 * w, g).repeat_interleave(2 * w)[:P], _sample(freq ** 0.75, P * N, g)]), 1)):
        ids, hits = torch.unique(draws, return_counts=True)
        rows = torch.randn((ids.numel(), D), generator=g, device="cuda")
        rows *= (0.125 / P) * torch.sqrt(hits.float() * per)[:, None]
        sides.append((ids, rows))
    (ids_in, rows_in), (ids_out, rows_out) = sides
    buf = (B.PackedBuffers if packed else B.GradBuffers)(ids_in.numel(), ids_out.numel(), D)
    if packed:
        rows_in, rows_out = (r.to(torch.bfloat16).view(torch.int16) for r in (rows_in, rows_out))
    buf.in_ids.copy_(ids_in)
    buf.out_ids.copy_(ids_out)
    buf.in_rows.copy_(rows_in)
    buf.out_rows.copy_(rows_out)
    buf.n_rows.copy_(torch.tensor([ids_in.numel(), ids_out.numel()], dtype=torch.int32))
    return buf


def _cleared(buf):
    for t in (buf.in_ids, buf.in_rows, buf.out_ids, buf.out_rows):
        t.zero_()
    return buf


def _stream_tokens(case):
    return max(case["batch"] * 64, min(STREAM, case["corpus"])) + 7


class State:
    pass


def prepare(case, seed):
    s = State()
    s.kind = kind = case["kind"]
    g = _gen(seed)
    if kind == "dense":
        td = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        s.theta = (torch.randn(case["n"], generator=g, device="cuda") * 0.1).to(td)
        s.grads = [torch.randn(case["n"], generator=g, device="cuda") * 1e-3 for _ in range(case["peers"] + 1)]
        return s
    if kind == "cosine":
        s.dim = case["dim"]
        s.a = _tables(case, g, 1)[0]
        s.b = (s.a.float() * (1 + 0.1 * torch.randn(s.a.shape, generator=g, device="cuda"))).to(s.a.dtype)
        s.diff = torch.zeros(case["vocab"], device="cuda")
        return s
    if kind == "lookup":
        s.tables = _tables(case, g)
        counts = np.maximum(np.rint(_zipf_p(case["vocab"], case["zipf"]) * 50 * case["vocab"]), 1).astype(np.uint64)
        s.model = B.Model(case["vocab"], case["dim"], DT[case["dtype"]], 5, 5, 64, 0, 7, counts, tables=s.tables,
                          row_stride=s.tables[0].shape[1])
        s.ids = _sample(counts.astype(np.float64), case["n"], g)
        s.out = torch.zeros((case["n"], case["dim"]), device="cuda")
        return s

    counts = _counts(case)
    s.tables = _tables(case, g)
    s.tokens = _sample(counts.astype(np.float64), _stream_tokens(case), g)
    s.model = B.Model(case["vocab"], case["dim"], DT[case["dtype"]], case["window"], case["negatives"], case["batch"],
                      case["peers"], int(seed), counts, tables=s.tables, row_stride=s.tables[0].shape[1])
    s.batch, s.peers_n = case["batch"], case["peers"]
    s.t, s.announced = 0, -1
    if kind in ("step", "step_packed", "grad"):
        s.own = _cleared(s.model.grad_buffers())
        s.peers = [_message(case, counts, g, packed=kind == "step_packed") for _ in range(case["peers"])]
        if kind == "step_packed":
            s.msg = _cleared(s.model.packed_buffers())
        if kind == "grad":
            s.loss = torch.zeros(1, device="cuda")
    elif kind == "apply":
        s.own = _message(case, counts, g)
        s.peers = [_message(case, counts, g) for _ in range(case["peers"])]
    else:
        s.sum_a, s.sum_b = _message(case, counts, g), _message(case, counts, g)
        own = s.model.cfg          # room for two mini-batches, as the trainer's send buffer has
        cap = [min(case["vocab"], 2 * f(own, case["batch"])) for f in (B.tensair_capacity_in, B.tensair_capacity_out)]
        s.sum = _cleared(B.GradBuffers(*cap, case["dim"]))
        s.msg = _cleared(B.PackedBuffers(*cap, case["dim"]))
    return s


# ---------------------------------------------------------------- one pass
def _batch(s, t):
    """Mini-batches are dealt round-robin to the workers; the stream is iterated again with the next epoch."""
    per_epoch = s.tokens.numel() // s.batch
    epoch, j = divmod(t * (s.peers_n + 1), per_epoch)
    return j * s.batch, s.batch, epoch % 65536


def _grad_out(buf, bf16=False):
    rows = (lambda r: r.view(torch.bfloat16)) if bf16 else (lambda r: r)
    return {"n": buf.n_rows, "in_ids": buf.in_ids, "in_rows": rows(buf.in_rows), "out_ids": buf.out_ids,
            "out_rows": rows(buf.out_rows)}


def run(s):
    kind = s.kind
    if kind == "dense":
        B.tensair_dense_apply(s.theta, s.grads, LR)
        return s.theta
    if kind == "cosine":
        B.tensair_cosine_difference(s.a, s.b, s.dim, s.diff)
        return s.diff
    if kind == "lookup":
        s.model.lookup(0, s.ids, s.out)
        return s.out
    if kind == "apply":
        s.model.dasgd_apply(s.own, s.peers, LR)
        return s.tables
    if kind == "buffer":
        s.model.grad_add(s.sum_a, s.sum_b, s.sum)
        s.model.grad_pack(s.sum, s.msg)
        return {"sum": _grad_out(s.sum), "message": _grad_out(s.msg, bf16=True)}
    begin, n, epoch = _batch(s, s.t)
    if kind == "grad":
        s.model.sgns_grad(s.tokens, begin, n, epoch, s.own, mean_loss=s.loss)
        s.t += 1
        return {"own": _grad_out(s.own), "loss": s.loss}
    if s.announced == s.t:
        s.announced = s.t + 1
        s.model.prefetch(s.tokens, *_batch(s, s.announced))
    if kind == "step":
        s.model.step(s.tokens, begin, n, epoch, s.peers, LR, s.own)
    else:
        s.model.step_packed(s.tokens, begin, n, epoch, s.peers, LR, s.own, s.msg)
    s.t += 1
    if s.announced < s.t:
        s.announced = s.t
        s.model.prefetch(s.tokens, *_batch(s, s.announced))
    out = {"own": _grad_out(s.own), "w_in": s.tables[0], "w_out": s.tables[1]}
    if kind == "step_packed":
        out["message"] = _grad_out(s.msg, bf16=True)
    return out


# ---------------------------------------------------------------- what a pass cannot do without
def _rows(case, times):
    """Expected rows of W_in and W_out that `times` mini-batches touch together."""
    freq = _counts(case).astype(np.float64)
    noise = freq ** 0.75
    p, q = freq / freq.sum(), noise / noise.sum()
    w, N, n = case["window"], case["negatives"], case["batch"]
    gone_in = np.exp(times * n * np.log1p(-p))
    gone_out = np.exp(times * ((n + 2 * w) * np.log1p(-p) + 2 * w * n * N * np.log1p(-q)))
    return float((1 - gone_in).sum()), float((1 - gone_out).sum())


def work(case):
    kind = case["kind"]
    e = 4 if case["dtype"] == "f32" else 2
    if kind == "dense":
        return {"bytes": case["n"] * (2 * e + 4 * (case["peers"] + 1)), "flops": case["n"] * (case["peers"] + 2)}
    if kind == "cosine":
        return {"bytes": case["vocab"] * (2 * case["dim"] * e + 4), "flops": 6 * case["vocab"] * case["dim"]}
    if kind == "lookup":
        return {"bytes": case["n"] * (case["dim"] * (e + 4) + 4), "flops": case["n"]}
    D, K = case["dim"], case["peers"]
    one = sum(_rows(case, 1))
    occurrences = 2 * case["window"] * case["batch"] * (case["negatives"] + 1)
    if kind == "grad":
        return {"bytes": one * D * (e + 4), "flops": 6 * D * occurrences}
    if kind == "buffer":
        both = sum(_rows(case, 2))
        return {"bytes": (2 * one * 4 + both * (4 + 2)) * D, "flops": both * D}
    union = sum(_rows(case, K + 1))
    pe = 2 if kind == "step_packed" else 4
    update = 2 * union * D * e + K * one * D * pe
    if kind == "apply":
        return {"bytes": update + one * D * 4, "flops": (K + 2) * one * D}
    # a step writes its own gradient (and its message) and reads what arrived; its rows of the tables are read once
    own = one * D * (4 + (2 if kind == "step_packed" else 0))
    return {"bytes": update + own, "flops": 6 * D * occurrences + (K + 2) * one * D}


def tolerance(case):
    kind = case["kind"]
    if kind in ("lookup", "buffer"):
        return "exact"             # a copy; sums of two numbers, rounded once
    if kind == "cosine":
        return {"rel": 6e-5}       # 1 - cos of rows that have hardly moved: the rounding of cos against a few thousandths
    if case["dtype"] == "bf16" or kind == "step_packed":
        # an element whose fp32 value lands on the other side of a rounding boundary is one bfloat16 step (2^-7) off;
        # few do (sums agree to 1e-7)
        return {"rel": 1e-4, "max": 1.6e-2}
    return {"rel": 1e-6, "max": 1e-5} if kind in ("dense", "apply") else {"rel": 2e-6, "max": 4e-4}


# ---------------------------------------------------------------- the same in 64 bits
_M32 = np.uint64(0xFFFFFFFF)


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 (Salmon et al., SC'11) over arrays of counters: the first two words."""
    c0, c1, c2, c3 = (np.asarray(c, dtype=np.uint64) for c in (c0, c1, c2, c3))
    for _ in range(10):
        a, b = np.uint64(0xD2511F53) * c0, np.uint64(0xCD9E8D57) * c2
        s = np.uint64(32)
        c0, c1, c2, c3 = (b >> s) ^ c1 ^ np.uint64(k0), b & _M32, (a >> s) ^ c3 ^ np.uint64(k1), a & _M32
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c0, c1


def _alias(counts):
    """Vose's table of count^0.75, work lists in ascending order and consumed from the back."""
    prob = np.array([math.pow(float(c), 0.75) for c in counts])
    prob = prob * float(len(prob)) / np.cumsum(prob)[-1]
    lo, hi = np.flatnonzero(prob < 1).tolist(), np.flatnonzero(prob >= 1).tolist()
    thr, alias, q = [0xFFFFFFFF] * len(prob), list(range(len(prob))), prob.tolist()
    while lo and hi:
        poor, rich = lo.pop(), hi.pop()
        thr[poor] = min(int(q[poor] * 4294967296.0), 0xFFFFFFFF)
        alias[poor] = rich
        q[rich] = (q[rich] + q[poor]) - 1.0
        (lo if q[rich] < 1 else hi).append(rich)
    return np.array(thr, dtype=np.uint64), np.array(alias, dtype=np.int64)


def _occurrences(case, counts, tokens, seed):
    """Centers, and every center's contexts and negatives, of the stream's first mini-batch: center word, out word and
    label of every occurrence, and the number of pairs."""
    w, N, n, V = case["window"], case["negatives"], case["batch"], case["vocab"]
    tok = tokens[: n + w].cpu().numpy().astype(np.int64)
    pos = np.repeat(np.arange(n), 2 * w)
    q = np.tile(np.arange(2 * w), n)
    ctx = pos + np.where(q < w, q - w, q - w + 1)
    ok = (ctx >= 0) & (ctx < len(tokens))
    pos, q, ctx = pos[ok], q[ok], ctx[ok]
    thr, alias = _alias(counts)
    slot = np.arange(N)
    r0, r1 = _philox(np.repeat(pos, N), 0, (q[:, None] * 65536 + slot).reshape(-1), 0, seed & 0xFFFFFFFF, seed >> 32)
    bucket = ((r0 * np.uint64(V)) >> np.uint64(32)).astype(np.int64)
    neg = np.where(r1 < thr[bucket], bucket, alias[bucket]).reshape(-1, N)
    out = np.concatenate([tok[ctx][:, None], neg], axis=1)
    label = np.zeros(out.shape)
    label[:, 0] = 1
    to = lambda x, d: torch.as_tensor(x, device="cuda", dtype=d)  # noqa: E731
    center = np.repeat(tok[pos], N + 1)
    return to(center, torch.int64), to(out.reshape(-1), torch.int64), to(label.reshape(-1), torch.float64), len(pos)


def _gradient64(case, s, seed):
    """Row ids and rows of both tables, and the mean loss."""
    D = case["dim"]
    c, u, label, P = _occurrences(case, _counts(case), s.tokens, int(seed))
    ids_in, at_in = torch.unique(c, return_inverse=True)
    ids_out, at_out = torch.unique(u, return_inverse=True)
    rows_in = torch.zeros((ids_in.numel(), D), dtype=torch.float64, device="cuda")
    rows_out = torch.zeros((ids_out.numel(), D), dtype=torch.float64, device="cuda")
    loss = 0.0
    for lo in range(0, c.numel(), 1 << 18):
        k = slice(lo, lo + (1 << 18))
        v, x = s.tables[0][c[k], :D].double(), s.tables[1][u[k], :D].double()
        dot = (v * x).sum(1)
        g = ((torch.sigmoid(dot) - label[k]) / P)[:, None]
        loss += float(torch.nn.functional.softplus(torch.where(label[k] > 0, -dot, dot)).sum())
        rows_in.index_add_(0, at_in[k], g * x)
        rows_out.index_add_(0, at_out[k], g * v)
    return (ids_in, rows_in), (ids_out, rows_out), loss / P


def _laid_out(rows, like):
    full = torch.zeros(like.shape, dtype=torch.float64, device="cuda")
    full[: rows.shape[0]] = rows
    return full


def exact(case, seed):
    kind = case["kind"]
    s = prepare(case, seed)
    if kind == "dense":
        return s.theta.double() - LR * sum(g.double() for g in s.grads)
    if kind == "cosine":
        a, b = s.a.double(), s.b.double()
        return 1 - (a * b).sum(1) / (a.norm(dim=1) * b.norm(dim=1))
    if kind == "lookup":
        return s.tables[0][s.ids.long(), : case["dim"]].double()
    D = case["dim"]
    if kind == "buffer":
        out = {"n": None, "in_ids": None, "out_ids": None}
        for side in ("in", "out"):
            total = torch.zeros((case["vocab"], D), dtype=torch.float64, device="cuda")
            hit = torch.zeros(case["vocab"], dtype=torch.bool, device="cuda")
            for m in (s.sum_a, s.sum_b):
                ids = getattr(m, side + "_ids").long()
                total[ids] += getattr(m, side + "_rows").double()
                hit[ids] = True
            out[side + "_rows"] = _laid_out(total[hit], getattr(s.sum, side + "_rows"))
        return {"sum": out, "message": out}
    lr = float(np.float32(LR))
    own = None
    if kind != "apply":
        own = _gradient64(case, s, seed)
        grad = {"n": None, "in_ids": None, "in_rows": _laid_out(own[0][1], s.own.in_rows), "out_ids": None,
                "out_rows": _laid_out(own[1][1], s.own.out_rows)}
        if kind == "grad":
            return {"own": grad, "loss": torch.tensor([own[2]], dtype=torch.float64)}
    tables = []
    for side, w in (("in", s.tables[0]), ("out", s.tables[1])):
        new = w.double()
        got = [(getattr(m, side + "_ids"), getattr(m, side + "_rows")) for m in s.peers + ([s.own] if own is None else [])]
        for ids, rows in got:
            rows = rows.view(torch.bfloat16) if rows.dtype == torch.int16 else rows
            new[:, :D].index_add_(0, ids.long(), -lr * rows.double())
        if own is not None:
            ids, rows = own[0] if side == "in" else own[1]
            new[:, :D].index_add_(0, ids, -lr * rows)
        tables.append(new)
    if kind == "apply":
        return tables
    out = {"own": grad, "w_in": tables[0], "w_out": tables[1]}
    if kind == "step_packed":
        out["message"] = grad
    return out
