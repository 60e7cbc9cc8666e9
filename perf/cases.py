"""Timed work of the replay buffer: what its users have it do, through the public Python entry points.

A *case* is a dict of plain values.  ``prepare`` builds the buffer a training program holds (filled, with its input
batches resident on the GPU), ``run`` is one pass of that program's loop, ``work`` the bytes and operations such a pass
cannot do without.  Every state keeps several input batches and takes them in turn, as a program whose batches differ
from iteration to iteration; results go to arrays the program keeps.

Forms (``"form"``):
  step     one iteration of a training loop in one call: new rows in, a batch out, that batch's priorities back
           (``PrioritizedReplay.step``, with ``insert=`` where the case inserts)
  graph    several such iterations captured once as a HIP graph and replayed (no insertion: that is host state)
  apart    ``sample`` with the rows, then, when the learner is through, ``update`` of that batch
  earlier  ``sample`` with the rows and, in the same call, the priorities of the batch drawn in the pass before
  td       ``sample`` with weights relative to the whole buffer, then ``update_td`` from temporal-difference errors
  fill     a chunk of many rows with given priorities (initial fill, demonstrations), then a first batch
  steps    a list of iterations in one launch on an on-chip tree (``run_steps``)
  queue    the same as a queue of op-coded requests (``run_requests``)
"""
from __future__ import annotations

import math

import torch

from paper_2311_09445_amd.per import OP_INSERT, OP_SAMPLE, OP_UPDATE, PrioritizedReplay

# Row layouts (bytes per field): classic control, frame indices, 17-float states, one packed row, two 84 x 84 frames.
CONTROL = "16,4,4,16,1"
FRAME_INDEX = "16,4,4,1"
STATES = "68,24,4,68,1"
PACKED = "128"
FRAMES = "7056,4,4,7056,1"

BASE = {"T": 1, "insert": 0, "iterations": 1, "positions": False, "rng": False, "beta": 0.4, "batches": 8}


def _case(name, form, **kw):
    c = dict(BASE, form=form, **kw)
    c.setdefault("filled", c["N"])
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest buffer and batch: a classic-control agent with a binary tree, four environments stepping.
        _case("control_step", "step", K=2, N=4096, B=64, insert=4, fields=CONTROL, prio="uniform"),
        # A deep Q-network with a million frame-index rows, not yet full: a small batch on a large tree.
        _case("dqn_step", "step", K=16, N=1 << 20, filled=700_001, B=32, insert=4, fields=FRAME_INDEX, prio="lognormal"),
        # An actor-critic with float states, a large batch, uniforms drawn by the library.
        _case("ddpg_step", "step", K=16, N=1 << 20, B=4096, insert=1, fields=STATES, prio="exponential", rng=True),
        # The largest tree with the metric's batch; a tenth of the update slots aim at another slot's leaf.
        _case("stress_graph", "graph", K=32, N=1 << 24, B=65536, fields=PACKED, prio="pareto", positions=True, iterations=8, batches=1),
        # Many independent buffers side by side: parallel actor-learners.
        _case("buffers_step", "step", K=16, N=1 << 18, T=64, B=1024, insert=16, fields=STATES, prio="uniform", rng=True, batches=4),
        # Thousands of environments stepped together: many new rows for every learner batch.
        _case("vector_step", "step", K=16, N=1 << 20, B=16384, insert=4096, fields=STATES, prio="exponential"),
        # A learner that hands back the priorities one batch late; nothing here is a power of two.
        _case("earlier_odd", "earlier", K=8, N=1_000_000, filled=900_001, B=10_007, fields=STATES, prio="exponential", beta=0.7),
        # A learner that takes very large batches, sampling and updating in separate calls.
        _case("large_apart", "apart", K=32, N=1 << 24, B=1 << 20, fields=PACKED, prio="pareto", batches=3),
        # Image observations stored whole, weights relative to the buffer, priorities from temporal-difference errors.
        _case("frames_td", "td", K=64, N=100_000, filled=80_000, B=512, fields=FRAMES, prio="lognormal", rng=True, beta=0.6),
        # Filling a large buffer, a chunk of 2^20 rows at a time.
        _case("fill_chunk", "fill", K=32, N=1 << 24, B=4096, insert=1 << 20, fields=PACKED, prio="pareto", batches=2),
        # The paper's example buffer and smaller batch, a hundred iterations handed over at once.
        _case("onchip_steps", "steps", K=16, N=10_000, B=32, insert=4, fields=CONTROL, prio="uniform", iterations=100, batches=2),
        # The larger batch of the paper as a queue of requests.
        _case("onchip_queue", "queue", K=16, N=30_000, B=512, insert=16, fields=CONTROL, prio="uniform", iterations=20, batches=2),
    ]


def _spread(rng, lo, hi):
    """A whole number from lo to hi, even over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _size(rng, lo, hi):
    """As _spread, now and then a power of two, as programs like to choose them."""
    n = _spread(rng, lo, hi)
    return max(lo, min(hi, 1 << int(round(math.log2(n))))) if rng.random() < 0.35 else n


def draw(rng):
    form = rng.choice(["step", "step", "step", "graph", "earlier", "apart", "td", "fill", "steps", "queue"])
    kw = {"prio": rng.choice(["uniform", "lognormal", "exponential", "pareto"]), "beta": round(rng.uniform(0.3, 1.0), 3)}
    if form in ("steps", "queue"):
        K = rng.choice([2, 4, 8, 16, 32])
        N = _size(rng, 1000, {2: 16_000, 4: 20_000, 8: 24_000}.get(K, 100_000))
        B = _size(rng, 16, 512)
        kw.update(K=K, N=N, B=B, insert=rng.choice([0, 1, 4, 16]), T=rng.choice([1, 1, 1, 4]), batches=2,
                  iterations=_spread(rng, 10, 100) if B <= 128 else _spread(rng, 5, 25), fields=rng.choice([CONTROL, FRAME_INDEX]))
    elif form == "fill":
        K, N = rng.choice([16, 32, 64]), _size(rng, 1 << 19, 1 << 24)
        fields = rng.choice([PACKED, STATES, FRAME_INDEX])
        kw.update(K=K, N=N, B=_size(rng, 256, 4096), insert=_size(rng, 1 << 14, min(N, 800_000 if fields == STATES else 1 << 20)),
                  batches=2, fields=fields)
    elif form in ("apart", "graph"):
        K, N = rng.choice([16, 32, 64]), _size(rng, 1 << 20, 1 << 24)
        B = _size(rng, 1 << 13, 1 << 20) if form == "apart" else _size(rng, 1 << 11, 1 << 16)
        kw.update(K=K, N=N, B=B, fields=PACKED, positions=form == "graph" and rng.random() < 0.5,
                  iterations=8 if form == "graph" else 1, batches=1 if form == "graph" else 3)
    elif form == "td":
        fields = rng.choice([FRAMES, STATES, CONTROL])
        N = _size(rng, 20_000, 100_000) if fields == FRAMES else _size(rng, 20_000, 1 << 20)
        kw.update(K=rng.choice([16, 32, 64]), N=N, B=_size(rng, 32, 1024 if fields == FRAMES else 8192), fields=fields, rng=True)
    elif form == "earlier":
        kw.update(K=rng.choice([8, 16, 32]), N=_size(rng, 50_000, 1 << 22), B=_size(rng, 64, 1 << 16), fields=rng.choice([STATES, PACKED]))
    else:
        T = rng.choice([1, 1, 1, 4, 16, 64])
        K = rng.choice([2, 4, 8, 16, 16, 32, 64])
        N = _size(rng, 4096, {1: 1 << 22, 4: 1 << 20, 16: 1 << 19, 64: 1 << 18}[T])
        B = _size(rng, 32, {1: 1 << 16, 4: 8192, 16: 4096, 64: 1024}[T])
        B = min(B, N)
        kw.update(K=K, N=N, T=T, B=B, insert=min(N // 4, rng.choice([0, 1, 4, 16, _spread(rng, 64, max(64, B))])),
                  rng=rng.random() < 0.5, positions=rng.random() < 0.15, batches=4,
                  fields=rng.choice([CONTROL, FRAME_INDEX, STATES, STATES, PACKED]))
    filled = kw["N"] if rng.random() < 0.6 else int(kw["N"] * rng.uniform(0.5, 1.0))
    return _case(None, form, **dict(kw, filled=max(1, filled)))


# ------------------------------------------------------------------------------------------------------------ inputs
def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * (seed + 1) + stream)
    return g


def _priorities(dist, shape, g):
    x = torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)
    if dist == "uniform":
        x = 1.0 - 0.999 * x
    elif dist == "exponential":
        x = -torch.log1p(-x)
    elif dist == "lognormal":
        x = torch.exp(torch.randn(shape, generator=g, device="cuda", dtype=torch.float64))
    else:   # pareto, one row in a hundred without priority
        zero = torch.rand(shape, generator=g, device="cuda") < 0.01
        x = ((1.0 - x) ** (-1.0 / 1.5)).masked_fill_(zero, 0.0)
    return x.float()


def _td_errors(shape, g):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _new_priorities(shape, g):
    """(|td| + eps)^0.6 in double, rounded once: what a learner writes back."""
    return ((_td_errors(shape, g).double().abs() + 1e-6) ** 0.6).float()


def _uniforms(shape, g):
    return torch.randint(0, 1 << 24, shape, generator=g, device="cuda", dtype=torch.int32).float() * 2.0 ** -24


def _rows(shape, widths, g):
    out = []
    for b in widths:
        n = math.prod(shape) * b
        words = torch.randint(-(1 << 31), (1 << 31) - 1, ((n + 3) // 4,), generator=g, device="cuda", dtype=torch.int32)
        out.append(words.view(torch.uint8)[:n].view(*shape, b))
    return out


def _positions(shape, g):
    """Position map: element j goes to the leaf of sample j, but for a tenth of them, which aim at another sample's."""
    B = shape[-1]
    pos = torch.arange(B, device="cuda", dtype=torch.int32).expand(shape).contiguous()
    other = torch.randint(0, B, shape, generator=g, device="cuda", dtype=torch.int32)
    return torch.where(torch.rand(shape, generator=g, device="cuda") < 0.1, other, pos)


def _widths(case):
    return tuple(int(b) for b in case["fields"].split(",") if b)


class _State:
    pass


def prepare(case, seed):
    K, N, T, B, n, S = (case[k] for k in ("K", "N", "T", "B", "insert", "iterations"))
    widths = _widths(case)
    s = _State()
    s.form, s.beta, s.n, s.B, s.turn = case["form"], case["beta"], n, B, 0
    s.buf = buf = PrioritizedReplay(K, N, T, widths)
    if case["rng"]:
        buf.set_rng(seed + 12345)
    if s.form == "td":
        buf.set_weight_norm("buffer")
    g = _gen(seed, 1)
    chunk = max(1, min(1 << 20, (1 << 28) // max(1, T * sum(widths))))
    for lo in range(0, case["filled"], chunk):
        m = min(chunk, case["filled"] - lo)
        buf.insert(m, _rows((T, m), widths, g), _priorities(case["prio"], (T, m), g))
    g = _gen(seed, 2)
    f32, i32, u8 = torch.float32, torch.int32, torch.uint8
    new = lambda *shape, dtype: torch.empty(shape, dtype=dtype, device="cuda")  # noqa: E731
    listed_form = s.form in ("graph", "steps", "queue")       # these take a list of iterations per pass
    lead = (S, T) if listed_form else (T,)
    s.sets = []
    for _ in range(case["batches"]):
        b = _State()
        b.u = None if case["rng"] else _uniforms((*lead, B), g)
        b.prio = _td_errors((*lead, B), g) if s.form == "td" else _new_priorities((*lead, B), g)
        b.pos = _positions((*lead, B), g) if case["positions"] else None
        b.rows = _rows((*lead, n), widths, g) if n else None
        b.row_prio = _priorities(case["prio"], (T, n), g) if s.form == "fill" else None
        s.sets.append(b)
    s.idx = [new(*lead, B, dtype=i32) for _ in range(2)]      # two: the form `earlier` still needs the last batch's
    s.weight, s.value = new(*lead, B, dtype=f32), new(*lead, B, dtype=f32)
    s.rows = [new(*lead, B, w, dtype=u8) for w in widths]
    s.slots = new(T, n, dtype=i32) if s.form == "fill" else None
    s.betas = torch.full((S,), s.beta, dtype=f32, device="cuda")
    if s.form == "earlier":     # the batch whose priorities the first pass brings back
        buf.sample(s.sets[-1].u, s.beta, out_idx=s.idx[1], out_weight=s.weight, out_prio=s.value)
    elif s.form == "queue":
        for b in s.sets:
            q = []
            for i in range(S):
                if n:
                    q.append({"op": OP_INSERT, "n": n, "rows": [r[i] for r in b.rows]})
                q.append({"op": OP_SAMPLE, "u": b.u[i], "beta": s.beta, "idx": s.idx[0][i], "out_weight": s.weight[i],
                          "out_prio": s.value[i], "rows": [r[i] for r in s.rows]})
                q.append({"op": OP_UPDATE, "prio": b.prio[i]})
            b.queue = buf.prepare_requests(q)
    elif s.form == "graph":
        b = s.sets[0]

        def iterations():
            for i in range(S):
                buf.step(b.u[i], s.beta, b.prio[i], None if b.pos is None else b.pos[i], out_idx=s.idx[0][i],
                         out_weight=s.weight[i], out_prio=s.value[i], rows_out=[r[i] for r in s.rows])

        torch.cuda.synchronize()
        s.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s.graph):
            iterations()
    return s


# --------------------------------------------------------------------------------------------------------- one pass
def run(s):
    b, buf = s.sets[s.turn % len(s.sets)], s.buf
    idx, before = s.idx[s.turn % 2], s.idx[(s.turn + 1) % 2]
    s.turn += 1
    if s.form == "step":
        buf.step(b.u, s.beta, b.prio, b.pos, out_idx=idx, out_weight=s.weight, out_prio=s.value, rows_out=s.rows, B=s.B,
                 insert=(s.n, b.rows, None, None) if s.n else None)
    elif s.form == "graph":
        s.graph.replay()
        buf.note_replay()
        idx = s.idx[0]
    elif s.form == "earlier":
        buf.sample(b.u, s.beta, out_idx=idx, out_weight=s.weight, out_prio=s.value, rows_out=s.rows, update=(before, b.prio))
    elif s.form == "apart":
        buf.sample(b.u, s.beta, out_idx=idx, out_weight=s.weight, out_prio=s.value, rows_out=s.rows)
        buf.update(idx, b.prio)
    elif s.form == "td":
        buf.sample(b.u, s.beta, out_idx=idx, out_weight=s.weight, out_prio=s.value, rows_out=s.rows, B=s.B)
        buf.update_td(idx, b.prio)
    elif s.form == "fill":
        buf.insert(s.n, b.rows, b.row_prio, s.slots)
        buf.sample(b.u, s.beta, out_idx=idx, out_weight=s.weight, out_prio=s.value, rows_out=s.rows)
        return [s.slots, idx, s.weight, s.value, *s.rows]
    elif s.form == "steps":
        idx = s.idx[0]
        buf.run_steps(b.u, s.betas, idx, s.weight, s.value, s.rows, upd_prio=b.prio, n_insert=s.n, ins_rows=b.rows)
    else:
        idx = s.idx[0]
        buf.run_requests(b.queue)
    return [idx, s.weight, s.value, *s.rows]


# ------------------------------------------------------------------------------------------- what a pass cannot spare
def _nodes(case):
    n = [case["N"]]
    while n[-1] > 1:
        n.append(-(-n[-1] // case["K"]))
    return n


def work(case):
    """Bytes: uniforms, indices, weights, values, rows (read where stored, written dense), new priorities, new rows;
    of the tree the distinct child groups that a batch spread over it meets, read once, and the touched nodes, written
    once.  A list of iterations on an on-chip tree reads and writes its tree once.  Operations: the sums of the
    touched groups and the walk through each."""
    K, T, B, n, S = (case[k] for k in ("K", "T", "B", "insert", "iterations"))
    E, levels = sum(_widths(case)), _nodes(case)
    per_batch = B * (4 * (4 + (not case["rng"]) + bool(case["positions"])) + 2 * E) + n * 2 * E
    if case["form"] == "fill":
        per_batch += n * 8
    groups = nodes = walk = 0.0
    for h, m in enumerate(levels):
        touched = m * -math.expm1(-B / m) + min(n, m) / (K ** h)
        nodes += min(m, touched)
        if h:
            groups += min(m, touched)
            walk += B * math.log2(K)
    if case["form"] in ("steps", "queue"):
        tree = 2 * 4 * sum(levels)
    else:
        tree = S * (groups * K * 4 + nodes * 4)
    return {"bytes": T * (S * per_batch + tree), "flops": T * S * (groups * (K - 1) + 2 * walk + 40 * B)}


def tolerance(case):
    """Indices, values and rows are the same to the bit; a weight is one rounding of a double to 32 bits.  Priorities
    made from temporal-difference errors go through a power function that may round the last bit otherwise, which can
    move a sample to the leaf beside it."""
    if case["form"] == "td":
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}
    return {"rel": 1e-6, "max": 2e-6, "differ": 0.0}
