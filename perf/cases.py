"""The workloads whose speed this framework is judged by, as a training program calls them.

Six kinds of case, each one pass through the Python entry points:

  replay     one off-policy iteration: the learner's priorities of its last batch
             and the actor's new transitions go in (`update_ingest`), the next
             batch comes out (`sample_gather`, or with n-step targets and the
             bootstrap states, `conduit_sample_gather_nstep`)
  tokens     the same for variable-length sequences, delivered packed with their
             advantages (`update_ingest`, `sample_pack_gae`)
  ingest     one bulk ingest of transitions (`ingest`)
  gae        advantages of a time-major rollout (`conduit_gae`, `conduit_gae_truncated`)
  packed     advantages of right-padded sequences with a critic (`conduit_gae_packed`)
  minibatch  the next shuffled minibatch of a rollout (`conduit_minibatch_gather`)

Inputs are seeded and synthetic.  `exact` works the outputs out again in 64 bits
with plain numpy and torch.
"""
import numpy as np
import torch

from paper_2609_24456_amd import conduit as cd

MEAN, STD = (0.485, 0.456, 0.406, 0.45), (0.229, 0.224, 0.225, 0.226)
XF = {"none": cd.XF_NONE, "f32": cd.XF_U8_F32, "bf16": cd.XF_U8_BF16_NORM}
OUT_DTYPE = {"none": None, "f32": torch.float32, "bf16": torch.bfloat16}
OUT_BYTES = {"none": 1, "f32": 4, "bf16": 2}
VOCAB = 128000
BETA = 0.4
FILL_BYTES = 256 << 20  # payload of one ingest while a buffer is filled


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest loop there is: a classic-control agent (8 fp32 observations), one process
        _replay("tiny-step", capacity=16384, dim=8, ingest=64, batch=256),
        # the ordinary one: DQN on 84x84 frames, stacks of 4, a replay of a million frames
        _replay("dqn-step", capacity=1_000_000, frame=(1, 84, 84), stack=4, ingest=512, batch=512, xf="f32"),
        # the same network trained on 3-step returns, a smaller replay
        _replay("dqn-3step", capacity=200_000, frame=(1, 84, 84), stack=4, ingest=256, batch=512, xf="f32", nstep=3),
        # off-policy learning from thousands of simulated environments: one vector step of all of them in, one large
        # batch of vector observations out
        _replay("simulated-envs-step", capacity=1_000_000, dim=48, action=48, ingest=4096, batch=16384),
        # large camera images, normalised per channel into bf16
        _replay("visual-step", capacity=20_000, frame=(3, 224, 224), action=24, ingest=256, batch=1024, xf="bf16"),
        # post-training of a language model on outcome rewards: 256 sequences of up to 4,096 tokens in and out
        _tokens("tokens-step", capacity=8192, max_len=4096, ingest=256, batch=256, values=False),
        # a bulk load of frames, as when a replay is filled from a recorded run
        _ingest("frames-ingest", capacity=65_536, frame=(1, 84, 84), n=32_768, prio=True),
        # one PPO rollout: 256 environments of 2,048 steps
        _gae("rollout-gae", T=2048, E=256, truncated=False),
        # a rollout of many simulated environments, with time limits
        _gae("simulated-envs-gae", T=128, E=16384, truncated=True),
        # token-level advantages with a critic, long sequences
        _packed("critic-gae", B=256, L=8192),
        # one PPO minibatch of images with advantages and returns
        _minibatch("image-minibatch", frame=(3, 84, 84), n_src=131_072, n=16_384, xf="f32", cols=2),
        # one PPO minibatch of vector observations: 4,096 environments of 24 steps in 4 minibatches, with advantages,
        # returns, old values, log-probabilities and entropies
        _minibatch("vector-minibatch", dim=48, n_src=98_304, n=24_576, xf="none", cols=5),
    ]


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    kind = rng.choice(["vector", "frames", "frames", "visual", "tokens", "ingest", "gae", "gae", "packed",
                       "minibatch", "minibatch"])
    norm = rng.choice(["batch", "batch", "buffer"])
    if kind == "vector":  # vector observations: the smallest agents to the widest simulations and stress transitions
        dim = _log(rng, 4, 4000)
        batch = _log(rng, 64, min(32768, 30_000_000 // dim))
        return _replay(None, capacity=_log(rng, 10_000, min(1_000_000, 500_000_000 // dim)), dim=dim,
                       action=4 * _log(rng, 1, 16), ingest=_log(rng, 16, min(4096, 2 * batch)), batch=batch,
                       nstep=rng.choice([0, 0, 0, 1, 5]), norm=norm)
    if kind == "frames":  # stacked frames
        side = 4 * rng.randint(10, 32)
        return _replay(None, capacity=_log(rng, 10_000, 300_000), frame=(1, side, side), stack=rng.choice([1, 2, 4]),
                       ingest=_log(rng, 32, 1024), batch=_log(rng, 32, 1024), xf=rng.choice(["f32", "f32", "none", "bf16"]),
                       nstep=rng.choice([0, 0, 1, 3, 5]), norm=norm)
    if kind == "visual":  # camera images of 1 to 4 planes
        side = 4 * rng.randint(24, 64)
        return _replay(None, capacity=rng.randint(4_000, 20_000), frame=(rng.choice([1, 3, 4]), side, side),
                       ingest=_log(rng, 16, 512), batch=_log(rng, 32, 1024), xf=rng.choice(["bf16", "bf16", "f32", "none"]))
    if kind == "tokens":
        max_len = 4 * _log(rng, 64, 2048)
        batch = _log(rng, 16, min(1024, 2_000_000 // max_len))
        return _tokens(None, capacity=rng.randint(1024, 8192), max_len=max_len, ingest=_log(rng, 16, batch),
                       batch=batch, values=rng.random() < 0.4, norm=norm)
    if kind == "ingest":
        if rng.random() < 0.5:
            side = 4 * rng.randint(10, 32)
            n = _log(rng, 512, 32_768)
            return _ingest(None, capacity=2 * n + rng.randint(0, 64), frame=(1, side, side), n=n, prio=rng.random() < 0.5)
        n = _log(rng, 2048, 200_000)
        return _ingest(None, capacity=2 * n + rng.randint(0, 64), dim=_log(rng, 4, 256), n=n, prio=rng.random() < 0.5,
                       prioritized=rng.random() < 0.5)
    if kind == "gae":
        E = _log(rng, 8, 65_536)
        T = _log(rng, 16, max(16, min(4096, 8_000_000 // E)))
        return _gae(None, T=T, E=E if rng.random() < 0.3 else (E + 3) // 4 * 4, truncated=rng.random() < 0.5)
    if kind == "packed":
        L = _log(rng, 256, 16_384)
        return _packed(None, B=_log(rng, 8, min(1024, 4_000_000 // L)), L=L if rng.random() < 0.3 else (L + 3) // 4 * 4)
    if rng.random() < 0.5:
        side = 4 * rng.randint(10, 32)
        planes = rng.choice([1, 3, 4])
        n = _log(rng, 256, min(12_288, 300_000_000 // (planes * side * side)))
        return _minibatch(None, frame=(planes, side, side), n_src=4 * n + rng.randint(0, 64), n=n,
                          xf=rng.choice(["f32", "f32", "bf16", "none"]), cols=rng.randint(0, 4))
    dim = _log(rng, 4, 1024)
    n = _log(rng, 256, min(65_536, 60_000_000 // dim))
    return _minibatch(None, dim=dim, n_src=4 * n + rng.randint(0, 64), n=n, xf="none", cols=rng.randint(0, 8))


def _log(rng, lo, hi):
    """A whole number in [lo, hi], uniform in its logarithm."""
    return max(lo, min(hi, int(round(lo * (max(lo, hi) / lo) ** rng.random()))))


def _case(name, **fields):
    return dict(fields, name=name) if name else fields


def _payload(dim, frame):
    """Fields that say what one observation is: `dim` fp32 values, or u8 planes of h x w."""
    c, h, w = frame or (0, 0, 0)
    return {"dim": dim, "planes": c, "height": h, "width": w}


def _replay(name, capacity, ingest, batch, dim=0, frame=None, action=4, stack=1, xf="none", nstep=0, norm="batch"):
    return _case(name, kind="replay", capacity=capacity, ingest=ingest, batch=batch, action=action, stack=stack, xf=xf,
                 nstep=nstep, norm=norm, **_payload(dim, frame))


def _tokens(name, capacity, max_len, ingest, batch, values, norm="batch"):
    return _case(name, kind="tokens", capacity=capacity, max_len=max_len, ingest=ingest, batch=batch, values=values,
                 norm=norm)


def _ingest(name, capacity, n, prio, dim=0, frame=None, prioritized=True):
    return _case(name, kind="ingest", capacity=capacity, n=n, prio=prio and prioritized, prioritized=prioritized,
                 **_payload(dim, frame))


def _gae(name, T, E, truncated):
    return _case(name, kind="gae", T=T, E=E, truncated=truncated)


def _packed(name, B, L):
    return _case(name, kind="packed", B=B, L=L)


def _minibatch(name, n_src, n, xf, cols, dim=0, frame=None):
    return _case(name, kind="minibatch", n_src=n_src, n=n, xf=xf, cols=cols, **_payload(dim, frame))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _dev(a):
    """A host array on the GPU (unsigned words as the signed type of their size)."""
    a = np.ascontiguousarray(a)
    a = a.view({"uint32": np.int32, "uint64": np.int64}.get(a.dtype.name, a.dtype))
    return torch.from_numpy(a).cuda()


def _obs_shape(c):
    if c["dim"]:
        return (c["dim"],)
    return (c["planes"], c["height"], c["width"]) if c["planes"] > 1 else (c["height"], c["width"])


def _obs_dtype(c):
    return torch.float32 if c["dim"] else torch.uint8


def _row_bytes(c):
    return 4 * c["dim"] if c["dim"] else c["planes"] * c["height"] * c["width"]


def _rows(c, n, g):
    """n observations: normal fp32 vectors, or uniformly distributed pixels."""
    if c["dim"]:
        return torch.randn((n, c["dim"]), generator=g, device="cuda")
    words = n * _row_bytes(c) // 4
    w = torch.randint(-2 ** 31, 2 ** 31, (words,), generator=g, device="cuda", dtype=torch.int32)
    return w.view(torch.uint8).view((n,) + _obs_shape(c))


def _priorities(rng, n):
    """Absolute TD errors, heavy-tailed, as the 32-bit priorities a learner writes."""
    return (np.minimum(np.round(1e4 * rng.lognormal(0.0, 1.0, n)), 2.0 ** 32 - 2) + 1).astype(np.uint32)


class _Columns:
    """Everything but the observations of a stream of n transitions, on the host."""

    def __init__(self, c, n, seed):
        rng = np.random.default_rng(seed)
        lo, hi = (200, 2000) if not c.get("dim") else (20, 500)
        lengths = rng.integers(lo, hi + 1, n // lo + 2)
        ends = np.cumsum(lengths)
        k = int(np.searchsorted(ends, n)) + 1  # episodes that reach into the stream
        lengths, ends = lengths[:k], ends[:k]
        self.episode = np.repeat(np.arange(k, dtype=np.uint32), lengths)[:n]
        self.step = (np.arange(n) - np.repeat(ends - lengths, lengths)[:n]).astype(np.int32)
        self.done = np.zeros(n, np.uint8)
        self.done[ends[ends <= n] - 1] = 1
        self.reward = rng.standard_normal(n).astype(np.float32)
        self.action = rng.integers(0, 256, (n, c.get("action", 4)), dtype=np.uint8)
        self.prio = _priorities(rng, n)

    def span(self, a, b, prio=True):
        out = {k: _dev(getattr(self, k)[a:b]) for k in ("action", "reward", "done", "step")}
        out["episode_id"] = _dev(self.episode[a:b])
        if prio:
            out["prio"] = _dev(self.prio[a:b])
        return out


def _uniforms(rng, n):
    return rng.integers(0, 2 ** 64, n, dtype=np.uint64)


class _ReplayInputs:
    """The inputs of a replay case in the order both prepare() and exact() need them."""

    def __init__(self, c, seed):
        self.case, self.filled = c, c["capacity"] + c["capacity"] // 8  # the ring has wrapped
        self.n = self.filled + c["ingest"]
        self.cols = _Columns(c, self.n, seed)
        rng = np.random.default_rng([seed, 1])
        # the last batch's slots (a batch has repeats) and its new priorities
        self.idx = rng.integers(0, c["capacity"], c["batch"])
        self.idx[c["batch"] // 2:][::7] = self.idx[: len(self.idx[c["batch"] // 2:][::7])]
        self.prio = _priorities(rng, c["batch"])
        self.u = _uniforms(rng, c["batch"])

    def chunks(self, seed):
        """(first, last, observations) over the whole stream, the pass's own transitions as the last chunk."""
        g = _generator(seed)
        per = max(1, min(self.case["capacity"], FILL_BYTES // _row_bytes(self.case)))  # an ingest takes at most a ring
        for a in range(0, self.filled, per):
            b = min(a + per, self.filled)
            yield a, b, _rows(self.case, b - a, g)
        yield self.filled, self.n, _rows(self.case, self.n - self.filled, g)


def _transform(c):
    if c["xf"] != "bf16":
        return cd.transform(XF[c["xf"]])
    return cd.transform(XF["bf16"], mean=MEAN[: c["planes"]], std=STD[: c["planes"]])


def _out_rows(c, n, stack):
    shape = (n,) + ((stack,) if stack > 1 else ()) + _obs_shape(c)
    return torch.empty(shape, dtype=OUT_DTYPE[c["xf"]] or _obs_dtype(c), device="cuda")


def prepare(case, seed):
    return {"replay": _prepare_replay, "tokens": _prepare_tokens, "ingest": _prepare_ingest, "gae": _prepare_gae,
            "packed": _prepare_packed, "minibatch": _prepare_minibatch}[case["kind"]](case, seed)


def _prepare_replay(c, seed):
    x = _ReplayInputs(c, seed)
    buf = cd.ReplayBuffer(c["capacity"], _obs_shape(c), _obs_dtype(c), frame_stack=c["stack"], action_bytes=c["action"],
                          beta=BETA, weight_norm=int(c["norm"] == "buffer"))
    for a, b, rows in x.chunks(seed):
        if a < x.filled:
            buf.ingest(rows, **x.cols.span(a, b))
    B = c["batch"]
    s = {"case": c, "buf": buf, "xf": _transform(c), "new": dict(x.cols.span(x.filled, x.n, prio=False), obs=rows),
         "u": _dev(x.u), "prio": _dev(x.prio)}
    s["idx"], s["w"] = _dev(x.idx), torch.empty(B, device="cuda")
    s["out"] = {"obs": _out_rows(c, B, c["stack"]), "action": torch.empty((B, c["action"]), dtype=torch.uint8, device="cuda"),
                "reward": torch.empty(B, device="cuda"), "done": torch.empty(B, dtype=torch.uint8, device="cuda")}
    if c["nstep"]:
        s["next"] = {"next_idx": torch.empty(B, dtype=torch.int64, device="cuda"), "ret": torch.empty(B, device="cuda"),
                     "discount": torch.empty(B, device="cuda"), "valid": torch.empty(B, dtype=torch.uint8, device="cuda"),
                     "next_obs": _out_rows(c, B, c["stack"])}
    return s


class _TokenInputs:
    def __init__(self, c, seed):
        self.case, self.filled = c, c["capacity"] + c["capacity"] // 8
        self.n = self.filled + c["ingest"]
        rng = np.random.default_rng([seed, 2])
        self.length = rng.integers(max(1, c["max_len"] // 8), c["max_len"] + 1, self.n)
        self.offsets = np.concatenate([[0], np.cumsum(self.length)])
        self.reward = rng.standard_normal(self.n).astype(np.float32)
        self.stored = _priorities(rng, self.n)
        self.idx = rng.integers(0, c["capacity"], c["batch"])
        self.prio = _priorities(rng, c["batch"])
        self.u = _uniforms(rng, c["batch"])

    def chunks(self, seed):
        g = _generator(seed)
        per = max(1, min(self.case["capacity"], FILL_BYTES // (8 * self.case["max_len"])))
        for a, b in [(a, min(a + per, self.filled)) for a in range(0, self.filled, per)] + [(self.filled, self.n)]:
            k = int(self.offsets[b] - self.offsets[a])
            tokens = torch.randint(0, VOCAB, (k,), generator=g, device="cuda", dtype=torch.int32)
            logp = torch.empty(k, device="cuda").exponential_(generator=g).neg_()
            yield a, b, tokens, logp

    def span(self, a, b):
        return {"offsets": _dev(self.offsets[a:b + 1] - self.offsets[a]), "reward": _dev(self.reward[a:b])}


def _prepare_tokens(c, seed):
    x = _TokenInputs(c, seed)
    buf = cd.ReplayBuffer(c["capacity"], (c["max_len"],), torch.int32, ragged=True, aux_elem_bytes=4, beta=BETA,
                          weight_norm=int(c["norm"] == "buffer"))
    for a, b, tokens, logp in x.chunks(seed):
        if a < x.filled:
            buf.ingest(tokens, aux=logp, prio=_dev(x.stored[a:b]), **x.span(a, b))
    B, L = c["batch"], c["max_len"]
    f = lambda *shape: torch.empty(shape, device="cuda")  # noqa: E731
    return {"case": c, "buf": buf, "xf": cd.transform(cd.XF_TOKENS_PAD), "new": dict(x.span(x.filled, x.n), obs=tokens, aux=logp),
            "u": _dev(x.u), "prio": _dev(x.prio), "idx": _dev(x.idx), "w": f(B),
            "values": torch.randn((B, L), generator=_generator(seed + 1), device="cuda") if c["values"] else None,
            "out": {"obs": torch.empty((B, L), dtype=torch.int32, device="cuda"), "aux": f(B, L),
                    "mask": torch.empty((B, L), dtype=torch.uint8, device="cuda"), "reward": f(B),
                    "length": torch.empty(B, dtype=torch.int32, device="cuda")},
            "adv": f(B, L), "ret": f(B, L)}


def _prepare_ingest(c, seed):
    opts = dict(prioritized=int(c["prioritized"]))
    shape = _obs_shape(c)
    dtype = cd.F32 if c["dim"] else cd.U8
    arena = torch.zeros(cd.conduit_buffer_required_bytes(c["capacity"], shape, dtype, cd.default_opts(**opts)),
                        dtype=torch.uint8, device="cuda")
    buf = cd.ReplayBuffer(c["capacity"], shape, _obs_dtype(c), prioritized=c["prioritized"], arena=arena)
    cols = _Columns(c, c["n"], seed)
    return {"case": c, "buf": buf, "arena": arena, "obs": _rows(c, c["n"], _generator(seed)),
            "cols": cols.span(0, c["n"], prio=c["prio"])}


def _prepare_gae(c, seed):
    g, T, E = _generator(seed), c["T"], c["E"]
    f = lambda *shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
    flags = lambda p: (torch.rand((T, E), generator=g, device="cuda") < p).to(torch.uint8)  # noqa: E731
    s = {"case": c, "r": f(T, E), "v": f(T, E), "done": flags(0.005), "boot": f(E)}
    if c["truncated"]:
        s["trunc"], s["final"] = flags(0.005), f(T, E)
    s["adv"], s["ret"] = torch.empty((T, E), device="cuda"), torch.empty((T, E), device="cuda")
    return s


def _prepare_packed(c, seed):
    g, B, L = _generator(seed), c["B"], c["L"]
    return {"case": c, "reward": torch.randn(B, generator=g, device="cuda"),
            "length": torch.randint(max(1, L // 8), L + 1, (B,), generator=g, device="cuda", dtype=torch.int32),
            "values": torch.randn((B, L), generator=g, device="cuda"),
            "adv": torch.empty((B, L), device="cuda"), "ret": torch.empty((B, L), device="cuda")}


def _prepare_minibatch(c, seed):
    g, n = _generator(seed), c["n"]
    rows = torch.empty((c["n_src"],) + _obs_shape(c), dtype=_obs_dtype(c), device="cuda")
    per = max(1, FILL_BYTES // _row_bytes(c))
    for a in range(0, c["n_src"], per):
        rows[a:a + per] = _rows(c, min(per, c["n_src"] - a), g)
    cols = [torch.randn(c["n_src"], generator=g, device="cuda") for _ in range(c["cols"])]
    perm = torch.randperm(c["n_src"], generator=g, device="cuda")
    return {"case": c, "rows": rows, "cols": cols, "perms": list(perm[: c["n_src"] // n * n].split(n)), "k": 0,
            "xf": _transform(c), "out": _out_rows(c, n, 1), "cols_out": [torch.empty(n, device="cuda") for _ in cols]}


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
GAMMA, LAMBDA = 0.99, 0.95


def run(s):
    c = s["case"]
    if c["kind"] == "replay":
        buf = s["buf"]
        buf.update_ingest(s["idx"], s["prio"], **s["new"])
        if c["nstep"]:
            nxt = s["next"]
            cd.conduit_sample_gather_nstep(buf.handle, c["batch"], s["u"], s["idx"], s["w"], s["xf"], c["nstep"], GAMMA,
                                           **nxt, **s["out"])
            return {"idx": s["idx"], "w": s["w"], "next": nxt, **s["out"]}
        buf.sample_gather(s["u"], s["xf"], idx_out=s["idx"], w_out=s["w"], **s["out"])
        return {"idx": s["idx"], "w": s["w"], **s["out"]}
    if c["kind"] == "tokens":
        buf = s["buf"]
        buf.update_ingest(s["idx"], s["prio"], **s["new"])
        cd.conduit_sample_pack_gae(buf.handle, c["batch"], s["u"], s["idx"], s["w"], s["xf"], s["values"], 1.0, LAMBDA,
                                   s["adv"], s["ret"], **s["out"])
        return {"idx": s["idx"], "w": s["w"], "adv": s["adv"], "ret": s["ret"], **s["out"]}
    if c["kind"] == "ingest":
        s["buf"].ingest(s["obs"], **s["cols"])
        return {"arena": s["arena"]}
    if c["kind"] == "gae":
        if c["truncated"]:
            cd.conduit_gae_truncated(s["r"], s["v"], s["done"], s["trunc"], s["final"], s["boot"], GAMMA, LAMBDA, s["adv"],
                                     s["ret"])
        else:
            cd.conduit_gae(s["r"], s["v"], s["done"], s["boot"], GAMMA, LAMBDA, s["adv"], s["ret"])
        return {"adv": s["adv"], "ret": s["ret"]}
    if c["kind"] == "packed":
        cd.conduit_gae_packed(s["reward"], s["length"], s["values"], c["L"], 1.0, LAMBDA, s["adv"], s["ret"])
        return {"adv": s["adv"], "ret": s["ret"]}
    perm = s["perms"][s["k"] % len(s["perms"])]
    s["k"] += 1
    cd.conduit_minibatch_gather(s["rows"], _row_bytes(c), c["n_src"], perm, s["xf"], s["out"], s["cols"], s["cols_out"])
    return {"out": s["out"], "cols": s["cols_out"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(c):
    """Bytes: each input read once, each output written once.  Flops: the arithmetic of the transforms and
    recursions (a handful per element), which never bounds these paths."""
    k = c["kind"]
    if k in ("replay", "ingest"):
        row = _row_bytes(c)
        meta = c.get("action", 4) + 4 + 1 + 4 + 4  # action, reward, done, episode, step
    if k == "ingest":
        return {"bytes": c["n"] * (2 * (row + meta) + (4 if c["prio"] else 0) + (4 if c["prioritized"] else 0)), "flops": c["n"]}
    if k == "replay":
        ingest = c["ingest"] * (2 * (row + meta) + 4)
        update = c["batch"] * (12 + 4)  # index and priority in, leaf out
        out = OUT_BYTES[c["xf"]]
        frames = c["stack"] + (min(c["nstep"], c["stack"]) if c["nstep"] else 0)  # distinct frames read
        deliver = c["batch"] * (frames * row + c["stack"] * row * out * (2 if c["nstep"] else 1) + 2 * (c["action"] + 5)
                                + 8 + 8 + 4 + 4)
        if c["nstep"]:
            deliver += c["batch"] * (c["nstep"] * 5 + 17)
        return {"bytes": ingest + update + deliver, "flops": c["batch"] * c["stack"] * row}
    if k == "tokens":
        mean = c["max_len"] * 9 // 16  # lengths are uniform in [max_len / 8, max_len]
        ingest = c["ingest"] * (mean * 16 + 20)
        B, L = c["batch"], c["max_len"]
        deliver = B * (mean * 8 + L * 9 + (mean * 4 if c["values"] else 0) + L * 8 + 40)
        return {"bytes": ingest + deliver + B * 16, "flops": 4 * B * L}
    if k == "gae":
        N = c["T"] * c["E"]
        return {"bytes": N * (17 + (1 if c["truncated"] else 0)) + 4 * c["E"], "flops": 6 * N}
    if k == "packed":
        return {"bytes": c["B"] * (c["L"] * 9 // 16 * 4 + c["L"] * 8 + 8), "flops": 6 * c["B"] * c["L"]}
    row = _row_bytes(c)
    return {"bytes": c["n"] * (row + row * OUT_BYTES[c["xf"]] + 8 + 8 * c["cols"]), "flops": c["n"] * row}


def tolerance(c):
    """Indices, copies and pixel transforms are exact.  Advantages, returns and weights are worked out in 64 bits
    and rounded to 32 once: another order of the sums moves a value by one unit of the last place (2^-23 of it,
    at worst) now and then; n-step returns and discounts likewise."""
    if c["kind"] in ("ingest", "minibatch"):
        return "exact"
    return {"rel": 1e-7, "max": 5e-7}


# ---------------------------------------------------------------------------
# the outputs in 64 bits
# ---------------------------------------------------------------------------
def exact(case, seed):
    f = {"replay": _exact_replay, "tokens": _exact_tokens, "gae": _exact_gae, "packed": _exact_packed,
         "minibatch": _exact_minibatch}.get(case["kind"])
    return f(case, seed) if f else None  # an ingest returns bytes


def _leaf(prio):
    """floor(2^12 p^(3/5)) of 32-bit priorities p >= 1: in floating point away from whole numbers, in integers near them."""
    p = prio.astype(np.int64)
    x = np.exp2(12 + 0.6 * np.log2(p.astype(np.float64)))
    q = np.floor(x).astype(np.int64)
    near = np.rint(x).astype(np.int64)
    for k in np.flatnonzero(np.abs(x - near) < 2.0 ** -12):
        n = int(near[k])
        q[k] = n if n ** 5 <= int(p[k]) ** 3 << 60 else n - 1
    return q


def _draw_slots(leaf, u):
    """The slot of every stratum: the first whose prefix sum of leaves exceeds (k + u_k / 2^64) Q / B."""
    B, prefix = len(u), np.cumsum(leaf)
    Q = int(prefix[-1])
    t = [((k << 64) + int(x)) * Q // (B << 64) for k, x in enumerate(u)]
    return np.searchsorted(prefix, np.array(t, np.int64), side="right")


def _weights(leaf, slots, norm):
    least = leaf[leaf > 0].min() if norm == "buffer" else leaf[slots].min()
    return torch.from_numpy((least / leaf[slots].astype(np.float64)) ** BETA)


def _positions(C, n):
    """The stream position that each of C slots holds after n transitions."""
    i = np.arange(C)
    return i + (n - 1 - i) // C * C


def _leaves_of_pass(x, stored, C):
    """The leaves that a pass samples from: the stored priorities, then the update, then the pass's new rows."""
    pos = _positions(C, x.filled)
    prio = stored[pos]
    top = max(1, int(stored[: x.filled].max()), int(x.prio.max()))
    prio[x.idx] = x.prio  # the last of a repeated index stays
    now = _positions(C, x.n)
    prio[now >= x.filled] = top
    return _leaf(prio), now


def _expand(c, rows):
    """Stored rows through the case's transform, in 64 bits."""
    v = rows.double()
    if c["xf"] == "f32":
        v /= 255.0
    elif c["xf"] == "bf16":
        shape = (-1, 1, 1) if c["planes"] > 1 else (1, 1)
        m = torch.tensor(MEAN[: c["planes"]], dtype=torch.float32, device="cuda").double().view(shape)
        d = torch.tensor(STD[: c["planes"]], dtype=torch.float32, device="cuda").double().view(shape)
        v = (v / 255.0 - m) / d
    return v


def _stacks(c, ring, x, now, slots):
    """The frame stacks of slots (-1: zeros)."""
    C, K = c["capacity"], c["stack"]
    flt = c["xf"] != "none" or c["dim"] > 0
    if not flt:
        return None
    ep, st = x.cols.episode[now], x.cols.step[now]
    out = torch.zeros((len(slots), K) + _obs_shape(c), dtype=torch.float64, device="cuda")
    for k in range(K):
        d = K - 1 - k
        j = (slots - d) % C
        ok = (slots >= 0) & (ep[j] == ep[slots]) & (st[j] == st[slots] - d)
        at = torch.from_numpy(np.flatnonzero(ok)).cuda()
        out[at, k] = _expand(c, ring[torch.from_numpy(j[ok]).cuda()])
    return out if K > 1 else out[:, 0]


def _exact_replay(c, seed):
    x, C = _ReplayInputs(c, seed), c["capacity"]
    ring = torch.empty((C,) + _obs_shape(c), dtype=_obs_dtype(c), device="cuda")
    for a, b, rows in x.chunks(seed):
        ring[torch.arange(a, b, device="cuda") % C] = rows
    leaf, now = _leaves_of_pass(x, x.cols.prio, C)
    slots = _draw_slots(leaf, x.u)
    out = {"idx": None, "w": _weights(leaf, slots, c["norm"]), "obs": _stacks(c, ring, x, now, slots), "action": None,
           "reward": torch.from_numpy(x.cols.reward[now[slots]].astype(np.float64)), "done": None}
    if c["nstep"]:
        ret, disc, nxt = np.zeros(len(slots)), np.zeros(len(slots)), np.full(len(slots), -1)
        for b, s in enumerate(slots):
            p, total, g = int(now[s]), 0.0, 1.0
            for k in range(c["nstep"] + 1):
                q = p + k
                if q >= x.n or x.cols.episode[q] != x.cols.episode[p]:
                    break  # not stored yet, or the episode is cut: no target
                if k == c["nstep"]:
                    ret[b], disc[b], nxt[b] = total, g, q % C
                    break
                total += g * float(x.cols.reward[q])
                g *= GAMMA
                if x.cols.done[q]:
                    ret[b] = total
                    break
        out["next"] = {"next_idx": None, "ret": torch.from_numpy(ret), "discount": torch.from_numpy(disc), "valid": None,
                       "next_obs": _stacks(c, ring, x, now, nxt)}
    return out


def _packed_gae(reward, length, values, gamma, lam):
    """Advantages and returns of padded rows in 64 bits, and 0 past a row's end."""
    B, L = values.shape
    r, n = reward.double(), length.long()
    adv, ret = torch.zeros_like(values), torch.zeros_like(values)
    A, after = torch.zeros_like(r), torch.zeros_like(r)
    for t in range(L - 1, -1, -1):
        last, live = n == t + 1, n > t
        v = values[:, t]
        A = torch.where(last, r - v, gamma * after - v + gamma * lam * A)
        A = torch.where(live, A, torch.zeros_like(A))
        after = v
        adv[:, t] = A
        ret[:, t] = torch.where(live, A + v, torch.zeros_like(A))
    return adv, ret


def _exact_tokens(c, seed):
    x, C, L = _TokenInputs(c, seed), c["capacity"], c["max_len"]
    leaf, now = _leaves_of_pass(x, x.stored, C)
    # the pass's own rows carry no priority: the largest so far
    slots = _draw_slots(leaf, x.u)
    at = now[slots]
    aux = torch.zeros((len(slots), L), dtype=torch.float64, device="cuda")
    for a, b, _, logp in x.chunks(seed):
        for row in np.flatnonzero((at >= a) & (at < b)):
            k = int(x.offsets[at[row]] - x.offsets[a])
            aux[row, : int(x.length[at[row]])] = logp[k:k + int(x.length[at[row]])].double()
    reward, length = _dev(x.reward[at]), _dev(x.length[at])
    if c["values"]:
        values = torch.randn((c["batch"], L), generator=_generator(seed + 1), device="cuda").double()
    else:
        values = torch.zeros((c["batch"], L), dtype=torch.float64, device="cuda")
    adv, ret = _packed_gae(reward, length, values, 1.0, LAMBDA)
    return {"idx": None, "w": _weights(leaf, slots, c["norm"]), "adv": adv, "ret": ret, "obs": None, "aux": aux,
            "mask": None, "reward": reward.double(), "length": None}


def _exact_gae(c, seed):
    s = _prepare_gae(c, seed)
    r, v, done = s["r"].double(), s["v"].double(), s["done"].bool()
    cut = done | s["trunc"].bool() if c["truncated"] else done
    adv, A, after = torch.empty_like(r), torch.zeros_like(r[0]), s["boot"].double()
    for t in range(c["T"] - 1, -1, -1):
        boot = torch.where(cut[t], torch.zeros_like(after), after)
        if c["truncated"]:
            boot = torch.where(cut[t] & ~done[t], s["final"][t].double(), boot)
        A = r[t] + GAMMA * boot - v[t] + GAMMA * LAMBDA * torch.where(cut[t], torch.zeros_like(A), A)
        adv[t], after = A, v[t]
    return {"adv": adv, "ret": adv + v}


def _exact_packed(c, seed):
    s = _prepare_packed(c, seed)
    adv, ret = _packed_gae(s["reward"], s["length"], s["values"].double(), 1.0, LAMBDA)
    return {"adv": adv, "ret": ret}


def _exact_minibatch(c, seed):
    s = _prepare_minibatch(c, seed)
    out = _expand(c, s["rows"][s["perms"][0]]) if c["xf"] != "none" or c["dim"] else None
    return {"out": out, "cols": [x[s["perms"][0]].double() for x in s["cols"]]}
