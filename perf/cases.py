"""The performance cases of this library: passes through its public entry points, as a serving program makes them.

A case is one pass of a program that holds a `Context` (weights registered, pools allocated) and its requests' block
tables: a decode step, a prefill pass, a hybrid batch, or both sides at once on a split chip, over one or more layers of
the shapes in `rs_synth`.  Inputs are random with the distributions of the workloads: hidden states N(0, 1), weights
N(0, 0.02), gains 1 + N(0, 0.02), cached keys and values N(0, 1), block tables a random permutation of the pool.

Lengths are a function of the case alone, so that every seed is the same amount of work; the seed draws the values, the
weights, the order of the requests and the block ids.  A pass only enqueues: passes are ordered by the streams of the one
`Context` that makes them all.
"""
import numpy as np
import torch

import paper_2601_11822_amd as rs
import rs_synth as S


def _case(kind, name=None, shape="llama3-8b-layer", layers=1, experts=0, vocab=0, prompts="", starts="", batch=0,
          ctx_lo=0, ctx_hi=0, steps=1, prefill_cus=256, decode_cus=256):
    c = dict(kind=kind, shape=shape, layers=layers, experts=experts, vocab=vocab, prompts=prompts, starts=starts, batch=batch,
             ctx_lo=ctx_lo, ctx_hi=ctx_hi, steps=steps, prefill_cus=prefill_cus, decode_cus=decode_cus)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one user's chat turn: a single row per step, where latency and the number of launches count
        _case("decode", "decode_1", layers=4, batch=1, ctx_lo=900, ctx_hi=900),
        # the benchmark's decode batch
        _case("decode", "decode_64", layers=2, batch=64, ctx_lo=512, ctx_hi=4096),
        # the closed-loop serving configuration at its batch cap: token embedding, layers, final norm and head
        _case("decode", "decode_256_head", layers=2, vocab=128256, batch=256, ctx_lo=64, ctx_hi=2047),
        # the 70B-shaped configuration's decode step, an odd batch above 64 rows
        _case("decode", "decode_100_70b", shape="llama3-70b-layer", batch=101, ctx_lo=130, ctx_hi=8100),
        # the long-context configuration: almost all of the step is reading the cache
        _case("decode", "decode_long", batch=32, ctx_lo=8192, ctx_hi=32767),
        # a short question: few rows, bound by reading the weights
        _case("prefill", "prefill_77", layers=4, prompts="77"),
        # the benchmark's prompt
        _case("prefill", "prefill_2048", layers=1, prompts="2048"),
        # the 70B-shaped configuration's pass: several prompts of uneven lengths
        _case("prefill", "prefill_ragged_70b", shape="llama3-70b-layer", prompts="1391,518,2730,805"),
        # the long-context configuration's whole prompt
        _case("prefill", "prefill_16384", prompts="16384"),
        # the mixture-of-experts model: short prompts that arrived together
        _case("prefill", "moe_prefill_1100", experts=8, prompts="611,173,316"),
        # hybrid batching: the third 512-token chunk of a prompt beside 64 decode rows
        _case("hybrid", "hybrid_512_64", layers=2, prompts="512", starts="1024", batch=64, ctx_lo=512, ctx_hi=4096),
        # the two sides at once on half of the chip each: one prefill pass beside four decode steps
        _case("corun", "corun_128_128", prompts="2048", batch=64, ctx_lo=512, ctx_hi=4096, steps=4, prefill_cus=128, decode_cus=128),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _prompt_lengths(rng, n, total):
    """n uneven lengths of at least 1 that add up to about `total`."""
    w = [0.2 + rng.random() for _ in range(n)]
    return [max(1, int(total * v / sum(w))) for v in w]


def draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "prefill", "prefill", "prefill", "hybrid", "corun"))
    big = rng.random() < 0.2
    shape = "llama3-70b-layer" if big else "llama3-8b-layer"
    experts = 8 if not big and kind in ("decode", "prefill") and rng.random() < 0.25 else 0
    join = lambda v: ",".join(str(x) for x in v)
    if kind == "decode":
        batch = _log_uniform(rng, 1, 256)
        hi = _log_uniform(rng, 128, min(32767, max(256, 600000 // batch)))
        lo = max(16, int(hi * rng.uniform(0.05, 1.0)))
        vocab = 128256 if not big and rng.random() < 0.25 else 0
        return _case(kind, shape=shape, layers=2 if batch <= 64 and not experts else 1, experts=experts, vocab=vocab, batch=batch,
                     ctx_lo=lo, ctx_hi=hi, decode_cus=rng.choice((256, 256, 128)), prefill_cus=0)
    if kind == "prefill":
        total = _log_uniform(rng, 16, 4000 if big or experts else 12000)
        n = rng.randint(1, 4)
        return _case(kind, shape=shape, layers=2 if total <= 512 and not experts else 1, experts=experts, prompts=join(_prompt_lengths(rng, n, total)),
                     prefill_cus=rng.choice((256, 256, 128)), decode_cus=0)
    if kind == "hybrid":
        chunk = rng.choice((512, 1024))
        lens = _prompt_lengths(rng, rng.randint(1, 3), chunk)
        starts = [16 * rng.randint(0, 192) for _ in lens]
        return _case(kind, shape=shape, prompts=join(lens), starts=join(starts), batch=rng.randint(1, 128), ctx_lo=rng.randint(16, 600),
                     ctx_hi=rng.randint(600, 4096))
    p = rng.choice((64, 96, 128, 160, 192))
    return _case(kind, prompts=join(_prompt_lengths(rng, rng.randint(1, 3), _log_uniform(rng, 512, 4096))), batch=rng.randint(8, 128),
                 ctx_lo=rng.randint(64, 1024), ctx_hi=rng.randint(1024, 4096), steps=4, prefill_cus=p, decode_cus=256 - p)


def _ints(text):
    return [int(v) for v in text.split(",")] if text else []


def _contexts(case):
    """Cached tokens of the decode rows: evenly spread over [ctx_lo, ctx_hi]."""
    return np.round(np.linspace(case["ctx_lo"], case["ctx_hi"], case["batch"])).astype(np.int32) if case["batch"] else np.zeros(0, np.int32)


class _Program:
    """What a program keeps from pass to pass: one `Context` and its pools, with room for the layers of `SLOTS` states (a
    state's passes go through layers of its own, with weights and cached tokens of its own, as a deep model's do)."""

    SLOTS = 4

    def __init__(self, case):
        sh, L, dev = S.SHAPES[case["shape"]], case["layers"], torch.device("cuda")
        self.key = {k: v for k, v in case.items() if k != "name"}
        held, rows = _held(case, _contexts(case)), sum(_ints(case["prompts"]))
        self.n_blocks = sum(S.blocks_for(n) for n in held) + 32
        pool = (self.SLOTS * L, self.n_blocks, sh.n_kv_heads, 16 * sh.head_dim)
        self.k_pool, self.v_pool = (torch.zeros(pool, device=dev, dtype=torch.bfloat16) for _ in range(2))
        self.ctx = rs.Context.from_shape(sh, n_layers=self.SLOTS * L, max_pos=max(held), n_blocks=self.n_blocks, k_pool=self.k_pool,
                                         v_pool=self.v_pool, max_prefill_tokens=rows + case["batch"] if case["kind"] == "hybrid" else rows,
                                         max_decode_batch=case["batch"], max_context=max(held), device=0)
        if case["vocab"]:
            normal, V, d = _normals(0), case["vocab"], sh.d_model
            self.ctx.set_head(normal(V, d), normal(d, std=0.02, mean=1.0), normal(V, d, std=0.02), V)
        self.ctx.set_cu_split(case["prefill_cus"], case["decode_cus"])
        self.free = list(range(self.SLOTS))


class _State:
    def __init__(self, program):
        self.program, self.slot = program, program.free.pop(0)

    def __del__(self):
        self.program.free.insert(0, self.slot)


_program = None


def _normals(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*dims, std=1.0, mean=0.0, out=None):
        t = torch.randn(*dims, generator=gen, device="cuda", dtype=torch.bfloat16) if out is None else out.normal_(generator=gen)
        if std != 1.0:
            t *= std
        return t + mean if mean else t

    return normal


def _held(case, ctx):
    """Tokens of each request after the pass, prompts first."""
    lens, starts = _ints(case["prompts"]), _ints(case["starts"])
    return [s + n for s, n in zip(starts or [0] * len(lens), lens)] + [int(c) + 1 for c in ctx]


def prepare(case, seed):
    global _program
    if _program is None or _program.key != {k: v for k, v in case.items() if k != "name"}:
        _program = None
        _program = _Program(case)
    st = _State(_program)
    c, sh, L, n_blocks = _program.ctx, S.SHAPES[case["shape"]], case["layers"], _program.n_blocks
    d, f, E = sh.d_model, sh.ffn_dim, case["experts"]
    normal, host = _normals(seed), np.random.Generator(np.random.Philox(key=[seed, 0]))
    st.kind, st.layers = case["kind"], range(st.slot * L, st.slot * L + L)
    st.k_pool, st.v_pool = _program.k_pool[st.layers.start:st.layers.stop], _program.v_pool[st.layers.start:st.layers.stop]
    if case["batch"] or case["starts"]:
        normal(out=st.k_pool), normal(out=st.v_pool)
    else:
        st.k_pool.zero_(), st.v_pool.zero_()

    lens, ctx = _ints(case["prompts"]), host.permutation(_contexts(case)).astype(np.int32)
    held = _held(case, ctx)
    st.width = max(S.blocks_for(n) for n in held)
    perm, at = host.permutation(n_blocks).astype(np.int32), 0
    tables = np.full((len(held), st.width), -1, np.int32)
    for i, n in enumerate(held):
        tables[i, :S.blocks_for(n)] = perm[at:at + S.blocks_for(n)]
        at += S.blocks_for(n)
    tables = torch.from_numpy(tables).cuda()
    st.ptab, st.dtab = tables[:len(lens)].contiguous(), tables[len(lens):].contiguous()
    st.cu, st.starts = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), _ints(case["starts"])
    st.lens, st.B, st.max_ctx = torch.from_numpy(ctx).cuda(), len(ctx), int(ctx.max()) + 1 if len(ctx) else 1

    st.xp = normal(sum(lens) + (st.B if st.kind == "hybrid" else 0), d)
    st.xd = normal(st.B, d)
    for layer in st.layers:
        gain = lambda: normal(d, std=0.02, mean=1.0)
        w = lambda *dims: normal(*dims, std=0.02)
        if E:
            router = normal(E, d, std=0.1)
            c.set_weights(layer, gain(), w(sh.qkv_dim, d), w(d, sh.q_dim), gain(), None, None, None)
            c.set_moe_weights(layer, router, w(E, f, d), w(E, f, d), w(E, d, f), E)
            # tokens lean towards two experts each, as they do in front of a trained router (of purely random tokens
            # some have their second and third expert closer than bf16 resolves)
            for x in (st.xp, st.xd):
                two = host.permuted(np.tile(np.arange(E), (x.shape[0], 1)), axis=1)[:, :2]
                x += 1.5 * router[torch.from_numpy(two).cuda()].sum(1)
        else:
            c.set_weights(layer, gain(), w(sh.qkv_dim, d), w(d, sh.q_dim), gain(), w(f, d), w(f, d), w(d, f))
    st.ctx, st.vocab, st.steps = c, case["vocab"], case["steps"]
    if st.vocab:
        st.tokens = torch.from_numpy(host.integers(0, st.vocab, st.B, dtype=np.int32)).cuda()
        st.logits = torch.empty(st.B, st.vocab, device="cuda", dtype=torch.float32)
    st.yp, st.yd = torch.empty_like(st.xp), torch.empty_like(st.xd)
    torch.cuda.synchronize()
    return st


def _prefill(st):
    x = st.xp
    for layer in st.layers:
        st.ctx.prefill_layer(layer, x, st.yp, st.cu, st.ptab, st.width)
        x = st.yp


def _decode(st):
    x = st.xd
    if st.vocab:
        st.ctx.embed(rs.RS_SIDE_DECODE, st.tokens, st.B, x)
    for layer in st.layers:
        st.ctx.decode_layer(layer, x, st.yd, st.lens, st.dtab, st.width, st.B, st.max_ctx)
        x = st.yd
    if st.vocab:
        st.ctx.lm_head_greedy(rs.RS_SIDE_DECODE, x, st.B, logits_out=st.logits)


def _hybrid(st):
    x = st.xp
    for layer in st.layers:
        st.ctx.hybrid_layer(layer, x, st.yp, st.cu, st.starts, st.ptab, st.width, st.lens, st.dtab, st.width, st.B, st.max_ctx)
        x = st.yp


def run(st):
    out = {"k_pool": st.k_pool, "v_pool": st.v_pool}
    if st.kind == "hybrid":
        _hybrid(st)
    if st.kind in ("prefill", "corun"):
        _prefill(st)
    if st.kind in ("decode", "corun"):
        for _ in range(st.steps):
            _decode(st)
        out["y_decode"] = st.yd
    if st.kind != "decode":
        out["y_prefill"] = st.yp
    if st.vocab:
        out["logits"] = st.logits
    return out


def work(case):
    """Weights, cached keys and values, and hidden states read once; appended keys and values and outputs written once."""
    sh = S.SHAPES[case["shape"]]
    d, f, hq, hkv, hd = sh.d_model, sh.ffn_dim, sh.n_q_heads, sh.n_kv_heads, sh.head_dim
    token = 2 * hkv * hd * 2
    lens, starts, ctx = _ints(case["prompts"]), _ints(case["starts"]), _contexts(case).astype(np.float64)
    starts = starts or [0] * len(lens)
    attn_params, ffn = d * sh.qkv_dim + sh.q_dim * d, 3 * d * f

    def dense(rows):
        if case["experts"]:
            active = min(case["experts"], 2 * rows)
            return 2 * (attn_params + active * ffn), 2 * rows * (attn_params + 2 * ffn)
        return 2 * (attn_params + ffn), 2 * rows * (attn_params + ffn)

    p_bytes = sum(n * 2 * 2 * d + (s + n) * token for n, s in zip(lens, starts))
    p_flops = sum(4 * hq * hd * (n * s + n * (n + 1) / 2) for n, s in zip(lens, starts))
    d_bytes = len(ctx) * 2 * 2 * d + float((ctx + 1).sum()) * token if len(ctx) else 0
    d_flops = 4 * hq * hd * float((ctx + 1).sum()) if len(ctx) else 0
    if case["kind"] == "hybrid":
        b, fl = dense(sum(lens) + len(ctx))
        b, fl = b + p_bytes + d_bytes, fl + p_flops + d_flops
    else:
        b = fl = 0
        if lens:
            w, x = dense(sum(lens))
            b, fl = b + w + p_bytes, fl + x + p_flops
        if len(ctx):
            w, x = dense(len(ctx))
            b, fl = b + case["steps"] * (w + d_bytes), fl + case["steps"] * (x + d_flops)
    b, fl = b * case["layers"], fl * case["layers"]
    if case["vocab"]:
        b += 2 * case["vocab"] * d + 4 * case["vocab"] * len(ctx)
        fl += 2 * case["vocab"] * d * len(ctx)
    return {"bytes": float(b), "flops": float(fl)}


def tolerance(case):
    """bf16 operands and stored intermediates, float32 sums.  Against a float64 evaluation of the same stack the outputs
    show a relative error of 0.005 after one layer, 0.006 after two, 0.008 (decode) to 0.012 (77-row prefill) after four,
    and a largest error of 0.03 to 0.05 of max(rms, value) (0.08 with experts); two evaluations of this precision differ by
    no more than twice that."""
    return {"rel": 0.008 + 0.004 * case["layers"], "max": 0.1 + 0.05 * case["layers"]}
