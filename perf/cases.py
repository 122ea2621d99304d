"""Performance cases: the calls that programs built on this library spend their time in.

Every case goes through the public binding, on models of this repository's own shapes (the tiny test model, the 7B shape
at full depth, the 13B widths at reduced depth) with synthetic weights.  The model is fixed, as it is in a serving
program: its handle is made once per process and kept.  What a seed changes is what a request brings: prompt lengths,
prompt ids, response lengths, draws.  Prompts and results are host arrays, as the library takes and returns them.

Kinds of work:
  decode    ss_forward_logits: a prompt forward, then one token per row and step (the caller supplies each next token);
            logits of every step.  The shape of a decode loop whose next tokens come from outside.
  prompt    ss_forward_logits: prompt forwards alone, logits of each prompt's last position.
  score     ss_forward_logits: every position's logits (perplexity, ranking).
  group     ss_run_group: schedule, generate every micro-batch, recompute the failures; then the logits that follow each
            whole response (one scoring call), as a program that ranks or continues its responses makes.
  generate  ss_generate_microbatch: sampled rows that end by themselves, polled by the host; then the same scoring call.

Weights: matrices ~ N(0, 0.02) like the repository's generator, the two matrices that write to the residual stream
smaller by 8 (the usual depth scaling), an embedding of unit variance, and a head that adds to its random rows a share of
the embedding of another token.  So the model is confident, as a trained one mostly is: after token t it says t + SHIFT
with a margin of several logits, and tokens do not hang on the last bits of near-ties.
"""
import functools

import numpy as np
import torch

from paper_2305_13144_amd import binding as ss
from paper_2305_13144_amd import synth

SHIFT = 7          # the head's favourite successor of token t is t + SHIFT
HEAD_SHARE = {"tiny": 0.06, "7b": 0.01, "13b-l8": 0.01}   # clear margins at each width, also at temperature 0.5

SHAPES = {
    "tiny": synth.TINY,
    "7b": synth.LLAMA7B,
    "13b-l8": synth.LLAMA13B.with_layers(8),   # the 13B widths; depth only repeats a layer
}


# ------------------------------------------------------------------------------------------------ cases
def listed():
    return [
        # The smallest whole call: the tiny model's group of 16, one vanilla micro-batch.  Launches and host latency.
        {"name": "tiny_group16", "kind": "group", "model": "tiny", "rows": 16, "plen": 19, "steps": 48, "vanilla": True},
        # One user alone: a single row's decode loop.
        {"name": "7b_decode_1row", "kind": "decode", "model": "7b", "rows": 1, "plen": 40, "steps": 24},
        # The baseline batch of 16 with ordinary prompts: the step that a scheduled group spends most of its time in.
        {"name": "7b_decode_16rows", "kind": "decode", "model": "7b", "rows": 16, "plen": 40, "steps": 24},
        # A wider batch, as variable batch sizes make for short responses; not a multiple of 16.
        {"name": "7b_decode_51rows", "kind": "decode", "model": "7b", "rows": 51, "plen": 24, "steps": 10},
        # A batch near the upper end of the variable batch sizes, odd.
        {"name": "7b_decode_163rows", "kind": "decode", "model": "7b", "rows": 163, "plen": 16, "steps": 6},
        # Long histories: long prompts, then a few steps over thousands of key/value slots.
        {"name": "7b_decode_long", "kind": "decode", "model": "7b", "rows": 3, "plen": 2400, "steps": 10},
        # The prompt forward of one baseline micro-batch.
        {"name": "7b_prompt_16", "kind": "prompt", "model": "7b", "rows": 16, "plen": 40},
        # The prompt forward of a large micro-batch: about 12 thousand token-rows.
        {"name": "7b_prompt_256", "kind": "prompt", "model": "7b", "rows": 256, "plen": 40},
        # Scoring: every position's logits of a few sequences.
        {"name": "7b_score_6", "kind": "score", "model": "7b", "rows": 6, "plen": 75},
        # The wider model: two strips of rows.
        {"name": "13b_decode_24rows", "kind": "decode", "model": "13b-l8", "rows": 24, "plen": 60, "steps": 16},
        # Sampled rows that end by themselves (temperature 0.5, the paper's), the host polling.
        {"name": "7b_generate_16", "kind": "generate", "model": "7b", "rows": 16, "plen": 40, "steps": 40},
        # The whole scheduled pipeline: bins, failure recomputation, variable batch size, compaction, lanes in flight.
        {"name": "7b_group_64", "kind": "group", "model": "7b", "rows": 64, "plen": 40, "steps": 48, "vanilla": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prompt", "prompt", "score", "generate", "group"])
    model = rng.choice(["7b", "7b", "7b", "13b-l8", "tiny"])
    if kind == "decode":
        if rng.random() < 0.25:
            return {"kind": kind, "model": model, "rows": rng.randint(1, 4), "plen": _log_int(rng, 300, 2000), "steps": rng.randint(4, 12)}
        rows = _log_int(rng, 1, 256)
        return {"kind": kind, "model": model, "rows": rows, "plen": rng.randint(8, 60), "steps": rng.randint(4, 24) if rows < 48 else rng.randint(3, 8)}
    if kind == "prompt":
        return {"kind": kind, "model": model, "rows": _log_int(rng, 1, 256), "plen": rng.randint(9, 48)}
    if kind == "score":
        return {"kind": kind, "model": model, "rows": rng.randint(1, 9), "plen": rng.randint(20, 90)}
    if kind == "generate":
        return {"kind": kind, "model": model, "rows": _log_int(rng, 1, 64), "plen": rng.randint(9, 60), "steps": rng.randint(8, 40)}
    return {"kind": kind, "model": model, "rows": _log_int(rng, 8, 56), "plen": rng.randint(9, 50), "steps": rng.randint(16, 44), "vanilla": rng.random() < 0.3}


# ------------------------------------------------------------------------------------------------ the model
@functools.lru_cache(maxsize=None)
def _pool(count):
    """Seeded N(0, 0.02) bf16 values; every matrix is a window of this pool."""
    children = np.random.SeedSequence(20230513).spawn((count + (1 << 22) - 1) >> 22)

    def one(child):
        v = np.random.Generator(np.random.PCG64(child)).standard_normal(1 << 22, dtype=np.float32)
        return synth.f32_to_bf16_bits(v * np.float32(0.02))

    from concurrent.futures import ThreadPoolExecutor
    with ThreadPoolExecutor(max_workers=8) as ex:
        return np.concatenate(list(ex.map(one, children)))[:count]


def _scaled(bits, factor):
    """bf16 bit patterns times a factor, rounded to bf16."""
    out = np.empty_like(bits)
    for r0 in range(0, len(bits), 1 << 22):
        out[r0:r0 + (1 << 22)] = synth.f32_to_bf16_bits(synth.bf16_bits_to_f32(bits[r0:r0 + (1 << 22)]) * np.float32(factor))
    return out


@functools.lru_cache(maxsize=None)
def _tensors(model):
    """The model's tensors (bf16 bit patterns) in the library's order."""
    shape = SHAPES[model]
    d, f, v = shape.d_model, shape.d_ffn, shape.vocab
    slack = 1 << 20
    pool = _pool(max(v * d, f * d) + slack)
    small = _scaled(pool[:f * d + slack], 0.125)
    embed = _scaled(pool[:v * d], 50.0).reshape(v, d)
    odd = slack - 12345   # not a multiple of the width: the noise rows are nobody's embedding
    head = np.empty((v, d), np.uint16)
    for r0 in range(0, v, 2048):
        r1 = min(v, r0 + 2048)
        e = synth.bf16_bits_to_f32(embed[(np.arange(r0, r1) - SHIFT) % v])
        noise = synth.bf16_bits_to_f32(pool[odd + r0 * d:odd + r1 * d].reshape(r1 - r0, d))
        head[r0:r1] = synth.f32_to_bf16_bits(noise + np.float32(HEAD_SHARE[model]) * e)
    starts = np.random.Generator(np.random.PCG64(20230517))
    out = []
    for name, shp in shape.tensor_specs():
        if name == "embed":
            out.append(embed)
        elif name == "lm_head":
            out.append(head)
        elif len(shp) == 1:
            out.append(synth.f32_to_bf16_bits(1.0 + 0.1 * starts.standard_normal(shp[0]).astype(np.float32)))
        else:
            src = small if name.endswith((".wo", ".wd")) else pool
            n = shp[0] * shp[1]
            at = int(starts.integers(0, len(src) - n + 1))
            out.append(src[at:at + n].reshape(shp))
    return out


@functools.lru_cache(maxsize=None)
def _handle(model):
    return ss.Weights(SHAPES[model], _tensors(model))


# ------------------------------------------------------------------------------------------------ a request
def _lognormal(rng, n, median, sigma, lo, hi):
    return np.clip(np.rint(median * np.exp(sigma * rng.standard_normal(n))), lo, hi).astype(np.int32)


def _request(case, seed):
    """Host data of one request.  The total of the lengths varies little between seeds: the spread is a fixed set of
    lognormal lengths in another order."""
    shape = SHAPES[case["model"]]
    fixed = np.random.Generator(np.random.PCG64([case["rows"], case["plen"], 11]))
    rng = np.random.Generator(np.random.PCG64([int(seed), case["rows"], 12]))
    rows, steps = case["rows"], case.get("steps", 0)
    long = case["plen"] >= 300
    plens = _lognormal(fixed, rows, case["plen"], 0.2 if long else 0.6, 8, 3900 if long else 256)
    plens = plens[rng.permutation(rows)]
    offs = np.concatenate([[0], np.cumsum(plens)]).astype(np.int32)
    prompts = [rng.integers(0, shape.vocab, p).astype(np.int32) for p in plens]
    r = {"plens": plens, "offs": offs, "prompts": prompts, "flat": np.concatenate(prompts)}
    if case["kind"] == "decode":
        seqs = [np.concatenate([p, rng.integers(0, shape.vocab, steps).astype(np.int32)]) for p in prompts]
        r["tokens"], r["seq_offs"] = np.concatenate(seqs), (offs + steps * np.arange(rows + 1)).astype(np.int32)
        r["seqs"] = seqs
    if case["kind"] in ("group", "generate"):
        tl = _lognormal(fixed, rows, 0.4 * steps, 0.7, 1, steps)
        tl[0] = steps
        order = rng.permutation(rows)
        r["targets"] = tl[order]
        noise = np.exp(0.3 * fixed.standard_normal(rows))
        r["preds"] = np.maximum(1, np.rint(tl * noise)).astype(np.int32)[order]
        # what the confident model answers: t, t + SHIFT, t + 2 * SHIFT, ...
        r["answers"] = [((int(p[-1]) + SHIFT * np.arange(1, n + 1)) % shape.vocab).astype(np.int32)
                        for p, n in zip(prompts, r["targets"])]
    return r


def prepare(case, seed):
    state = {"case": case, "w": _handle(case["model"]), **_request(case, seed)}
    if case["kind"] == "group":
        if case["vanilla"]:
            state["policy"] = ss.make_policy((), 16, case["steps"], 256)
        else:
            state["policy"] = ss.make_policy(("SORT", "BIN", "FCR", "VBS", "COMPACT"), 16, case["steps"], 256)
    if case["kind"] == "generate":
        state["seed"] = int(seed) + 1
    return state


def _score_responses(state, tokens, lens):
    """The logits that follow each whole response."""
    seqs = [np.concatenate([p, tokens[i, :lens[i]]]) for i, p in enumerate(state["prompts"])]
    n = np.array([len(q) for q in seqs], np.int32)
    offs = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    return ss.ss_forward_logits(state["w"], np.concatenate(seqs), offs, n)


def run(state):
    case, w = state["case"], state["w"]
    kind = case["kind"]
    if kind == "decode":
        return {"logits": ss.ss_forward_logits(w, state["tokens"], state["seq_offs"], state["plens"])}
    if kind == "prompt":
        return {"logits": ss.ss_forward_logits(w, state["flat"], state["offs"], state["plens"])}
    if kind == "score":
        return {"logits": ss.ss_forward_logits(w, state["flat"], state["offs"], state["plens"], all_prompt_logits=True)}
    if kind == "generate":
        r = ss.ss_generate_microbatch(w, state["flat"], state["offs"], case["steps"], temperature=0.5, seed=state["seed"],
                                      target_lens=state["targets"], sync_every=1, flags=ss.SS_COMPACT)
        return {"tokens": r["tokens"], "lens": r["lens"], "failed": r["failed"],
                "logits": _score_responses(state, r["tokens"], r["lens"])}
    r = ss.ss_run_group(w, state["flat"], state["offs"], state["targets"], None if case["vanilla"] else state["preds"],
                        0 if case["vanilla"] else 10, state["policy"])
    return {"tokens": r["tokens"], "lens": r["lens"], "logits": _score_responses(state, r["tokens"], r["lens"])}


# ------------------------------------------------------------------------------------------------ work
def _forward_work(shape, rows, kv_read, logit_rows):
    """(bytes, flops) of one forward of `rows` token-rows that reads `kv_read` cached slots; the pairs of attention apart."""
    d, f, v = shape.d_model, shape.d_ffn, shape.vocab
    layer = 4 * d * d + 3 * d * f
    kv = shape.kv_bytes_per_token()
    nbytes = (shape.n_layers * (layer + 2 * d) + v * d + d) * 2 + kv_read * kv + rows * (kv + 2 * d + 4) + logit_rows * v * 4
    return nbytes, 2.0 * (shape.n_layers * layer * rows + v * d * logit_rows)


def work(case):
    shape = SHAPES[case["model"]]
    r = _request(case, 0)
    plens = r["plens"].astype(np.int64)
    pair_flops = 4.0 * shape.d_model * shape.n_layers   # per (query, slot): scores and the weighted sum
    total = np.zeros(2)

    def prompt(lens, logit_rows):
        b, fl = _forward_work(shape, int(lens.sum()), 0, logit_rows)
        total[:] += (b, fl + pair_flops * float((lens * (lens + 1) // 2).sum()))

    def step(ctx, logit_rows):
        b, fl = _forward_work(shape, len(ctx), int(ctx.sum()), logit_rows)
        total[:] += (b, fl + pair_flops * float(ctx.sum()))

    if case["kind"] in ("prompt", "score"):
        prompt(plens, int(plens.sum()) if case["kind"] == "score" else len(plens))
    elif case["kind"] == "decode":
        prompt(plens, len(plens))
        for g in range(1, case["steps"] + 1):
            step(plens + g, len(plens))
    else:
        # every micro-batch of the schedule streams the model once per forward; rows leave when they are done
        targets = r["targets"].astype(np.int64)
        if case["kind"] == "generate":
            plan = [(list(range(case["rows"])), case["steps"])]
        elif case["vanilla"]:
            plan = ss.ss_schedule(None, case["rows"], 0, ss.make_policy((), 16, case["steps"], 256))
        else:
            pol = ss.make_policy(("SORT", "BIN", "FCR", "VBS", "COMPACT"), 16, case["steps"], 256)
            plan = ss.ss_schedule(r["preds"], case["rows"], 10, pol)
            failed = [i for idx, cap in plan for i in idx if targets[i] > cap]
            plan = plan + (ss.ss_schedule_failures(r["preds"], case["rows"], sorted(failed), 10, pol) if failed else [])
        for idx, cap in plan:
            t = np.minimum(targets[idx], cap)
            prompt(plens[idx], 0)
            for g in range(1, int(t.max())):
                step((plens[idx] + g)[t > g], 0)
        prompt(plens + targets, len(plens))   # the scoring call
        total[0] += case["rows"] * case["steps"] * 4
    return {"bytes": float(total[0]), "flops": float(total[1])}


# Relative error of the logits.  Activations are rounded to 11 significand bits once per projection input and cached keys
# and values likewise: measured against 64 bits 1.9e-4 (tiny), 6.5e-4 (7B), 4.9e-4 (13B widths, 8 layers), and four times
# that.  Tokens, lengths and flags are whole numbers and decided by margins of several logits: no share may differ.
_REL = {"tiny": 8e-4, "7b": 2.6e-3, "13b-l8": 2e-3}


def tolerance(case):
    return {"rel": _REL[case["model"]]}


# ------------------------------------------------------------------------------------------------ 64 bits
def _reference(model, seqs, want):
    """Logits of positions want[i] (a slice) of every sequence, in 64 bits with plain torch operations."""
    shape = SHAPES[model]
    dev = "cuda"
    d, hn, hd, f = shape.d_model, shape.n_heads, shape.head_dim, shape.d_ffn
    tens = iter(_tensors(model))

    def mat(bits):
        return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(dev).view(torch.bfloat16).double()

    lens = [len(q) for q in seqs]
    offs = np.concatenate([[0], np.cumsum(lens)])
    pos = torch.cat([torch.arange(n) for n in lens]).to(dev).double()
    inv = shape.rope_base ** (-2.0 * torch.arange(hd // 2, device=dev, dtype=torch.float64) / hd)
    cos, sin = torch.cos(pos[:, None] * inv)[:, None, :], torch.sin(pos[:, None] * inv)[:, None, :]
    embed = next(tens)
    x = mat(embed[np.concatenate(seqs)])

    def norm(z, g):
        return z * torch.rsqrt((z * z).mean(-1, keepdim=True) + shape.rms_eps) * g

    def rotate(z):
        z = z.view(-1, hn, hd)
        a, b = z[..., :hd // 2], z[..., hd // 2:]
        return torch.cat([a * cos - b * sin, a * sin + b * cos], -1)

    for _ in range(shape.n_layers):
        h = norm(x, mat(next(tens)))
        q, k = rotate(h @ mat(next(tens)).T), rotate(h @ mat(next(tens)).T)
        v = (h @ mat(next(tens)).T).view(-1, hn, hd)
        att = torch.empty_like(q)
        for i, n in enumerate(lens):
            s = slice(int(offs[i]), int(offs[i + 1]))
            qi, ki, vi = (z[s].transpose(0, 1).contiguous() for z in (q, k, v))
            mask = torch.ones(n, n, dtype=torch.bool, device=dev).triu(1)
            p = torch.matmul(qi, ki.transpose(1, 2).contiguous()) * hd ** -0.5
            p = torch.softmax(p.masked_fill(mask, float("-inf")), -1)
            att[s] = torch.matmul(p, vi).transpose(0, 1)
        x = x + att.reshape(-1, d) @ mat(next(tens)).T
        h = norm(x, mat(next(tens)))
        g, u = h @ mat(next(tens)).T, h @ mat(next(tens)).T
        x = x + (torch.nn.functional.silu(g) * u) @ mat(next(tens)).T
    keep = torch.cat([torch.arange(int(offs[i]), int(offs[i + 1]))[w] for i, w in enumerate(want)]).to(dev)
    h = norm(x[keep], mat(next(tens)))
    return h @ mat(next(tens)).T


def exact(case, seed):
    r = _request(case, seed)
    kind = case["kind"]
    if int(r["plens"].sum()) * SHAPES[case["model"]].n_layers > 32 * 13000:
        return None
    if kind == "decode":
        return {"logits": _reference(case["model"], r["seqs"], [slice(int(p) - 1, None) for p in r["plens"]])}
    if kind == "prompt":
        return {"logits": _reference(case["model"], r["prompts"], [slice(-1, None)] * case["rows"])}
    if kind == "score":
        return {"logits": _reference(case["model"], r["prompts"], [slice(None)] * case["rows"])}
    seqs = [np.concatenate([p, a]) for p, a in zip(r["prompts"], r["answers"])]
    out = {"tokens": None, "lens": None, "logits": _reference(case["model"], seqs, [slice(-1, None)] * case["rows"])}
    if kind == "generate":
        out["failed"] = None
    return out
