"""The work that the speculative-verification library is given in use, as timed cases.

Two kinds of pass, both through the public Python entry points:

* ``round``: one rollout round -- ``verify_step`` over the whole batch, then ``kv_commit`` of its own decisions.  With
  budgets of zero this is plain decoding.  A last ``seq_rewind`` puts the sequences back to where they were, so that the
  same pass can run again; it is host bookkeeping of a few integers per sequence.
* ``prefill``: a batch of prompts enters the KV cache (``prefill``) and its sequences are released again (``seq_free``).

Model shapes, context-length recipes and draft-budget recipes are the ones of ``das_inputs.workloads`` (the tiny, 1.5B and 7B
shapes; ``range`` is log-uniform between two bounds).  Greedy drafts are the model's own plain continuation with every token
kept with probability ``accept``, as the repository's benchmark proposes them; sampled rounds force an acceptance with the
same probability and judge the other drafts honestly.
"""
import dataclasses
import math

import numpy as np

import das_inputs as di
import paper_2511_13841_amd as das

DEFAULTS = {
    "kind": "round",        # "round" or "prefill"
    "model": "7b",          # a key of das_inputs.MODELS
    "batch": 1,             # sequences
    "contexts": "range",    # recipe of the context (or prompt) lengths; "range": log-uniform in [lo, hi]
    "lo": 0,
    "hi": 0,
    "lengths_seed": 1,      # the lengths belong to the case, everything else is drawn from prepare()'s seed
    "budgets": "k0",        # recipe of the draft budgets ("k4": four drafts each)
    "accept": 0.7,          # share of draft tokens that are the target's own
    "temperature": 0.0,     # 0: greedy; above: sampling at this temperature
    "logits": False,        # keep the pass's logits and read them back (log-probabilities for training, inspection)
}


def _case(name=None, **kw):
    c = dict(DEFAULTS, **kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: a unit-test-sized model, four short sequences.  Launches and host work are all of it.  Its vocabulary is
        # small enough that every pass has its logits, and a caller of this size looks at them.
        _case("tiny round logits", model="tiny", batch=4, contexts="uniform16_64", lengths_seed=1001, budgets="k4", logits=True),
        # The end of a rollout: most sequences have finished, the few long ones left are decoded without a drafter.
        _case("1.5b decode last few", model="1.5b", batch=6, lo=1024, hi=8192, lengths_seed=11),
        # A training step that wants the log-probabilities of a few verified tokens; odd sizes.
        _case("1.5b round logits", model="1.5b", batch=3, lo=200, hi=2000, lengths_seed=12, budgets="k3", logits=True),
        # Plain sampling of a batch of short responses at the temperature of the paper's runs.
        _case("1.5b decode sampled", model="1.5b", batch=24, contexts="pareto512", lengths_seed=13, temperature=0.6),
        # The repository's second workload: uniform short chains over a lognormal batch.
        _case("1.5b round batch 64", model="1.5b", batch=64, contexts="lognormal2048", lengths_seed=1002, budgets="k4", accept=0.6),
        # Plain decoding in the middle of a rollout (class "short" of the budget policy: no speculation).
        _case("7b decode batch 64", batch=64, contexts="pareto512", lengths_seed=14),
        # Stragglers: three sequences left, long contexts, long chains.
        _case("7b round stragglers", batch=3, lo=16384, hi=32768, lengths_seed=15, budgets="k16", accept=0.8),
        # The benchmark's headline workload: long-tailed batch, budgets by length quartile.
        _case("7b round long-tail batch", batch=128, contexts="mix_1k4k_16k32k", lengths_seed=1003, budgets="quartile"),
        # The benchmark's tail workload: sixteen contexts of 32k to 64k tokens.
        _case("7b round 32k-64k contexts", batch=16, contexts="uniform32k_64k", lengths_seed=1004, budgets="k16", accept=0.8),
        # The benchmark's stochastic workload: a large batch, budgets that grow with the logarithm of the length.
        _case("7b round sampled", batch=256, contexts="pareto512", lengths_seed=1005, budgets="loglen", temperature=1.0),
        # The start of a rollout: a batch of ordinary prompts.
        _case("1.5b prefill prompts", kind="prefill", model="1.5b", batch=32, lo=60, hi=1500, lengths_seed=16),
        # Long prompts (re-prefilled contexts after a weight update); the largest case.
        _case("7b prefill long", kind="prefill", batch=3, lo=4000, hi=16384, lengths_seed=17),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the same models, both kinds of pass, any batch, context and budget up to the listed extremes."""
    model = rng.choice(["tiny", "1.5b", "1.5b", "7b", "7b"])
    seed = rng.randrange(1 << 20)
    temperature = rng.choice([0.0, 0.0, 0.0, 0.6, 1.0])
    if rng.random() < 0.25:
        hi = _log_uniform(rng, 32, {"tiny": 2048, "1.5b": 16384, "7b": 12000}[model])
        lo = max(1, int(hi * rng.uniform(0.1, 0.9)))
        batch = max(1, min(_log_uniform(rng, 1, 96), 24000 // hi))
        return _case(kind="prefill", model=model, batch=batch, lo=lo, hi=hi, lengths_seed=seed, temperature=temperature)
    hi = _log_uniform(rng, 48, {"tiny": 2048, "1.5b": 32768, "7b": 65000}[model])
    lo = max(16, int(hi * rng.uniform(0.1, 0.9)))
    batch = max(1, min(_log_uniform(rng, 1, {"tiny": 64, "1.5b": 160, "7b": 256}[model]), 700000 // hi))
    budgets = rng.choice(["k0", "quartile", "loglen", "k%d" % rng.randint(1, 16), "k%d" % rng.randint(1, 16)])
    if budgets[0] == "k":
        budgets = "k%d" % min(int(budgets[1:]), 1600 // batch - 1)
    c = _case(model=model, batch=batch, lo=lo, hi=hi, lengths_seed=seed, budgets=budgets, accept=round(rng.uniform(0.5, 0.9), 3),
              temperature=temperature)
    c["logits"] = temperature == 0 and budgets[0] == "k" and batch * (int(budgets[1:]) + 1) <= 16 and rng.random() < 0.5
    return c


def _lengths(case):
    if case["contexts"] == "range":
        rng = np.random.default_rng(case["lengths_seed"])
        return np.rint(np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), case["batch"]))).astype(np.int32)
    wl = dataclasses.replace(di.workload("c1"), lengths=case["contexts"], batch=case["batch"])
    return di.context_lengths(wl, seed=case["lengths_seed"])


def _budgets(case, lengths):
    return di.draft_budgets(dataclasses.replace(di.workload("c1"), budgets=case["budgets"]), lengths)


def _prepare_prefill(case, shape, lengths, seed):
    pages = int(sum(-(-int(n) // 16) for n in lengths)) + 8
    max_ctx = -(-int(lengths.max()) // 16) * 16 + 16
    model = das.DasModel(das.config_for(shape, max_seqs=case["batch"], max_ctx=max_ctx, max_rows=2048, max_draft=0, num_pages=pages),
                         None, seed=seed)
    rng = np.random.default_rng([seed, 2])
    sampling = (case["temperature"], None, rng.random(case["batch"], dtype=np.float32)) if case["temperature"] else None
    return {"kind": "prefill", "model": model, "ids": np.arange(case["batch"], dtype=np.int32),
            "prompts": di.prompts(lengths, shape.vocab, seed), "sampling": sampling}


def _continuations(model, ids, lengths, pending, steps):
    """The next `steps` tokens of every sequence by plain decoding; the sequences are put back afterwards."""
    out = np.empty((len(ids), steps), np.int32)
    for t in range(steps):
        acc, nxt = model.verify_step(ids, lengths + t, [[] for _ in ids])
        model.kv_commit(ids, acc, nxt)
        out[:, t] = nxt
    model.seq_rewind(ids, lengths, pending)
    return out


def _prepare_round(case, shape, lengths, seed):
    n, ks = case["batch"], _budgets(case, lengths)
    kmax = int(ks.max())
    pages = int(sum(-(-(int(c) + kmax + 2) // 16) for c in lengths)) + 8
    max_ctx = -(-(int(lengths.max()) + kmax + 2) // 16) * 16 + 16
    model = das.DasModel(das.config_for(shape, max_seqs=n, max_ctx=max_ctx, max_rows=max(int((ks + 1).sum()), 16), max_draft=kmax,
                                        num_pages=pages), None, keep_logits=case["logits"], seed=seed)
    rng = np.random.default_rng([seed, 1])
    ids = np.arange(n, dtype=np.int32)
    pending = rng.integers(0, shape.vocab, size=n, dtype=np.int32)
    for i in range(n):
        model.seq_create(i, int(lengths[i]), int(pending[i]))
        model.kv_synth(i, seed, i)
    drafts = rng.integers(0, shape.vocab, size=(n, kmax), dtype=np.int32)
    sampling = None
    if case["temperature"]:
        rows = int((ks + 1).sum())
        forced = rng.random(rows) < case["accept"]
        u_accept = np.where(forced, 0.0, rng.random(rows)).astype(np.float32)
        sampling = (case["temperature"], u_accept, rng.random(rows, dtype=np.float32))
    elif kmax:
        own = rng.random((n, kmax)) < case["accept"]
        drafts = np.where(own, _continuations(model, ids, lengths, pending, kmax), drafts)
    return {"kind": "round", "model": model, "ids": ids, "lengths": lengths, "pending": pending, "logits": case["logits"],
            "drafts": [drafts[i, :ks[i]] for i in range(n)], "sampling": sampling}


def prepare(case, seed):
    case = dict(DEFAULTS, **case)
    shape, lengths = di.MODELS[case["model"]], _lengths(case)
    return (_prepare_prefill if case["kind"] == "prefill" else _prepare_round)(case, shape, lengths, seed)


def run(state):
    m, ids = state["model"], state["ids"]
    if state["kind"] == "prefill":
        pending = m.prefill(ids, state["prompts"], state["sampling"])
        m.seq_free(ids)
        return {"pending": pending}
    accepted, following = m.verify_step(ids, state["lengths"], state["drafts"], state["sampling"])
    out = {"accepted": accepted, "next": following}
    if state["logits"]:
        out["logits"] = m.debug_logits()
    m.kv_commit(ids, accepted, following)
    m.seq_rewind(ids, state["lengths"], state["pending"])
    return out


def work(case):
    """Every matrix once (the LM head for the rows that get logits), every visible K and V once, the new rows' K and V written;
    two operations per multiply-add of the matrices and of causal attention."""
    case = dict(DEFAULTS, **case)
    s, c = di.MODELS[case["model"]], _lengths(case).astype(np.float64)
    head = s.vocab * s.d_model
    weights = s.n_layers * s.layer_params + head
    per_key = 4.0 * s.n_layers * s.n_q_heads * s.head_dim           # operations of one query row on one key
    if case["kind"] == "prefill":
        rows, scored, read, keys = c.sum(), len(c), 0.0, (c * (c + 1) / 2).sum()
    else:
        n = _budgets(case, _lengths(case)).astype(np.float64) + 1
        rows, scored, read, keys = n.sum(), n.sum(), c.sum(), (n * c + n * (n + 1) / 2).sum()
    out = 4.0 * scored * s.vocab if case["logits"] else 0.0
    return {"bytes": 2.0 * weights + (read + rows) * s.kv_bytes_per_token + out,
            "flops": 2.0 * (rows * s.n_layers * s.layer_params + scored * head) + per_key * keys}


def tolerance(case):
    """Logits: bf16 activations through 28 layers.  The same arithmetic with its sums in another order (fp32 matrix products of the
    same rounded operands) differs by 2.3e-2 in the 2-norm and 0.12 at most, the path without roundings in 64 bits by 2.1e-2; two
    layers differ by a quarter of that.  Decisions are whole numbers; the library defines the order of every sum, so that a row's
    decision does not depend on the batch around it: they may differ only where two candidates tie."""
    return {"rel": 0.03 if di.MODELS[case["model"]].n_layers > 4 else 0.02, "max": 0.5, "differ": 0.01}
