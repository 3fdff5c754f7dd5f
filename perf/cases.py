"""What a program built on this library has it do, as cases to be timed: the verification pass on both model shapes,
from one interactive trace to the ragged batch of 128, the pass that writes its tokens into the cache, candidates on a
shared context, greedy generation and the two-tier cascade.

The models are the ones of confspec_workloads (random weights, no checkpoint exists for them).  A program loads its
models once, so they are kept here from case to case; batches, caches and token ids are new with every seed.

Random weights alone would decide most steps by a few thousandths of a logit, which no trained verifier does and which
makes a decision depend on the rounding of the last bit.  As in a real cache the values of a trace therefore have a
mean of their own (its "topic"), and the head's rows of the verdict tokens, and of one token per topic, point along
what that mean adds to the hidden state: decisions are clear (confidence about 0.99, or about 0.75 for the unsure ones),
and so is the greedy next token.
"""
import random
from types import SimpleNamespace

import numpy as np
import torch

import confspec_workloads as W
from paper_2602_18447_amd.runner import Cascade, Verifier

DEVICE = "cuda:0"
SHAPES = {"tiny": W.config(1).model, "draft": W.config(2).model, "target": W.config(5).model}
BLOCK = 16
KV_STD = 0.5
N_TOPICS = 8                        # two of each kind, in the order of LEANS
LEANS = (5.0, -5.0, 1.1, -0.6)      # logit of "accept" minus logit of "reject": sure yes, sure no, unsure
KINDS = (0.55, 0.15, 0.20, 0.10)    # how often a trace is of each kind
# length of the hidden state's component along its topic, after the final norm, for long contexts (measured)
ALONG = {"tiny": 14.0, "draft": 22.0, "target": 14.0}
GAMMA = 0.9


def listed():
    return [
        # the fp32 configuration: the smallest call there is, all latency
        dict(name="verify_tiny_fp32", do="verify", model="tiny", B=4, L_lo=128, L_hi=128, S_lo=32, S_hi=32, n_tau=1),
        # one user's trace: a drafted step and the prompt on a context of ordinary length, the user waits for it
        dict(name="verify_one_trace", do="verify", model="draft", B=1, L_lo=2048, L_hi=2048, S_lo=96, S_hi=96, n_tau=1),
        # the ordinary serving batch
        dict(name="verify_b32", do="verify", model="draft", B=32, L_lo=2048, L_hi=2048, S_lo=96, S_hi=96, n_tau=1),
        # long chains of thought, thresholds swept in one call
        dict(name="verify_b64_long", do="verify", model="draft", B=64, L_lo=8192, L_hi=8192, S_lo=128, S_hi=128, n_tau=3),
        # a full GPU: 128 traces of any length
        dict(name="verify_b128_ragged", do="verify", model="draft", B=128, L_lo=512, L_hi=16384, S_lo=32, S_hi=256, n_tau=1),
        # the large model on the traces that were escalated to it
        dict(name="verify_target_b16", do="verify", model="target", B=16, L_lo=4096, L_hi=4096, S_lo=96, S_hi=96, n_tau=1),
        # tree-structured drafting: four candidates for the next step of each of eight requests, short steps of uneven length
        dict(name="verify_candidates", do="shared", model="draft", B=32, group=4, L_lo=1024, L_hi=4096, S_lo=16, S_hi=48, n_tau=1),
        # accepted steps join the context: the pass writes its keys and values into the cache (a chunk of prefill)
        dict(name="append_chunk", do="append", model="draft", B=16, L_lo=512, L_hi=1536, S_lo=512, S_hi=512, n_tau=1),
        # the small model drafts: one user, and a serving batch
        dict(name="generate_one", do="generate", model="draft", B=1, L_lo=4096, L_hi=4096, steps=16),
        dict(name="generate_b32", do="generate", model="draft", B=32, L_lo=2048, L_hi=2048, steps=16),
        # the large model writes the step itself where the draft was rejected
        dict(name="generate_target_b8", do="generate", model="target", B=8, L_lo=1024, L_hi=4096, steps=4),
        # the cascade over both models: requests of one to five drafted steps
        dict(name="cascade_b32", do="cascade", model="draft", B=32, L_lo=2048, L_hi=2048, S_lo=96, S_hi=96),
    ]


def draw(rng):
    def log_int(lo, hi):
        return min(hi, max(lo, round(lo * (hi / lo) ** rng.random())))

    def span(lo, hi):
        a = log_int(lo, hi)
        return (a, a) if rng.random() < 0.25 else (max(lo, int(a * rng.uniform(0.1, 1.0))), a)

    do = rng.choice(("verify",) * 5 + ("shared", "append", "append") + ("generate",) * 4 + ("cascade",))
    if do == "verify":
        model = rng.choice(("tiny", "draft", "draft", "draft", "target"))
        b, l, s = {"tiny": ((1, 16), (16, 512), (4, 64)), "draft": ((1, 128), (512, 16384), (16, 256)),
                   "target": ((1, 16), (512, 4096), (32, 128))}[model]
        (l_lo, l_hi), (s_lo, s_hi) = span(*l), span(*s)
        c = dict(do=do, model=model, B=log_int(*b), L_lo=l_lo, L_hi=l_hi, S_lo=s_lo, S_hi=s_hi, n_tau=rng.choice((1, 1, 3)))
    elif do == "shared":
        group = rng.randint(2, 5)
        (l_lo, l_hi), (s_lo, s_hi) = span(512, 8192), span(8, 96)
        c = dict(do=do, model="draft", B=group * log_int(1, 16), group=group, L_lo=l_lo, L_hi=l_hi, S_lo=s_lo, S_hi=s_hi, n_tau=1)
    elif do == "append":
        (l_lo, l_hi), (s_lo, s_hi) = span(256, 4096), span(64, 512)
        c = dict(do=do, model="draft", B=log_int(1, 32), L_lo=l_lo, L_hi=l_hi, S_lo=s_lo, S_hi=s_hi, n_tau=1)
    elif do == "generate":
        model = rng.choice(("draft", "draft", "draft", "target"))
        l_lo, l_hi = span(512, 8192 if model == "draft" else 4096)
        c = dict(do=do, model=model, B=log_int(1, 64 if model == "draft" else 16), L_lo=l_lo, L_hi=l_hi,
                 steps=rng.randint(4, 16) if model == "draft" else rng.randint(2, 6))
    else:
        (l_lo, l_hi), (s_lo, s_hi) = span(512, 4096), span(32, 128)
        c = dict(do=do, model="draft", B=log_int(2, 32), L_lo=l_lo, L_hi=l_hi, S_lo=s_lo, S_hi=s_hi)
    largest = max(_price(x) for x in listed())
    while _price(c) > largest or c["B"] * (c["L_lo"] + c["L_hi"]) > 2_200_000:      # no larger than the largest listed one
        step = c.get("group", 1)
        c["B"] = max(step, c["B"] * 3 // 4 // step * step)
    return c


# ---------------------------------------------------------------------------------------------------------------------
# what follows from the case alone: lengths, kinds of traces, requests, work
# ---------------------------------------------------------------------------------------------------------------------
def _rng(case, what):
    return random.Random(what + repr(sorted((k, v) for k, v in case.items() if k != "name")))


def _lengths(case):
    r = _rng(case, "lengths")
    group = case.get("group", 1)
    L = [r.randint(case["L_lo"], case["L_hi"]) for _ in range(case["B"] // group)]
    L = [v for v in L for _ in range(group)]
    S = [1] * case["B"] if case["do"] == "generate" else [r.randint(case["S_lo"], case["S_hi"]) for _ in range(case["B"])]
    return L, S


def _kinds(case):
    r = _rng(case, "kinds")
    group = case.get("group", 1)
    return [k for _ in range(case["B"] // group) for k in [r.choices(range(4), KINDS)[0]] * group]


def _requests(case):
    starts, k = [0], 1
    while starts[-1] < case["B"]:
        starts.append(min(starts[-1] + k, case["B"]))
        k = k % 5 + 1
    return starts


def _escalated(case):
    """The traces that the large model's pass holds: unsure, and no step before them surely rejected."""
    kinds, starts = _kinds(case), _requests(case)
    return [b for lo, hi in zip(starts, starts[1:]) for b in range(lo, hi) if kinds[b] >= 2 and 1 not in kinds[lo:b]]


def _layer_params(m):
    return m.d_model * ((2 * m.n_q_heads + 2 * m.n_kv_heads) * m.head_dim + 3 * m.d_ffn)


def _pass_work(m, L, S, contexts, append=False, head=False):
    """One pass: every weight read once, every cached context once, the last layer's rows only where they are needed."""
    size = 4 if m.dtype == "fp32" else 2
    T, B, n = sum(S), len(S), m.n_layers
    qw, kw = m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim
    row_key = 4.0 * m.n_q_heads * m.head_dim
    attn = row_key * ((n - 1) * sum(s * (l + (s + 1) / 2) for l, s in zip(L, S)) + sum(l + s for l, s in zip(L, S)))
    rows = (n - 1) * T + B
    flops = 2.0 * m.d_model * (n * T * (qw + 2 * kw) + rows * (qw + 3 * m.d_ffn)) + attn
    moved = size * (n * _layer_params(m) + 2 * n * kw * sum(contexts) + m.d_model * (T + (m.vocab if head else 2)))
    if head:
        flops += 2.0 * B * m.d_model * m.vocab
    if append:
        moved += size * 2 * n * kw * T
    return moved, flops


def work(case):
    m = SHAPES[case["model"]]
    L, S = _lengths(case)
    if case["do"] == "generate":
        parts = [_pass_work(m, [l + i for l in L], S, [l + i for l in L], True, True) for i in range(case["steps"])]
    elif case["do"] == "cascade":
        up = _escalated(case)
        parts = [_pass_work(m, L, S, L)]
        if up:
            l_up = [L[b] for b in up]
            parts.append(_pass_work(SHAPES["target"], l_up, [S[b] for b in up], l_up))
    else:
        parts = [_pass_work(m, L, S, L[::case.get("group", 1)], case["do"] == "append")]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def _price(case):
    w = work(case)
    return w["bytes"] / 8e12 + w["flops"] / 2.5e15


def tolerance(case):
    """bf16 activations through 28 or 64 layers leave a relative error of some 1e-3 in the logits; fp32 sums 1e-5.
    Decisions are clear of their thresholds, so whole values hardly ever differ."""
    if case["model"] == "tiny":
        return {"rel": 3e-5, "max": 1e-3, "differ": 0.002}
    return {"rel": 1e-2, "max": 0.2, "differ": 0.01}


# ---------------------------------------------------------------------------------------------------------------------
# models: loaded once
# ---------------------------------------------------------------------------------------------------------------------
_models = {}


def _model(name):
    if name in _models:
        return _models[name]
    m = SHAPES[name]
    seed = {"tiny": 1001, "draft": 1002, "target": 1005}[name]
    weights = W.make_weights(m, seed, DEVICE)
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    # the means of the cached values, and the direction in which each topic moves the hidden state
    topics = torch.randn(N_TOPICS, m.n_layers, m.n_kv_heads, m.head_dim, generator=g, device=DEVICE) * 0.7
    along = torch.zeros(N_TOPICS, m.d_model, device=DEVICE)
    for l in range(m.n_layers):
        heads = topics[:, l].repeat_interleave(m.group, dim=1).reshape(N_TOPICS, -1)
        along += heads @ weights.wo[l].float().t()
    along /= along.norm(dim=1, keepdim=True)
    ids = np.random.default_rng(1).choice(SHAPES["tiny"].vocab, N_TOPICS + 2, replace=False)    # the same for all models
    leans = torch.tensor(LEANS, device=DEVICE).repeat_interleave(N_TOPICS // 4) / ALONG[name]
    verdict = torch.linalg.lstsq(along, leans[:, None]).solution[:, 0]
    said = torch.as_tensor(ids[2:], device=DEVICE)
    weights.lm_head[said] = (weights.lm_head[said].float() + along * (20.0 / ALONG[name])).to(weights.lm_head.dtype)
    weights.lm_head[int(ids[0])] = (verdict / 2).to(weights.lm_head.dtype)
    weights.lm_head[int(ids[1])] = (-verdict / 2).to(weights.lm_head.dtype)
    _models[name] = SimpleNamespace(cfg=m, verifier=Verifier(m, weights), topics=topics, verdict_ids=[int(i) for i in ids[:2]])
    return _models[name]


def _cache(name, topic_of_block, g):
    m, topics = SHAPES[name], _model(name).topics
    dt = W.torch_dtype(m.dtype)
    shape = (m.n_layers, topic_of_block.numel(), m.n_kv_heads, BLOCK, m.head_dim)
    k, v = torch.empty(shape, dtype=dt, device=DEVICE), torch.empty(shape, dtype=dt, device=DEVICE)
    for l in range(m.n_layers):
        k[l].normal_(0.0, KV_STD, generator=g)
        v[l].normal_(0.0, KV_STD, generator=g)
        v[l].add_(topics[:, l].to(dt)[topic_of_block][:, :, None, :])
    return SimpleNamespace(k_pages=k, v_pages=v, block_size=BLOCK)


# ---------------------------------------------------------------------------------------------------------------------
# one case
# ---------------------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    L, S = _lengths(case)
    kinds = np.asarray(_kinds(case))
    B, group, do = case["B"], case.get("group", 1), case["do"]
    grow = [case["steps"]] * B if do == "generate" else S if do == "append" else [0] * B
    need = [-(-(l + e) // BLOCK) for l, e in zip(L, grow)]
    owners = range(0, B, group)                                     # candidates name the pages of their group's first trace
    n_blocks = sum(need[b] for b in owners)
    perm = rng.permutation(n_blocks)
    topic = kinds * (N_TOPICS // 4) + rng.integers(0, N_TOPICS // 4, B)
    table = np.zeros((B, max(need)), dtype=np.int32)
    topic_of_block = np.zeros(n_blocks, dtype=np.int64)
    at = 0
    for b in owners:
        mine = perm[at:at + need[b]]
        table[b:b + group, :need[b]] = mine
        topic_of_block[mine] = topic[b]
        at += need[b]
    topic_of_block = torch.from_numpy(topic_of_block).to(DEVICE)
    cu = np.concatenate([[0], np.cumsum(S)]).astype(np.int32)
    lens = np.asarray(L, dtype=np.int32)
    vocab = SHAPES[case["model"]].vocab
    ids = rng.integers(0, vocab, cu[-1]).astype(np.int32)
    batch = SimpleNamespace(suffix_ids=torch.from_numpy(ids).to(DEVICE), cu_suffix=torch.from_numpy(cu).to(DEVICE),
                            prefix_lens=torch.from_numpy(lens).to(DEVICE), block_table=torch.from_numpy(table).to(DEVICE),
                            n_blocks=n_blocks, max_blocks_per_seq=max(need), block_size=BLOCK, h_cu_suffix=cu, h_prefix_lens=lens)
    model = _model(case["model"])
    s = SimpleNamespace(case=case, model=model, batch=batch, kv=_cache(case["model"], topic_of_block, g),
                        taus=[0.8, 0.9, 0.95] if case.get("n_tau") == 3 else [0.9])
    if do == "shared":
        s.groups = list(range(0, B + 1, group))
    elif do == "append":
        s.n_append = np.asarray(S, dtype=np.int32)
    elif do == "cascade":
        # the large model has its own cache of the same contexts; it is sure wherever it is asked
        target = _model("target")
        sure = torch.from_numpy(rng.integers(0, N_TOPICS // 2, N_TOPICS)).to(DEVICE)
        s.target_kv = _cache("target", sure[topic_of_block], g)
        both = (model.verifier, target.verifier)
        s.cascade, s.requests = Cascade(*both), _requests(case)
    return s


def run(s):
    ver, ids, do = s.model.verifier, s.model.verdict_ids, s.case["do"]
    if do == "generate":
        b = s.batch
        out = ver.generate_greedy(s.kv, b.block_table, b.n_blocks, b.max_blocks_per_seq, b.suffix_ids, b.h_prefix_lens,
                                  s.case["steps"])
        return list(out) + [s.kv.k_pages, s.kv.v_pages]
    if do == "cascade":
        out, n_target = s.cascade.run(s.kv, s.target_kv, s.batch, s.requests, ids, GAMMA)
        return [out, n_target]
    if do == "shared":
        return list(ver.verify_shared(s.kv, s.batch, s.groups, ids, s.taus))
    if do == "append":
        return list(ver.verify_append(s.kv, s.batch, s.n_append, ids, s.taus)) + [s.kv.k_pages, s.kv.v_pages]
    return list(ver.verify(s.kv, s.batch, ids, s.taus))
