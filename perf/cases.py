"""What the speed of this library is measured on.

The cases are the work of one RL step as its Data Coordinator issues it through the binding: the reshard of a GRPO
rollout batch (balance, advantage, plan, gather), its form without a rollout-layout copy of the advantages, the way back
(scatter) and PPO's advantage stage.  Shapes are those of ``workloads.py`` and of the tests, and what lies around them:
a handful of prompts, short answers (a granule of the gather holds many sequences), more data-parallel ranks than a
wavefront has lanes, more sequences than one workgroup's LDS holds.

Inputs are made on the GPU from the seed (lengths and rewards on the host: they are small).  A state holds what a
training program holds between two steps: the rollout buffers, the arenas and the workspaces, all allocated once.
"""
from __future__ import annotations

import heapq
import math

import numpy as np
import torch

from paper_2507_13833_amd import binding as B

DEV = "cuda:0"

# per-token payloads that move beside the advantages: (name, type)
PAYLOADS = {
    "grpo32": (("token_id", "i32"), ("old_logprob", "f32"), ("mask", "u8")),
    "grpo16": (("token_id", "i32"), ("old_logprob", "bf16"), ("ref_logprob", "bf16"), ("mask", "u8")),
    "critic": (("token_id", "i32"), ("old_logprob", "f32"), ("ref_logprob", "f32"), ("value", "f32"), ("mask", "u8")),
    "critic_entropy": (("token_id", "i32"), ("old_logprob", "f32"), ("ref_logprob", "f32"), ("value", "f32"),
                       ("entropy", "bf16"), ("mask", "u8")),
    # what a training-layout stage gives back
    "logprob": (("new_logprob", "f32"),),
    "logprob_entropy": (("new_logprob", "bf16"), ("entropy", "bf16")),
    "logprob_value": (("new_logprob", "f32"), ("value", "f32"), ("entropy", "bf16")),
}
BYTES = {"i32": 4, "f32": 4, "bf16": 2, "u8": 1}
TYPES = {"i32": torch.int32, "f32": torch.float32, "bf16": torch.bfloat16, "u8": torch.uint8}


def _case(name, kind, prompts, group, shards, budget, **more):
    c = {"name": name, "kind": kind, "prompts": prompts, "group": group, "shards": shards, "budget": budget,
         "rollout_shards": 1, "align": 1, "prompt_lo": 64, "prompt_hi": 256, "answer": "lognormal", "mu": 5.5, "sigma": 0.8,
         "answer_lo": 16, "answer_hi": 1024, "turns": 1, "payload": "critic", "kl": 0.0}
    c.update(more)
    return c


def listed():
    large = dict(prompt_lo=256, prompt_hi=2048, mu=7.0, sigma=1.1, answer_lo=64, answer_hi=8192)
    tail = dict(prompt_lo=512, prompt_hi=4096, answer="pareto", answer_hi=32768, turns=4)
    return [
        # the last, partial batch of an epoch or a trial run: 64 sequences
        _case("step-tiny", "step", 16, 4, 2, 2048, prompt_lo=32, prompt_hi=128, mu=5.0, answer_hi=512, payload="grpo32"),
        # a small run on four ranks (workload 1)
        _case("step-small", "step", 64, 8, 4, 8192, payload="grpo32"),
        # eight ranks, log-probabilities kept in bf16 (workload 2)
        _case("step-mid-bf16", "step", 256, 8, 8, 16384, prompt_lo=128, prompt_hi=1024, mu=6.5, sigma=1.0, answer_lo=32,
              answer_hi=4096, payload="grpo16"),
        # many short question / answer pairs, shard starts on multiples of 8 tokens
        _case("step-short-answers", "step", 1920, 8, 24, 16384, align=8, prompt_lo=20, prompt_hi=150, mu=4.7, sigma=0.6,
              answer_lo=8, answer_hi=512),
        # 8192 sequences for 32 ranks, advantages made by the gather (workload 3)
        _case("lean-large", "lean", 512, 16, 32, 32768, **large),
        # eight rollout engines hand over to 16 ranks (workload 4)
        _case("step-layout-change", "step", 512, 16, 16, 65536, rollout_shards=8, **large),
        # long-tailed multi-turn answers on 64 ranks, every field a critic needs (workload 5)
        _case("step-long-tail", "step", 1024, 16, 64, 131072, payload="critic_entropy", **tail),
        # a large job: more ranks than a wavefront has lanes
        _case("step-128-ranks", "step", 512, 16, 128, 32768, align=16, **large),
        # a large batch of short answers: more sequences than one workgroup's LDS holds
        _case("step-65536-sequences", "step", 8192, 8, 64, 32768),
        # log-probabilities and values of the training layout go back to the eight rollout shards
        _case("back-layout-change", "back", 512, 16, 16, 65536, rollout_shards=8, payload="logprob_value", **large),
        # PPO's advantage stage, reward model score only
        _case("gae-mid", "gae", 2048, 1, 8, 16384, prompt_lo=128, prompt_hi=1024, mu=6.5, sigma=1.0, answer_lo=32,
              answer_hi=4096),
        # the same with the KL penalty on long-tailed multi-turn answers
        _case("gae-kl-long-tail", "gae", 1024, 16, 64, 131072, kl=0.05, **tail),
    ]


def draw(rng):
    """One more case of the same ranges; about 24 M tokens and 40 000 sequences at most, 2048 on a rank."""
    kind = rng.choice(("step", "step", "step", "step", "lean", "back", "gae", "gae"))
    group = rng.choice((4, 5, 8, 8, 12, 16)) if kind != "gae" else rng.choice((1, 1, 4, 8))
    seqs = int(math.exp(rng.uniform(math.log(48), math.log(40000))))
    shards = rng.choice([p for p in (1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 40, 48, 64, 96, 128, 192, 256) if 2048 * p >= seqs])
    mean = math.exp(rng.uniform(math.log(120.0), math.log(4000.0)))       # tokens of a sequence, about
    mean = min(mean, 24e6 / seqs)
    unit = shards // math.gcd(shards, group)                             # Algorithm 1: equal shards
    prompts = max(1, round(seqs / group / unit)) * unit
    share = rng.uniform(0.15, 0.6)                                       # of the prompt
    prompt_hi = max(8, int(mean * share * 1.8))
    sigma = rng.uniform(0.3, 1.1)
    answer_hi = max(64, int(mean * rng.uniform(4.0, 10.0)))
    payload = rng.choice(("grpo32", "grpo16", "critic", "critic_entropy")) if kind in ("step", "lean") else \
        rng.choice(("logprob", "logprob_entropy", "logprob_value")) if kind == "back" else "critic"
    c = _case("", kind, prompts, group, shards, 1 << max(11, (prompt_hi + answer_hi).bit_length() + rng.randrange(3)),
              rollout_shards=rng.choice((1, 1, 2, 4, 8)), align=rng.choice((1, 1, 1, 8, 16, 64)),
              prompt_lo=max(4, prompt_hi // 8), prompt_hi=prompt_hi, answer=rng.choice(("lognormal", "lognormal", "pareto")),
              mu=round(math.log(max(8.0, mean * (1 - share))) - sigma * sigma / 2, 3), sigma=round(sigma, 3),
              answer_lo=8, answer_hi=answer_hi, turns=rng.choice((1, 1, 4)), payload=payload,
              kl=0.05 if kind == "gae" and rng.random() < 0.5 else 0.0)
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------------- inputs

def _host(case, seed):
    """Lengths, rewards and offsets of a batch, on the host.  A case has its own prompts and answers (so its buffers have
    the same sizes for every seed); the seed says which answers meet which prompt, and in which order they come."""
    r = np.random.default_rng(7)
    group, engines = case["group"], case["rollout_shards"]
    n = case["prompts"] * group
    prompt = r.integers(case["prompt_lo"], case["prompt_hi"] + 1, case["prompts"])
    if case["answer"] == "pareto":
        answer = np.floor(max(8.0, math.exp(case["mu"]) / 3.8) * (1.0 - r.random(n)) ** (-1.0 / 1.3))
    else:
        answer = np.rint(r.lognormal(case["mu"], case["sigma"], n))
    answer = np.clip(answer, case["answer_lo"], case["answer_hi"]).astype(np.int64)
    # a prompt's answers come from one rollout engine
    cut = [case["prompts"] * s // engines * group for s in range(engines + 1)]
    r = np.random.default_rng(seed)
    for a, b in zip(cut, cut[1:]):
        r.shuffle(prompt[a // group:b // group])
        r.shuffle(answer[a:b])
    prompt = np.repeat(prompt, group)
    length = (prompt + answer).astype(np.int32)
    # a verifier's 0 / 1 rewards, every third group one of graded rewards, some groups all alike
    reward = (r.random(n) < 0.35).astype(np.float32).reshape(-1, group)
    reward[::3] = np.round(r.random(reward[::3].shape), 2).astype(np.float32)
    reward[4::8] = reward[4::8, :1]
    off = np.zeros(n, np.int64)
    tokens = []
    for a, b in zip(cut, cut[1:]):
        run = np.cumsum(length[a:b], dtype=np.int64)
        off[a + 1:b] = run[:-1] if b > a else 0
        tokens.append(int(run[-1]) if b > a else 0)
    return {"prompt": prompt, "length": length, "reward": reward.reshape(-1), "cut": cut, "off": off, "tokens": tokens}


def _values(kind, name, n, gen):
    if kind == "i32":
        return torch.randint(0, 152064, (n,), generator=gen, device=DEV, dtype=torch.int32)
    x = torch.randn(n, generator=gen, device=DEV)
    if name != "value":
        x = x.abs_() if name == "entropy" else x.abs_().neg_()
    return x.to(TYPES[kind])


def _mask(case, h, r):
    """Loss mask of the whole batch in index order: 0 on the prompt, 1 on the answer; answers of several turns are cut
    into up to four runs, of which every second one (a tool's output) bears no loss."""
    n = len(h["length"])
    length = torch.from_numpy(h["length"]).to(DEV).long()
    start = torch.cumsum(length, 0) - length
    at = torch.arange(int(length.sum()), device=DEV) - torch.repeat_interleave(start, length)
    at = at - torch.repeat_interleave(torch.from_numpy(h["prompt"]).to(DEV), length)
    m = at >= 0
    if case["turns"] > 1:
        runs = r.integers(1, case["turns"] + 1, n)
        odd = torch.zeros_like(m)
        for k in range(case["turns"] - 1):
            place = np.where(k + 1 < runs, (h["length"] - h["prompt"]) * r.random(n), 1 << 30).astype(np.int64)
            odd ^= at >= torch.repeat_interleave(torch.from_numpy(place).to(DEV), length)
        m &= ~odd
    return m.to(torch.uint8)


def _split(h, x):
    """Index order -> one buffer per rollout shard (each an allocation of its own)."""
    return [p.clone() for p in torch.split(x, h["tokens"])]


class _State:
    pass


def prepare(case, seed):
    h = _host(case, seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    r = np.random.default_rng([seed, 1])
    s = _State()
    n, p = len(h["length"]), case["shards"]
    total = sum(h["tokens"])
    s.case, s.n, s.groups = case, n, case["prompts"]
    s.capacity = total + p * (case["align"] - 1)
    s.prm = B.make_params(n, p, case["budget"], align_tokens=case["align"])
    s.seq_len = torch.from_numpy(h["length"]).to(DEV)
    s.reward = torch.from_numpy(h["reward"]).to(DEV)
    s.group_off = (torch.arange(case["prompts"] + 1, device=DEV) * case["group"]).to(torch.int32)
    s.src = B.Source(h["cut"], h["tokens"], torch.from_numpy(h["off"]).to(DEV))
    s.status = torch.zeros(1, dtype=torch.int32, device=DEV)
    payload = PAYLOADS[case["payload"]]

    if case["kind"] == "gae":
        s.value = _split(h, _values("f32", "value", total, gen))
        s.mask = _split(h, _mask(case, h, r))
        s.logp = _split(h, _values("f32", "old_logprob", total, gen)) if case["kl"] else None
        s.ref = _split(h, _values("f32", "ref_logprob", total, gen)) if case["kl"] else None
        s.adv = [torch.zeros(t, device=DEV) for t in h["tokens"]]
        s.ret = [torch.zeros(t, device=DEV) for t in h["tokens"]]
        return s

    def ints(k, dtype=torch.int32):
        return torch.zeros(k, dtype=dtype, device=DEV)

    s.perm, s.seq_off, s.shard_of, s.load = ints(n), ints(p + 1), ints(n), ints(p, torch.int64)
    s.tok_off, s.shard_tok, s.shard_mb = ints(n + 1, torch.int64), ints(p + 1, torch.int64), ints(p + 1)
    s.mb_seq, s.cu, s.n_mb = ints(n + 1), ints(2 * n), ints(1)
    s.large = n > B.DC_MAX_SEQ
    s.bal_bytes = B.dc_balance_workspace_bytes(s.prm)
    s.bal_ws = ints(s.bal_bytes, torch.uint8) if s.bal_bytes else None
    s.ws_bytes = B.dc_workspace_bytes(s.prm, s.capacity)
    s.ws = ints(s.ws_bytes, torch.uint8)

    if case["kind"] == "back":
        _balance(s)
        B.dc_plan(s.prm, s.src, s.seq_len, s.perm, s.seq_off, s.capacity, s.tok_off, s.shard_tok, s.shard_mb, s.mb_seq,
                  s.cu, s.n_mb, s.ws, s.ws_bytes, s.status)
        s.arena = {f: _values(k, f, s.capacity, gen) for f, k in payload}
        s.out = {f: [torch.zeros(t, dtype=TYPES[k], device=DEV) for t in h["tokens"]] for f, k in payload}
        s.fields = B.Fields([(s.out[f], s.arena[f], BYTES[k]) for f, k in payload])
        s.back_bytes = B.dc_scatter_workspace_bytes(s.prm, s.src)
        s.back_ws = ints(s.back_bytes, torch.uint8)
        return s

    s.rollout = {f: _split(h, _mask(case, h, r) if f == "mask" else _values(k, f, total, gen)) for f, k in payload}
    s.adv_seq = torch.zeros(n, device=DEV)
    s.dst = {f: torch.zeros(s.capacity, dtype=TYPES[k], device=DEV) for f, k in payload}
    s.dst["adv"] = torch.zeros(s.capacity, device=DEV)
    s.adv_tok = [torch.zeros(t, device=DEV) for t in h["tokens"]] if case["kind"] == "step" else None
    moved = [(s.rollout[f], s.dst[f], BYTES[k]) for f, k in payload]
    s.mask_at = [f for f, _ in payload].index("mask")
    s.fields = B.Fields(moved + ([(s.adv_tok, s.dst["adv"], 4)] if case["kind"] == "step" else []))
    return s


# ---------------------------------------------------------------------------------------------- the pass

def _balance(s):
    if s.large:
        B.dc_balance_ws(s.prm, s.seq_len, s.perm, s.seq_off, s.shard_of, s.load, s.bal_ws, s.bal_bytes, s.status)
    else:
        B.dc_balance(s.prm, s.seq_len, s.perm, s.seq_off, s.shard_of, s.load, s.status)


def run(s):
    kind = s.case["kind"]
    if kind == "gae":
        B.dc_gae(s.prm, s.src, s.seq_len, s.reward, s.value, s.mask, s.logp, s.ref, 1.0, 0.95, s.case["kl"], s.adv, s.ret,
                 s.status)
        return {"adv": s.adv, "ret": s.ret, "status": s.status}
    if kind == "back":
        B.dc_scatter(s.prm, s.src, s.seq_len, s.perm, s.fields, s.capacity, s.tok_off, s.back_ws, s.back_bytes, s.status)
        return {"out": s.out, "status": s.status}

    mask = s.rollout["mask"] if kind == "step" else None
    if s.large:                                     # the calls in one launch end at DC_MAX_SEQ sequences
        B.dc_group_advantage(s.prm, s.src, s.seq_len, s.reward, s.group_off, s.groups, mask, s.adv_seq, s.adv_tok, s.status)
        _balance(s)
        B.dc_plan(s.prm, s.src, s.seq_len, s.perm, s.seq_off, s.capacity, s.tok_off, s.shard_tok, s.shard_mb, s.mb_seq,
                  s.cu, s.n_mb, s.ws, s.ws_bytes, s.status)
    else:
        B.dc_balance_plan_group_advantage(s.prm, s.src, s.seq_len, s.perm, s.seq_off, s.shard_of, s.load, s.reward,
                                          s.group_off, s.groups, mask, s.adv_seq, s.adv_tok, s.capacity, s.tok_off,
                                          s.shard_tok, s.shard_mb, s.mb_seq, s.cu, s.n_mb, s.ws, s.ws_bytes, s.status)
    if kind == "step":
        B.dc_gather(s.prm, s.src, s.fields, s.capacity, s.tok_off, s.ws, s.ws_bytes, s.status)
    else:
        B.dc_gather_advantage(s.prm, s.src, s.fields, s.mask_at, s.perm, s.adv_seq, s.dst["adv"], s.capacity, s.tok_off,
                              s.ws, s.ws_bytes, s.status)
    return {"perm": s.perm, "seq_off": s.seq_off, "shard_of": s.shard_of, "load": s.load, "adv_seq": s.adv_seq,
            "adv_tok": s.adv_tok, "tok_off": s.tok_off, "shard_tok": s.shard_tok, "shard_mb": s.shard_mb,
            "mb_seq": s.mb_seq, "cu": s.cu, "n_mb": s.n_mb, "dst": s.dst, "status": s.status}


# ---------------------------------------------------------------------------------------------- what it has to do

def work(case):
    h = _host(case, 0)                              # the sizes are the case's own, whatever the seed
    n, t = len(h["length"]), sum(h["tokens"])
    payload = sum(BYTES[k] for _, k in PAYLOADS[case["payload"]])
    if case["kind"] == "gae":                       # value, mask and the two log-probabilities in, two arrays out
        return {"bytes": t * (13 + (8 if case["kl"] else 0)) + 16 * n, "flops": 0}
    if case["kind"] == "back":
        return {"bytes": 2 * payload * t + 24 * n, "flops": 0}
    # every field read and written once, the advantages written; the rollout-layout copy of them is an output of its own
    # (once written, it need not be read again)
    per_token = 2 * payload + 4 + (4 if case["kind"] == "step" else 0)
    return {"bytes": per_token * t + 60 * n, "flops": 0}


def tolerance(case):
    if case["kind"] == "back":
        return "exact"
    # evaluated in 64 bits and rounded once: another order of the sums turns the rounding of single values
    return {"rel": 1e-7, "max": 5e-7}


# ---------------------------------------------------------------------------------------------- the same in 64 bits

def _exact_partition(length, shards):
    """Algorithm 1 as printed: the members of every shard in insertion order."""
    order = np.argsort(-length.astype(np.int64), kind="stable")
    room = len(length) // shards
    heap, parts = [(0, k) for k in range(shards)], [[] for _ in range(shards)]
    for i in order.tolist():
        load, k = heap[0]
        parts[k].append(i)
        if len(parts[k]) < room:
            heapq.heapreplace(heap, (load + int(length[i]), k))
        else:
            heapq.heappop(heap)
    return parts


def _exact_advantage(h, group):
    r = h["reward"].astype(np.float64).reshape(-1, group)
    if group == 1:
        return np.zeros(r.size)
    a = (r - r.mean(1, keepdims=True)) / (r.std(1, ddof=1, keepdims=True) + 1e-6)
    a[(h["reward"].reshape(-1, group) == h["reward"].reshape(-1, group)[:, :1]).all(1)] = 0.0
    return a.reshape(-1)


def exact(case, seed):
    h = _host(case, seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    r = np.random.default_rng([seed, 1])
    n, total = len(h["length"]), sum(h["tokens"])
    length = torch.from_numpy(h["length"]).to(DEV).long()
    first = torch.cumsum(length, 0) - length                              # a sequence's first token, index order
    payload = PAYLOADS[case["payload"]]

    if case["kind"] == "gae":
        value = _values("f32", "value", total, gen).double()
        mask = _mask(case, h, r).bool()
        step = torch.zeros_like(value)
        if case["kl"]:
            logp = _values("f32", "old_logprob", total, gen).double()
            step = -case["kl"] * (logp - _values("f32", "ref_logprob", total, gen).double())
        seq = torch.repeat_interleave(torch.arange(n, device=DEV), length)[mask]   # the tokens that bear loss
        v, d = value[mask], step[mask]
        last = torch.ones_like(seq, dtype=torch.bool)
        last[:-1] = seq[1:] != seq[:-1]
        d[last] += torch.from_numpy(h["reward"]).to(DEV).double()[seq[last]]
        nxt = torch.zeros_like(v)
        nxt[:-1] = v[1:]
        nxt[last] = 0.0
        a, w = d + nxt - v, 0.95 * (~last).double()                       # A_k = a_k + w_k A_{k+1}, by doubling
        hop = 1
        while hop < int(length.max()):
            a[:-hop] = a[:-hop] + w[:-hop] * a[hop:].clone()
            w[:-hop] = w[:-hop] * w[hop:].clone()
            w[-hop:] = 0.0
            hop *= 2
        adv, ret = torch.zeros_like(value), torch.zeros_like(value)
        adv[mask], ret[mask] = a, a + v
        return {"adv": _split(h, adv), "ret": _split(h, ret), "status": None}

    parts = _exact_partition(h["length"], case["shards"])
    perm = np.concatenate([np.array(q, np.int64) for q in parts])
    loads = np.array([int(h["length"][q].sum()) for q in parts], np.int64)
    step = (loads + case["align"] - 1) // case["align"] * case["align"]
    base = np.repeat(np.cumsum(step) - step, [len(q) for q in parts])
    inside = np.concatenate([np.cumsum(h["length"][q], dtype=np.int64) - h["length"][q] for q in parts])
    place = np.zeros(n, np.int64)
    place[perm] = base + inside                                           # a sequence's first token, training layout
    capacity = total + case["shards"] * (case["align"] - 1)
    to = torch.arange(total, device=DEV) + torch.repeat_interleave(torch.from_numpy(place).to(DEV) - first, length)

    if case["kind"] == "back":
        arena = {f: _values(k, f, capacity, gen) for f, k in payload}
        return {"out": {f: _split(h, arena[f][to]) for f, _ in payload}, "status": None}

    adv = torch.from_numpy(_exact_advantage(h, case["group"])).to(DEV)
    rollout = {f: _mask(case, h, r) if f == "mask" else _values(k, f, total, gen) for f, k in payload}
    rollout["adv"] = torch.repeat_interleave(adv, length) * rollout["mask"]
    dst = {}
    for f, x in rollout.items():
        dst[f] = torch.zeros(capacity, dtype=x.dtype, device=DEV)
        dst[f][to] = x
    return {"adv_seq": adv, "adv_tok": _split(h, rollout["adv"]) if case["kind"] == "step" else None, "dst": dst}
