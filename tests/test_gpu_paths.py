"""The branches that a call's sizes choose between, each at the sizes where it can go wrong, against the CPU oracle
(bit-exact but for the float32 advantages: float64 arithmetic on both sides, see test_gpu_parity)."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import _check_balance_ws, _custom, _gpu, _with_ppo_fields, check_gae, check_gather_advantage, check_scatter, check_step, compare_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("length", [341, 256, 205, 204, 22, 21, 17, 16, 15, 4, 3])
def test_slots_of_a_granule(length):
    """Equal lengths round the counts at which a 1024-token granule changes its path: 4 slots (its record holds them), 5 (a
    wave stages them), 47 and 48, 63 and 64 (one pass or two over the staged slots), more slots than 16-byte chunks."""
    n = max(64, 9000 // length) // 32 * 32
    lens = np.full(n, length, np.int32)
    lens[::7] += np.arange(len(lens[::7])) % 3
    for align in (1, 5):
        w = _custom(lens, 4, 4, 4096, n_src=2, seed=length)
        check_step(w, align=align, label=f"length {length}", two_calls=True)
        check_gather_advantage(w, align=align, label=f"length {length}")
    check_scatter(_custom(lens, 4, 4, 4096, n_src=2, seed=length), label=f"length {length}")


def _lengths(kind, n, rng):
    if kind == "geometric":
        return np.minimum(rng.geometric(0.004, n), 6000)
    if kind == "tail":                                   # a few workers far above the others: rounds that few workers join
        x = np.minimum(64 * (1.0 - rng.random(n)) ** (-1 / 1.1), 30000).astype(np.int64) + rng.integers(1, 60, n)
        x[: max(1, n // 50)] = rng.integers(1, 4, max(1, n // 50))
        return x
    if kind == "equal":
        return np.full(n, 77)
    assert kind == "long"                                # one sequence of 2^16 tokens or more: the general rounds
    x = rng.integers(1, 300, n)
    x[n // 2] = 70000
    return x


@pytest.mark.parametrize("kind", ["geometric", "tail", "equal", "long"])
@pytest.mark.parametrize("shards", [33, 48, 63, 65, 96, 127, 128, 129, 200, 255, 256, 257])
def test_one_wave_with_up_to_256_workers(shards, kind):
    """33 to 63 workers on a sort of 64 lanes, above 64 two and four keys to a lane, with and without lanes that keep no worker, plan in
    the same launch up to 256."""
    rng = np.random.default_rng(shards)
    for per in (1, 2, 21) if kind != "tail" else (3, 16384 // shards):
        lens = _lengths(kind, shards * per, rng).astype(np.int32)
        if per > 100:
            lens = np.minimum(lens, 2000)
        w = _custom(lens, 1, shards, 1 << 17, fields=())
        check_step(w, align=7, label=f"{shards} shards of {per}, {kind}", two_calls=True)


@pytest.mark.parametrize("shards", [1, 3, 8, 12, 24, 40, 63, 65, 96, 128, 200, 256])
def test_portions_of_a_long_list(shards):
    """More sequences than the LDS holds on every width of the packed rounds: rows fill up and are emptied in between."""
    rng = np.random.default_rng(shards)
    for kind, n in (("tail", 16385), ("geometric", 40000)):
        per = -(-n // shards)
        _check_balance_ws(_lengths(kind, per * shards, rng).astype(np.int32), shards, label=f"{shards} shards of {per}, {kind}")


@pytest.mark.parametrize("n,shards,budget,align,cap", [
    (16385, 1, 64, 1, 0),               # one slot more than the LDS holds, a shard of one wave's whole walk
    (16640, 65, 8, 3, 0),               # most micro-batches hold one or two slots
    (33000, 1, 1 << 20, 1, 0),          # a shard that is probed in global memory; few micro-batches
    (32768, 1, 300, 64, 0),             # the first that is
    (32767, 1, 300, 64, 0),             # the last that is staged
    (20000, 1000, 4096, 16, 0),
    (20480, 16, 40, 1, 20480),          # partitions of unequal size, tiles that end with the last slot
])
def test_plan_of_many_slots(n, shards, budget, align, cap):
    """dc_plan above DC_MAX_SEQ sequences: tiles, staged and unstaged shards, budgets from one slot to a whole shard."""
    lens = np.random.default_rng(n).integers(1, 40, n).astype(np.int32)
    w = _custom(lens, 1, shards, max(budget, 40), n_src=1, fields=())
    check_step(w, align=align, cap=cap, label=f"{n} slots on {shards} shards, budget {budget}")


@pytest.mark.parametrize("n,shards,budget", [(64, 1, 41), (1024, 2, 64), (1025, 2, 64), (2040, 8, 41), (2048, 1, 4096),
                                             (8192, 1, 100), (8193, 3, 100), (300, 150, 41)])
def test_plan_of_few_slots_and_long_chains(n, shards, budget):
    """Dozens of micro-batches per shard: every slot's own end, then the chain; 8192 slots are the most that takes."""
    lens = np.random.default_rng(n).integers(1, 41, n).astype(np.int32)
    for align in (1, 6):
        check_step(_custom(lens, 1, shards, budget, fields=()), align=align, two_calls=n % shards == 0,
                   cap=0 if n % shards == 0 else n, label=f"{n} slots on {shards} shards, budget {budget}")


@pytest.mark.parametrize("kind", ["geometric", "equal", "tail"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 500, 1023, 1024, 1025, 1990, 2047, 2048, 2049])
def test_sort_of_few_sequences(n, kind):
    """Up to 2048 sequences: one wave, several, all sixteen, one and two words to a lane, and the first size of the bins."""
    lens = _lengths(kind, n, np.random.default_rng(n)).astype(np.int32)
    if kind == "tail":
        lens = np.sort(lens)[:: 1 if n % 2 else -1].copy()       # ascending and descending input
    check_step(_custom(lens, 1, 1, 1 << 17, fields=()), label=f"{n} sequences, {kind}", two_calls=True)


@pytest.mark.parametrize("entries", [17, 1023, 1024, 1025, 2047, 2048, 2049])
@pytest.mark.parametrize("align", [1, 48])
@pytest.mark.parametrize("n,shards", [(128, 4), (256, 4), (512, 4)])
def test_granule_tables_of_a_small_batch(entries, align, n, shards):
    """Up to 256 sequences on shards of 64 and 2048 table entries (the arena's granules and 16 more) the balance workgroup makes
    them itself, a lane one or two of them, beyond either the launch that plans by shards does; the arena ends with the last
    granule and one token into it."""
    for tokens in ((entries - 16) * 1024, (entries - 17) * 1024 + 1):
        if tokens < n + shards * (align - 1):
            continue
        room = tokens - shards * (align - 1)
        lens = np.random.default_rng(tokens).integers(max(1, room // n // 2), max(2, room // n), n)
        lens[0] += room - int(lens.sum())
        w = _custom(lens.astype(np.int32), 4, shards, 1 << 22, n_src=2, seed=entries, fields=("i32", "bf16"))
        assert w.total_tokens + shards * (align - 1) == tokens and -(-tokens // 1024) + 16 == entries and lens.min() > 0
        check_step(w, align=align, label=f"{tokens} tokens of capacity", two_calls=True)
        check_gather_advantage(w, align=align, label=f"{tokens} tokens")


@pytest.mark.parametrize("kl", [0.0, 0.05])
@pytest.mark.parametrize("n,mean", [(1024, 300), (1025, 40), (1025, 1100), (2048, 1030), (2049, 30), (2049, 380), (2049, 400), (2500, 1270),
                                    (2500, 1300), (1100, 2100)])
def test_gae_waves_and_tokens_per_lane(n, mean, kl):
    """Each way of sharing a sequence among waves and lanes, on both sides of the lines between them, with sequences that
    start and end anywhere in a lane's tokens, single tokens, and a few of many iterations."""
    rng = np.random.default_rng(n + mean)
    lens = rng.integers(1, 2 * mean - 1, n)
    lens[:: n // 3] = 4 * mean + rng.integers(0, 9)
    lens[1:: n // 3] = 1
    w = _with_ppo_fields(_custom(lens.astype(np.int32), 1, 1, 1 << 20, fields=()), seed=n)
    check_gae(w, 0.99, 0.95, kl, label=f"{n} sequences of {mean}")


@pytest.mark.parametrize("n,group,n_src", [(16384, 8, 1), (16385, 1, 1), (16386, 2, 2), (20000, 5, 4), (16384, 64, 8), (16400, 82, 1)])
@pytest.mark.parametrize("kind", ["geometric", "ones", "mixed"])
def test_advantages_of_many_short_sequences(n, group, n_src, kind):
    """Eight sequences to a wave: the last wave's remainder, sequences of one token and of more than its four steps, groups
    larger than a wave's share, rollout shards that end inside a wave."""
    rng = np.random.default_rng(n + group)
    lens = np.minimum(rng.geometric(0.01, n), 900) if kind == "geometric" else np.ones(n, np.int64)
    if kind == "mixed":
        lens = rng.integers(1, 12, n)
        lens[:: n // 40] = rng.integers(1000, 5000, len(lens[:: n // 40]))
    w = _custom(lens.astype(np.int32), group, 1, 1 << 17, n_src=n_src, seed=n, fields=())
    check_step(w, label=f"{n} sequences, groups of {group}, {kind}")


def test_advantages_of_many_short_sequences_in_uneven_groups():
    rng = np.random.default_rng(3)
    n = 16384
    w = _custom(np.minimum(rng.geometric(0.02, n), 500).astype(np.int32), 1, 1, 1 << 17, fields=())
    cuts = np.unique(np.concatenate([[0, n], rng.integers(0, n, 700)])).astype(np.int32)
    w.group_off = cuts
    w.reward[cuts[5]:cuts[6]] = 0.25                     # rewards all alike: exactly +0
    check_step(w, label="uneven groups")


def test_plan_of_many_slots_without_permutation_and_shard_table():
    """dc_plan above DC_MAX_SEQ sequences that keeps the rollout shards: no notes to check, the shard
    table made on the device."""
    torch, binding, runner = _gpu()
    lens = np.random.default_rng(5).integers(1, 60, 20000).astype(np.int32)
    w = _custom(lens, 1, 4, 512, n_src=4, fields=())
    d = runner.DeviceBatch(w, poison=True)
    binding.dc_plan(d.prm, d.source, d.seq_len, None, None, d.capacity, d.dst_tok_off, d.shard_tok_off, d.shard_mb_off,
                    d.mb_seq_off, d.cu_seqlens, d.n_mb, d.ws, d.ws_bytes, d.status)
    torch.cuda.synchronize()
    assert d.read_status() == 0
    pl = oracle.plan(w.seq_len, np.arange(w.n_seq, dtype=np.int32), w.src_shard_seq_off, w.token_budget)
    M = int(d.n_mb.item())
    assert M == pl.n_mb
    for got, want in ((d.dst_tok_off, pl.dst_tok_off), (d.shard_tok_off, pl.shard_tok_off), (d.shard_mb_off, pl.shard_mb_off),
                      (d.mb_seq_off[:M + 1], pl.mb_seq_off), (d.cu_seqlens[:w.n_seq + M], pl.cu_seqlens)):
        assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("shards", [3, 8, 9, 16, 17, 24, 31, 32, 64])
@pytest.mark.parametrize("copies", [0.7, 1.5, 4.0, 70.0])
def test_rounds_of_one_length(shards, copies):
    """Lengths that occur `copies` times the number of shards each: rounds that need no sort, single ones and long runs of
    them, up to the list's end; in one launch and in portions."""
    rng = np.random.default_rng(int(10 * copies) + shards)
    for n in (2049, 6000, 16384, 33000):
        per = -(-n // shards) if n != 16384 else n // shards
        n = per * shards
        values = max(1, int(n / (copies * shards)))
        lens = (40 + rng.integers(0, values, n)).astype(np.int32)
        if n <= 16384:
            check_step(_custom(lens, 1, shards, 8192, fields=()), two_calls=True, label=f"{n} on {shards} shards, {values} lengths")
        else:
            _check_balance_ws(lens, shards, label=f"{n} on {shards} shards, {values} lengths")


def _plan_alone(lens, shards, budget, align=1, perm=None, n_src=1):
    """dc_plan as a call of its own, d_perm null unless given, every output against the oracle; shards: number of slots of each."""
    torch, binding, runner = _gpu()
    w = _custom(np.asarray(lens, np.int32), 1, len(shards), budget, n_src=n_src, fields=())
    d = runner.DeviceBatch(w, align_tokens=align, cap=w.n_seq, poison=True)
    off = np.concatenate([[0], np.cumsum(shards)]).astype(np.int32)
    assert off[-1] == w.n_seq
    d.shard_seq_off = torch.from_numpy(off).to(d.dev)
    d_perm = None if perm is None else torch.from_numpy(perm.astype(np.int32)).to(d.dev)
    binding.dc_plan(d.prm, d.source, d.seq_len, d_perm, d.shard_seq_off, d.capacity, d.dst_tok_off, d.shard_tok_off, d.shard_mb_off,
                    d.mb_seq_off, d.cu_seqlens, d.n_mb, d.ws, d.ws_bytes, d.status)
    torch.cuda.synchronize()
    assert d.read_status() == 0
    pl = oracle.plan(w.seq_len, np.arange(w.n_seq, dtype=np.int32) if perm is None else perm.astype(np.int32), off, budget, align)
    M = int(d.n_mb.item())
    assert M == pl.n_mb
    for got, want in ((d.dst_tok_off, pl.dst_tok_off), (d.shard_tok_off, pl.shard_tok_off), (d.shard_mb_off, pl.shard_mb_off),
                      (d.mb_seq_off[:M + 1], pl.mb_seq_off), (d.cu_seqlens[:w.n_seq + M], pl.cu_seqlens)):
        assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("slots,n_shards", [(150, 1), (300, 4), (150, 17), (150, 64), (9000, 1), (1000, 16), (256, 64), (150, 70), (16384, 1),
                                            (20000, 1), (16000, 2), (600, 64), (27000, 3), (33000, 1), (40000, 2), (300, 200)])
def test_micro_batches_where_long_sequences_come_last(slots, n_shards):
    """Slots in ascending length (a caller's order; the balance leaves them descending): behind a micro-batch of many short
    ones fewer slots are left than it held, and they do not fit.  Few shards and many, one that is walked in the LDS and one
    (32 768 slots and more) in global memory, the last one of a batch among them, without a permutation and with one."""
    longer = min(slots // 3, 200)
    budget = slots - longer                              # all the short ones in one micro-batch, then two at a time
    shard = np.concatenate([np.full(budget, 1), np.full(longer, budget // 2)])
    lens = np.tile(shard, n_shards)
    _plan_alone(lens, [slots] * n_shards, budget)
    _plan_alone(lens, [slots] * n_shards, budget, align=24)
    perm = np.random.default_rng(slots).permutation(len(lens))
    back = np.empty_like(lens)
    back[perm] = lens                                    # the same lengths in slot order
    _plan_alone(back, [slots] * n_shards, budget, perm=perm)


def _plan_of(lens, shards, budget, align):
    """The plan of slots of these lengths (0: an empty slot), straight from the header's text."""
    tok, stok, smb, mb, cu, base = [], [], [], [], [], 0
    j = 0
    for n in shards:
        stok.append(base); smb.append(len(mb))
        at = base
        used = None
        for ln in lens[j:j + n]:
            if used is None or used + ln > budget:
                if used is not None:
                    cu.append(used)
                mb.append(len(tok)); used = 0
            cu.append(used); tok.append(at)
            at += ln; used += ln
        if used is not None:
            cu.append(used)
        base += -(-(at - base) // align) * align
        j += n
    return dict(tok=tok + [base], stok=stok + [base], smb=smb + [len(mb)], mb=mb + [len(tok)], cu=cu)


@pytest.mark.parametrize("n,shards,align", [(1000, 8, 1), (1000, 8, 16), (16384, 16, 1), (16640, 16, 1), (20480, 16, 16), (66048, 129, 1)])
def test_a_repeat_in_perm_moves_nothing(n, shards, align):
    """Of the slots that name one sequence all but one (any) are empty: they take no room in the layout and move nothing, up
    to DC_MAX_SEQ slots and above.  The second call finds the first one's words in its buffers."""
    torch, binding, runner = _gpu()
    rng = np.random.default_rng(n)
    w = _custom(rng.integers(20, 200, n).astype(np.int32), 4, shards, 1024, n_src=2, fields=("i32",))
    d = runner.DeviceBatch(w, align_tokens=align, poison=True)
    d.balance(); torch.cuda.synchronize()
    perm = d.perm.cpu().numpy().copy()
    a, b, c = n - 2, n // 2 + 1, 5
    perm[a] = perm[b]                                    # one sequence twice, far apart; one three times, side by side
    perm[c + 1] = perm[c + 2] = perm[c]
    d.perm.copy_(torch.from_numpy(perm))
    off = np.concatenate([[0], np.cumsum(w.src_shard_tokens)])
    side = np.searchsorted(w.src_shard_seq_off, np.arange(n), side="right") - 1
    source = np.concatenate(w.fields[0].shards)
    for call in range(2):
        d.plan(); d.gather(); torch.cuda.synchronize()
        assert d.read_status() == binding.DC_ERR_BAD_LAYOUT
        d.status.zero_()
        M = int(d.n_mb.item())
        got = dict(tok=d.dst_tok_off, stok=d.shard_tok_off, smb=d.shard_mb_off, mb=d.mb_seq_off[:M + 1], cu=d.cu_seqlens[:n + M])
        got = {k: v.cpu().numpy() for k, v in got.items()}
        lens = w.seq_len[perm].astype(np.int64)
        fits = []
        for keep2 in (a, b):
            for keep3 in (c, c + 1, c + 2):
                x = lens.copy()
                x[[k for k in (a, b, c, c + 1, c + 2) if k not in (keep2, keep3)]] = 0
                want = _plan_of(x.tolist(), [n // shards] * shards, 1024, align)
                if all(np.array_equal(got[k], want[k]) for k in want):
                    fits.append(x)
        assert len(fits) == 1, (n, call)
        x = fits[0]
        arena = np.full(d.capacity, 0x5A5A5A5A, np.int32)
        for j in range(n):
            i = perm[j]
            at = off[side[i]] + w.src_tok_off[i]
            arena[got["tok"][j]:got["tok"][j] + x[j]] = source[at:at + x[j]]
        name = w.fields[0].name
        assert np.array_equal(d.dst_fields[name].cpu().numpy(), arena), (n, call)
        d.dst_fields[name].fill_(0x5A5A5A5A)


@pytest.mark.parametrize("kl", [0.0, 0.05])
@pytest.mark.parametrize("n,mean", [(2049, 200), (2049, 384), (2049, 386), (4097, 690), (4097, 715), (8192, 765), (8193, 955), (8193, 965),
                                    (4097, 2040), (4097, 2060), (8200, 2830)])
def test_gae_long_sequences_among_short_ones(n, mean, kl):
    """Each side of the lines between the ways of sharing, with sequences of up to 32 K tokens among them: alone in their
    set, more in one set than workgroups share it, and lengths round what counts as long."""
    rng = np.random.default_rng(n + mean)
    long_len = max(4 * mean, 2048)
    sets = -(-n // 64)
    at = np.concatenate([np.arange(7) * sets + 3, np.arange(2) * sets + sets - 1, [n - 1, n // 2, 11, 12, 13]])
    longs = np.concatenate([[long_len + 5, 9000, 9000, long_len, 12001, long_len + 1, 4096], [7000, 8192], [20000, 32768],
                            [long_len - 1, long_len, long_len + 1]])
    lens = rng.integers(max(1, mean // 4), max(2, 2 * mean - mean // 4), n)
    lens = np.maximum(1, (lens * (mean - longs.sum() / n) / lens.mean()).astype(np.int64))
    lens[at] = longs
    short = np.setdiff1d(np.arange(n), at)
    more, rest = divmod(mean * n - int(lens.sum()), len(short))
    lens[short] += more                                  # (exactly `mean` on average)
    lens[short[:rest]] += 1
    assert lens.min() > 0 and lens.sum() == mean * n
    w = _with_ppo_fields(_custom(lens.astype(np.int32), 1, 1, 1 << 20, fields=()), seed=n)
    check_gae(w, 0.99, 0.95, kl, label=f"{n} sequences of {mean}, long ones among them")


def _time(torch, call):
    for _ in range(3):
        call()
    best = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        for _ in range(20):
            call()
        b.record()
        torch.cuda.synchronize()
        best.append(a.elapsed_time(b) / 20)
    return min(best)


@pytest.mark.parametrize("kl", [0.0, 0.05])
@pytest.mark.parametrize("n,mean,longs", [(4096, 300, 1), (16384, 300, 1), (4096, 1200, 1), (16384, 1000, 1), (4096, 150, 64), (16384, 150, 64),
                                          (16384, 150, 128)])
def test_gae_is_not_held_up_by_long_sequences(n, mean, longs, kl):
    """A 32 K-token sequence among short ones, or one of 8192 at the same place in every group of a power of two, starts early
    and has the waves of a batch of its own: the call takes no longer than the batch without them and twice them alone
    together (a third to two thirds of that are measured; left to one or two waves' iterations it took 0.8 to 1.5 times
    that, left to a few workgroups one after the other up to 7)."""
    torch, binding, runner = _gpu()
    rng = np.random.default_rng(n)
    lens = np.maximum(1, rng.integers(mean // 2, mean * 3 // 2, n))
    mixed = lens.copy()
    mixed[:: n // longs] = 32768 if longs == 1 else 8192
    times = []
    for x in (lens, mixed, mixed[:: n // longs]):
        d = runner.DeviceBatch(_with_ppo_fields(_custom(x.astype(np.int32), 1, 1, 1 << 20, fields=()), seed=n))
        d.prepare_gae()
        times.append(_time(torch, lambda: d.gae(1.0, 0.95, kl)))
    print([round(1e3 * t, 1) for t in times], round(times[1] / (times[0] + 2.0 * times[2]), 2))
    assert times[1] < times[0] + 2.0 * times[2], times


@pytest.mark.parametrize("n,shards,n_src", [(24576, 2, 1), (24577, 1, 1), (49152, 3, 8), (140000, 4, 4)])
def test_advantages_of_long_sequences_among_short_ones(n, shards, n_src):
    """Eight short sequences to a wave and long ones (4096 tokens and more) to whole workgroups: neighbours, one set's, the
    first and the last sequence, lengths round the line, ends anywhere in a 16-byte chunk; sets that take more than one look."""
    rng = np.random.default_rng(n)
    lens = rng.integers(1, 40, n)
    at = np.unique(np.concatenate([[0, n - 1], np.arange(9) + n // 3, np.arange(4) * 509 + 77]))
    lens[at] = rng.integers(4080, 4120, len(at))
    lens[at[::3]] = 4096 + np.arange(len(at[::3])) - 2
    lens[at[1]] = 40001
    lens[n // 2:n // 2 + 12] = rng.integers(1020, 4096, 12)      # longer than a wave's four steps, not long
    w = _custom(lens.astype(np.int32), 1 if n % 2 else 4, shards, 1 << 17, n_src=n_src, seed=n, fields=())
    check_step(w, label=f"{n} sequences, long ones among them")


@pytest.mark.parametrize("together", [True, False])
@pytest.mark.parametrize("n,mean", [(16384, 200), (65536, 100)])
def test_advantages_are_not_held_up_by_long_sequences(n, mean, together):
    """64 sequences of 32 K tokens among short ones, side by side or all over the batch: no more than the batch without them
    and twice the 64 alone together (half of that is measured; one wave after the other through them took 2 to 9 times it)."""
    torch, binding, runner = _gpu()
    rng = np.random.default_rng(n)
    lens = rng.integers(mean // 2, mean * 3 // 2, n)
    mixed = lens.copy()
    mixed[np.arange(64) + n // 3 if together else np.arange(64) * (n // 64) + 5] = 32768
    times = []
    for x in (lens, mixed, np.full(64, 32768)):
        d = runner.DeviceBatch(_custom(x.astype(np.int32), 8, 1, 1 << 20, fields=()))
        times.append(_time(torch, d.group_advantage))
    assert times[1] < times[0] + 2.0 * times[2], times


@pytest.mark.parametrize("empties", [3, 15, 17, 40, 130])
def test_empty_slots_in_a_crowded_granule(empties):
    """Slots that fail a check take no tokens; however many stand in a row, the sequences on both sides of them are moved whole
    (every field width, and the advantages made on the way)."""
    torch, binding, runner = _gpu()
    rng = np.random.default_rng(empties)
    n = 6000
    lens = rng.integers(1, 30, n).astype(np.int32)
    w = _custom(lens, 1, 3, 4096, n_src=3, seed=empties, fields=("i32", "bf16"))
    none = np.zeros(n, bool)
    at = 5
    while at + empties < n:
        none[at:at + empties] = True
        at += empties + int(rng.integers(1, 70))
    d = runner.DeviceBatch(w, poison=True)
    d.seq_len[torch.from_numpy(np.flatnonzero(none)).to(d.dev)] = 0
    off = torch.from_numpy(w.src_shard_seq_off).to(d.dev)
    d.perm.copy_(torch.arange(n))
    d.adv_seq.copy_(torch.from_numpy(rng.standard_normal(n).astype(np.float32)))
    binding.dc_plan(d.prm, d.source, d.seq_len, d.perm, off, d.capacity, d.dst_tok_off, d.shard_tok_off, d.shard_mb_off, d.mb_seq_off,
                    d.cu_seqlens, d.n_mb, d.ws, d.ws_bytes, d.status)
    torch.cuda.synchronize()
    assert d.read_status() == binding.DC_ERR_ZERO_LENGTH_SEQ
    left = np.where(none, 0, lens).astype(np.int64)
    tok = np.cumsum(left) - left
    assert np.array_equal(d.dst_tok_off.cpu().numpy()[:n], tok)
    base = np.repeat(np.concatenate([[0], np.cumsum(w.src_shard_tokens)[:-1]]), n // 3)
    source = np.concatenate([np.arange(ln) + b + o for ln, b, o in zip(left, base, w.src_tok_off)])
    total = int(left.sum())
    d.gather(); torch.cuda.synchronize()
    for f in w.fields:
        got = d.dst_fields[f.name].cpu().numpy()
        want = np.concatenate([np.frombuffer(s.tobytes(), got.dtype) for s in f.shards])[source]
        assert np.array_equal(got[:total], want), f.name
        assert np.all(got[total:] == np.frombuffer(b"\x5a" * f.elem_bytes, got.dtype)[0]), f.name
        d.dst_fields[f.name].fill_(0)
    d.gather_advantage(); torch.cuda.synchronize()
    mask = np.concatenate(w.field_by_name("mask").shards)[source]
    want = np.where(mask != 0, np.repeat(d.adv_seq.cpu().numpy(), left), np.float32(0))
    assert np.array_equal(d.dst_fields["mask"].cpu().numpy()[:total], mask)
    assert np.array_equal(d.dst_fields["adv_tok"].view(torch.float32).cpu().numpy()[:total].view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("n", [300, 5000, 40000])
def test_scatter_with_offsets_that_do_not_rise(n):
    """Rollout offsets in another order than the sequences' are refused; what is written all the same stands in its place."""
    torch, binding, runner = _gpu()
    rng = np.random.default_rng(n)
    lens = rng.integers(1, 60, n).astype(np.int32)
    w = _custom(lens, 1, 1, 4096, fields=("i32",))
    d = runner.DeviceBatch(w)
    d.balance(); d.plan(); torch.cuda.synchronize()
    order = rng.permutation(n)
    start = np.empty(n, np.int64)
    start[order] = np.cumsum(lens[order], dtype=np.int64) - lens[order]
    name = w.fields[0].name
    d.dst_fields[name].copy_(torch.arange(d.capacity, dtype=torch.int32))
    d.prepare_scatter([name], fill=0x7F)
    d.src_tok_off.copy_(torch.from_numpy(start))
    d.scatter(); torch.cuda.synchronize()
    assert d.read_status() == binding.DC_ERR_BAD_LAYOUT
    slot = np.empty(n, np.int64)
    slot[d.perm.cpu().numpy()] = np.arange(n)
    want = np.empty(w.total_tokens, np.int64)
    tok = d.dst_tok_off.cpu().numpy()
    for i in range(n):
        want[start[i]:start[i] + lens[i]] = tok[slot[i]] + np.arange(lens[i])
    got = d.back_fields[name][0].cpu().numpy()
    assert np.all((got == 0x7F7F7F7F) | (got == want))


@pytest.mark.parametrize("n,shards,budget,align", [
    (2049, 3, 41, 1), (2560, 5, 4096, 1),                # 512 slots of a shard and more: one and two steps of the workgroup
    (2044, 4, 97, 9000), (2048, 4, 97, 9000), (2052, 4, 97, 9000),
    (4094, 2, 1000, 6), (4096, 2, 41, 1), (4098, 2, 41, 1),      # the last whose sources are staged, and the first beyond
    (16384, 1, 77, 1), (16384, 1, 1 << 20, 1), (16383, 3, 300, 16), (16384, 4, 5000, 1),
    (16384, 64, 41, 1), (16320, 64, 2000, 16), (16380, 65, 41, 1), (16320, 255, 60, 3), (16384, 256, 2000, 1),
])
def test_plan_by_shards(n, shards, budget, align):
    """Two launches: Algorithm 1, then workgroups that each plan a shard; shards of one slot to all of them, budgets from one
    slot to a whole shard, a word and a byte for a shard's number of micro-batches."""
    lens = np.random.default_rng(n + budget).integers(1, 41, n).astype(np.int32)
    w = _custom(lens, 1, shards, budget, n_src=3 if n % 3 == 0 else 1, seed=n, fields=("i32",))
    check_step(w, align=align, two_calls=True, label=f"{n} slots on {shards} shards, budget {budget}")


@pytest.mark.parametrize("shards,per", [(256, 1), (256, 2), (200, 3), (128, 5), (100, 9), (64, 17)])
@pytest.mark.parametrize("longest", [60000, 70000])
def test_granules_that_many_small_shards_share(shards, per, longest):
    """Granules whose record holds slots of the next shards, of which one granule holds dozens, beside long sequences."""
    n = shards * per
    rng = np.random.default_rng(n)
    lens = rng.integers(1, 12, n)
    at = rng.permutation(n)[: 3200000 // longest]
    lens[at] = rng.integers(longest - 2000, longest, len(at))
    w = _custom(lens.astype(np.int32), 1, shards, 1 << 20, n_src=2 if n % 2 == 0 else 1, seed=n, fields=("i32",))
    check_step(w, align=1 if per % 2 else 5, two_calls=True, label=f"{shards} shards of {per}")
    check_gather_advantage(w, label=f"{shards} shards of {per}")


@pytest.mark.parametrize("n,shards", [(4096, 64), (2560, 256), (12288, 3)])
def test_plan_by_shards_with_slots_that_fail_a_check(n, shards):
    """Sequences whose place in the rollout layout is refused take their tokens' room but move nothing, however many of them
    stand in a row at a shard's end; all others are moved whole."""
    torch, binding, runner = _gpu()
    rng = np.random.default_rng(n)
    w = _custom(rng.integers(1, 90, n).astype(np.int32), 1, shards, 4096, seed=n, fields=("i32",))
    bal = oracle.balance(w.seq_len, shards)
    bad = np.zeros(n, bool)                                      # (by slot)
    per = n // shards
    for k in range(1, shards, 3):
        bad[k * per - rng.integers(0, per): k * per + rng.integers(0, 40)] = True
    bad[-5:] = True
    d = runner.DeviceBatch(w, align_tokens=3, poison=True)
    d.adv_tok_src = None
    grown = d.capacity + 3000 * 1024                             # (an arena above the single launch's limit)
    d.capacity = grown
    d.ws_bytes = binding.dc_workspace_bytes(d.prm, grown)
    d.ws = torch.full((d.ws_bytes,), 0x7F, dtype=torch.uint8, device=d.dev)
    dst = torch.full((grown,), 0x5A5A5A5A, dtype=torch.int32, device=d.dev)
    name = w.fields[0].name
    d.src_tok_off[torch.from_numpy(bal.perm[bad].astype(np.int64)).to(d.dev)] = -1
    binding.dc_balance_plan_group_advantage(
        d.prm, d.source, d.seq_len, d.perm, d.shard_seq_off, d.shard_of_seq, d.shard_load, d.reward, d.group_off, w.n_groups,
        None, d.adv_seq, None, grown, d.dst_tok_off, d.shard_tok_off, d.shard_mb_off, d.mb_seq_off, d.cu_seqlens, d.n_mb,
        d.ws, d.ws_bytes, d.status)
    binding.dc_gather(d.prm, d.source, binding.Fields([(d.src_fields[name], dst, 4)]), grown, d.dst_tok_off, d.ws, d.ws_bytes,
                      d.status)
    torch.cuda.synchronize()
    assert d.read_status() == binding.DC_ERR_BAD_LAYOUT
    pl = oracle.plan(w.seq_len, bal.perm, bal.shard_seq_off, w.token_budget, 3)
    assert np.array_equal(d.perm.cpu().numpy(), bal.perm) and np.array_equal(d.dst_tok_off.cpu().numpy(), pl.dst_tok_off)
    assert np.array_equal(d.shard_mb_off.cpu().numpy(), pl.shard_mb_off)
    want = np.full(grown, 0x5A5A5A5A, np.int32)
    for j in np.flatnonzero(~bad):
        i = bal.perm[j]
        want[pl.dst_tok_off[j]:pl.dst_tok_off[j] + w.seq_len[i]] = w.fields[0].shards[0][w.src_tok_off[i]:][:w.seq_len[i]]
    assert np.array_equal(dst.cpu().numpy(), want)


@pytest.mark.parametrize("n,shards", [(1, 1), (64, 4), (127, 127), (128, 2), (128, 128), (129, 3), (130, 2), (192, 3), (256, 4), (256, 256),
                                      (195, 3), (260, 5)])
@pytest.mark.parametrize("entries", [17, 1040, 2048, 2049])
def test_single_launch_of_a_very_small_batch(n, shards, entries):
    """Up to 128 sequences, 256 on shards of up to 64, and 2048 table entries in one launch; a little more of any in two."""
    tokens = (entries - 16) * 1024
    rng = np.random.default_rng(n + entries)
    lens = rng.integers(max(1, tokens // n // 3), max(2, tokens // n), n)
    lens[n // 2] += tokens - int(lens.sum())
    w = _custom(lens.astype(np.int32), 1, shards, 1 << 22, n_src=3 if n % 3 == 0 else 1, seed=n, fields=("i32",))
    check_step(w, two_calls=True, label=f"{n} sequences, {entries} entries")


@pytest.mark.parametrize("align", [1, 7, 16])
@pytest.mark.parametrize("lo,hi", [(300, 900), (900, 5000)])
def test_edges_of_granules_with_riders(lo, hi, align):
    """Up to four slots to a granule, their ends and starts anywhere in a 16-byte chunk, with and without padding between
    shards, in an arena large enough that the narrow fields ride on the 4-byte fields' waves; both directions."""
    rng = np.random.default_rng(lo + align)
    n = 12 * (6400000 // 12 // ((lo + hi) // 2))
    lens = rng.integers(lo, hi, n).astype(np.int32)
    w = _custom(lens, 4, 12, 1 << 15, n_src=3, seed=lo + align)
    check_step(w, align=align, label=f"{n} sequences, riders", two_calls=n <= 16384)
    if align == 7:
        check_gather_advantage(w, align=align, label=f"{n} sequences, riders")
        check_scatter(w, label=f"{n} sequences, riders")


@pytest.mark.parametrize("n_src", [1, 3])
def test_two_byte_field_beside_one_four_byte_field(n_src):
    """3000 workgroups of one 4-byte field, where a 2-byte field has its own, and 6000 of two, where it rides with a 1-byte field."""
    lens = np.random.default_rng(n_src).integers(1000, 5000, 4200).astype(np.int32)
    w = _custom(lens, 4, 12, 1 << 15, n_src=n_src, seed=n_src)
    assert 3000 <= w.total_tokens // 4096 < 8192
    check_gather_advantage(w, align=7, label="one 4-byte and one 2-byte carrier")
    check_scatter(w, label="the same, back")


@pytest.mark.parametrize("kind", ["geometric", "equal", "long", "rising", "few"])
@pytest.mark.parametrize("n", [16385, 24576, 24577, 32769, 65536, 65537, 131072, 131073])
def test_sort_by_portions(n, kind):
    """Portions of 8192 sequences, sorted each and merged by counting: the last portion of one sequence and a whole one, four,
    eight and sixteen portions and one more, lengths that many sequences of every portion share, and lengths of 2^16 and more."""
    rng = np.random.default_rng(n)
    lens = np.arange(n) % 40000 + 1 if kind == "rising" else rng.integers(5, 9, n) if kind == "few" else _lengths(kind, n, rng)
    _check_balance_ws(lens.astype(np.int32), 8, cap=-(-n // 8) if n % 8 else 0, label=f"{n} sequences, {kind}")


@pytest.mark.parametrize("n,n_src,longest", [(16384, 1, 14), (16390, 2, 14), (32767, 1, 14), (32768, 4, 14), (32772, 3, 14), (22527, 1, 14),
                                             (22528, 2, 14), (22528, 4, 470), (32767, 1, 470), (32768, 1, 470)])
def test_heads_and_tails_of_short_sequences(n, n_src, longest):
    """Four and eight short sequences to a wave, each starting and ending anywhere in a 16-byte chunk: sequences inside one
    chunk, of one chunk, and without a whole one."""
    rng = np.random.default_rng(n)
    lens = rng.integers(1, longest, n)
    lens[::11] = rng.integers(250, 262, len(lens[::11]))
    lens[5::1001] = rng.integers(1020, 1030, len(lens[5::1001]))
    check_step(_custom(lens.astype(np.int32), 1 if n % 2 else 2, 1, 1 << 16, n_src=n_src, seed=n, fields=()), label=f"{n} sequences")


@pytest.mark.parametrize("n,shards", [(3072, 24), (2560, 160)])
def test_plan_by_shards_replayed_and_on_two_streams(n, shards):
    """The shards' counts travel through words of the workspace that the launch before clears: a captured step gives the same
    whatever the workspace holds before a replay, and steps of two buffer sets on two streams do not see each other's."""
    torch, binding, runner = _gpu()
    rng = np.random.default_rng(n)
    ws = [_custom(rng.integers(1, 400, n).astype(np.int32), 8, shards, b, n_src=2, seed=b, fields=("i32",)) for b in (512, 4096)]
    ds = [runner.DeviceBatch(w, poison=True) for w in ws]
    for d in ds:
        d.step_two_calls()
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        ds[0].step_two_calls()
    for rep in range(3):
        ds[0].ws.fill_(0x7F if rep else 0)
        for t in (ds[0].perm, ds[0].cu_seqlens, ds[0].dst_tok_off, ds[0].shard_mb_off, ds[0].shard_of_seq):
            t.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        compare_step(ds[0], ws[0])
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    for rep in range(6):
        with torch.cuda.stream(streams[rep % 2]):
            ds[rep % 2].step_two_calls()
    torch.cuda.synchronize()
    for d, w in zip(ds, ws):
        compare_step(d, w)


@pytest.mark.parametrize("n,shards,budget,longest,whole", [
    (2049, 1, 1 << 25, 1 << 24, False), (4100, 2, (1 << 31) - 1, 1 << 24, False), (16384, 4, 1 << 24, 1 << 24, False),
    (16384, 1, (1 << 31) - 1, 1 << 24, False), (2112, 1, 100_000_000, 1 << 22, True),
])
def test_plan_by_shards_of_more_than_32_bits_of_tokens(n, shards, budget, longest, whole):
    """Shards of 2^32 tokens and more, in an arena that ends early (the overflow is reported, and every table is still what dc_plan
    makes of the same batch) and in one that takes them all."""
    torch, binding, _ = _gpu()
    rng = np.random.default_rng(n)
    lens = rng.integers(longest - longest // 8, longest + 1, n).astype(np.int32)
    off = np.cumsum(lens, dtype=np.int64) - lens
    total = int(lens.sum(dtype=np.int64))
    assert total // shards > 1 << 32
    capacity = total if whole else 1 << 20
    dev = "cuda:0"

    def ints(k, dtype=torch.int32):
        return torch.zeros(k, dtype=dtype, device=dev)

    prm = binding.make_params(n, shards, budget)
    seq_len = torch.from_numpy(lens).to(dev)
    src = binding.Source([0, n], [total], torch.from_numpy(off).to(dev))
    reward, adv_seq = torch.zeros(n, device=dev), torch.zeros(n, device=dev)
    group_off = torch.arange(n + 1, dtype=torch.int32, device=dev)
    perm, seq_off, shard_of, load = ints(n), ints(shards + 1), ints(n), ints(shards, torch.int64)
    ws_bytes = binding.dc_workspace_bytes(prm, capacity)
    got = []
    for separate in (False, True):
        out = [ints(n + 1, torch.int64), ints(shards + 1, torch.int64), ints(shards + 1), ints(n + 1), ints(2 * n), ints(1)]
        ws, status = torch.full((ws_bytes,), 0x7F, dtype=torch.uint8, device=dev), ints(1)
        if separate:
            binding.dc_plan(prm, src, seq_len, perm, seq_off, capacity, *out, ws, ws_bytes, status)
        else:
            binding.dc_balance_plan_group_advantage(prm, src, seq_len, perm, seq_off, shard_of, load, reward, group_off, n, None,
                                                    adv_seq, None, capacity, *out, ws, ws_bytes, status)
        torch.cuda.synchronize()
        assert int(status.item()) == (binding.DC_OK if whole else binding.DC_ERR_OVERFLOW)
        got.append((out, ws[:ws_bytes - 512]))                    # (behind the tables: the plan's own words)
    bal = oracle.balance(lens, shards)
    assert np.array_equal(perm.cpu().numpy(), bal.perm) and np.array_equal(load.cpu().numpy(), bal.shard_load)
    pl = oracle.plan(lens, bal.perm, bal.shard_seq_off, budget)
    for out, _ in got:
        tok, shard_tok, shard_mb, mb, cu, n_mb = (t.cpu().numpy() for t in out)
        assert n_mb[0] == pl.n_mb and np.array_equal(tok, pl.dst_tok_off) and np.array_equal(shard_tok, pl.shard_tok_off)
        assert np.array_equal(shard_mb, pl.shard_mb_off) and np.array_equal(mb[:pl.n_mb + 1], pl.mb_seq_off)
        assert np.array_equal(cu[:n + pl.n_mb], pl.cu_seqlens)
    assert torch.equal(got[0][1], got[1][1])                      # the granule tables and the slots' sources


@pytest.mark.parametrize("looks", [0, 1, 3])
@pytest.mark.parametrize("n,shards,budget,align", [(2048, 2, 41, 1), (3072, 24, 300, 6), (4096, 64, 97, 1), (2600, 65, 97, 8), (2560, 256, 60, 1),
                                                   (4098, 2, 41, 1), (12288, 4, 5000, 3), (16383, 3, 300, 1)])
def test_plan_by_shards_whose_counts_do_not_come(n, shards, budget, align, looks, monkeypatch):
    """Walkers that do not find another shard's count count that shard themselves and walk their own again: with no looks at all
    shards before their own, with one or three at those that come late."""
    import ctypes
    _, binding, _ = _gpu()
    lib = binding.load()
    call = lib.dc_test_balance_plan_looks
    call.restype, call.argtypes = ctypes.c_int, [ctypes.c_int32] + lib.dc_balance_plan_group_advantage.argtypes
    monkeypatch.setattr(lib, "dc_balance_plan_group_advantage", lambda *a: call(looks, *a))
    lens = np.random.default_rng(n + budget).integers(1, 41, n).astype(np.int32)
    w = _custom(lens, 1, shards, budget, n_src=3 if n % 3 == 0 else 1, seed=n, fields=("i32",))
    check_step(w, align=align, two_calls=True, label=f"{n} slots on {shards} shards, {looks} looks")


@pytest.mark.parametrize("n,shards", [(64, 16), (256, 4), (512, 4), (2560, 256), (4096, 64), (4100, 2), (16384, 4)])
def test_status_codes_of_balance_and_plan_in_one_call(n, shards):
    """What the call refuses on the device, in one launch, planned by shards, and with shards of more than 2048 slots; what a
    refusal leaves whole is right."""
    torch, binding, runner = _gpu()
    rng = np.random.default_rng(n)
    lens = rng.integers(1, 60, n).astype(np.int32)
    lens[n // 3] = 200
    w = _custom(lens, 1, shards, 100, n_src=2, seed=n, fields=("i32",))
    d = runner.DeviceBatch(w)
    d.step_two_calls(); torch.cuda.synchronize()
    assert d.read_status() == binding.DC_ERR_SEQ_EXCEEDS_BUDGET        # 200 > budget 100: alone in its micro-batch
    bal = oracle.balance(w.seq_len, shards)
    assert np.array_equal(d.perm.cpu().numpy(), bal.perm) and np.array_equal(d.shard_of_seq.cpu().numpy(), bal.shard_of_seq)
    assert np.array_equal(d.dst_tok_off.cpu().numpy(), oracle.plan(w.seq_len, bal.perm, bal.shard_seq_off, 1 << 20).dst_tok_off)

    w = _custom(lens, 1, shards, 4096, n_src=2, seed=n, fields=("i32",))
    for at in (0, n // 2, n - 1):
        for bad in (0, -7, (1 << 24) + 1):
            d = runner.DeviceBatch(w)
            d.seq_len[at] = bad
            d.capacity = 1 << 17                                       # (what its arenas do not have is not gathered)
            d.ws_bytes = binding.dc_workspace_bytes(d.prm, d.capacity)
            d.ws = torch.zeros(d.ws_bytes, dtype=torch.uint8, device=d.dev)
            d.balance_plan_group_advantage(); torch.cuda.synchronize()
            assert d.read_status() == binding.DC_ERR_ZERO_LENGTH_SEQ
    for align in (1, 5):
        d = runner.DeviceBatch(w, align_tokens=align)
        pl = oracle.plan(w.seq_len, bal.perm, bal.shard_seq_off, w.token_budget, align)
        d.capacity = int(pl.dst_tok_off[-1]) - 1                       # arena one token short
        d.step_two_calls(); torch.cuda.synchronize()
        assert d.read_status() == binding.DC_ERR_OVERFLOW
        assert np.array_equal(d.dst_tok_off.cpu().numpy(), pl.dst_tok_off) and int(d.n_mb.item()) == pl.n_mb
        assert np.array_equal(d.cu_seqlens.cpu().numpy()[:n + pl.n_mb], pl.cu_seqlens)
    for at in (1, n - 1):
        d = runner.DeviceBatch(w)
        d.src_tok_off[at] = int(w.src_shard_tokens[at // (n // 2)])    # a sequence that would start beyond its buffer
        d.step_two_calls(); torch.cuda.synchronize()
        assert d.read_status() == binding.DC_ERR_BAD_LAYOUT


@pytest.mark.parametrize("kind", ["geometric", "equal", "tail", "long"])
@pytest.mark.parametrize("n,shards", [(1, 1), (63, 1), (129, 1), (2048, 1), (2049, 1), (16384, 1), (2, 2), (6, 2), (130, 2), (2050, 2), (16384, 2),
                                      (3, 3), (21, 3), (387, 3), (2052, 3), (16383, 3), (4, 4), (12, 4), (128, 4), (260, 4), (2052, 4), (16384, 4)])
def test_up_to_four_workers(n, shards, kind):
    """Sorts of two and four lanes, and the one partition that needs none: the ends of the kernels' ranges, rounds left over."""
    lens = _lengths(kind, n, np.random.default_rng(n + 31 * shards)).astype(np.int32)
    w = _custom(np.minimum(lens, 2000) if kind == "tail" and n > 1000 else lens, 1, shards, 1 << 17, fields=())
    check_step(w, align=7, label=f"{n} on {shards}, {kind}, one call", two_calls=True)
    check_step(w, align=7, label=f"{n} on {shards}, {kind}")


@pytest.mark.parametrize("kind", ["geometric", "equal", "tail"])
@pytest.mark.parametrize("shards,per", [(65, 1), (65, 2), (66, 3), (100, 2), (127, 3), (128, 2), (129, 2), (200, 3), (255, 4), (256, 2), (256, 5), (96, 40)])
def test_last_items_of_many_workers(shards, per, kind):
    """More than 64 workers: the last 64 items are placed by the 64 smallest keys alone, whichever rounds come before them."""
    lens = _lengths(kind, shards * per, np.random.default_rng(shards * per)).astype(np.int32)
    w = _custom(lens, 1, shards, 1 << 17, fields=())
    check_step(w, label=f"{shards} shards of {per}, {kind}", two_calls=True)


@pytest.mark.parametrize("kind", ["geometric", "long"])
@pytest.mark.parametrize("shards", [1, 4, 5, 16, 17, 32, 33, 63, 64, 65, 256])
def test_balance_calls_of_their_own(shards, kind):
    """dc_balance and dc_balance_group_advantage at the ends of their kernels' ranges of workers, equal partitions and unequal ones
    (64 workers: two kernels)."""
    rng = np.random.default_rng(7 * shards)
    for n, cap in ((shards * 7, 0), (2048 // shards * shards, 0), (2049 // shards * shards + (shards > 1), 2049 // shards + 3)):
        lens = _lengths(kind, n, rng).astype(np.int32)
        _check_balance_ws(lens, shards, cap=cap, label=f"{n} on {shards}, {kind}, cap {cap}")
        check_step(_custom(lens, 1, shards, 1 << 17, fields=()), cap=cap, align=7, fused=True, label=f"{n} on {shards}, {kind}, cap {cap}")


@pytest.mark.parametrize("shards", [2, 3, 4, 33, 40, 63])
def test_packed_keys_rebased_at_the_narrow_widths_and_with_idle_lanes(shards):
    """More than 2^24 tokens to a worker, so that its key passes 2^30 inside the packed rounds: sorts of two and four lanes, and 64 lanes
    of which some keep no worker, whose keys must stay where they are; in one launch and in portions."""
    rng = np.random.default_rng(shards)
    for per in (16384 // shards, 33000 // shards + 1):
        _check_balance_ws(rng.integers(40000, 65536, shards * per), shards, label=f"{shards} workers, {per} long sequences each")


@pytest.mark.parametrize("shards", [33, 40, 63])
@pytest.mark.parametrize("copies", [1.5, 70.0])
def test_rounds_of_one_length_with_idle_lanes(shards, copies):
    """33 to 63 workers: rounds that need no sort, which only the kernel that works in portions leaves unsorted."""
    rng = np.random.default_rng(int(10 * copies) + shards)
    for n in (2049, 16384, 33000):
        per = n // shards + (n != 16384)
        values = max(1, int(per / copies))
        lens = (40 + rng.integers(0, values, per * shards)).astype(np.int32)
        _check_balance_ws(lens, shards, label=f"{per * shards} on {shards} shards, {values} lengths")
