"""The work that a user of this library has it do, as cases to be timed.

A case names a reference (its length and the kind of its repeats), a batch of
reads and the entry point that takes it.  The recipes are those of the
benchmark and the tests: order-3 Markov references of GC 0.41 with tandem or
interspersed repeats, reads copied from the reference with substitutions and
a share of unrelated reads, and now and then a base that the sequencer could
not call (N).

entry        what is called
"device"     match_batch_dev on reads resident in device memory
"host"       match_batch on reads in host memory
"locate"     locate_dev on the results of a batch
"build"      sa_build_device on a new reference, then the first batch
"serve"      a burst of requests to a Server over two resident references

settings     "default" (no configuration given) or "graph" (the launch
             settings that the autotuner found for 150-base reads, replayed
             as a hipGraph on a stream of the program's own)
"""
import zlib

import torch

import paper_1303_3692_amd as S

MAX_BASES = 1 << 29  # a drawn batch holds at most this many bases


def _case(name, entry, n, reads, lo, hi, *, repeats="tandem", random=0.3, rate_lo=0.0, rate_hi=0.02, unknown=0.0,
          settings="default", cap=0, requests=0):
    c = {"name": name, "entry": entry, "n": n, "reads": reads, "lo": lo, "hi": hi, "repeats": repeats,
         "random": random, "rate_lo": rate_lo, "rate_hi": rate_hi, "unknown": unknown, "settings": settings,
         "cap": cap, "requests": requests}
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # an interactive lookup, or the tail of a stream: one small call against a resident genome
        _case("few_reads", "device", 16_000_000, 64, 30, 300),
        # a spike-in control or an amplicon: a reference of a few kilobases, below the size that gets a prefix table
        _case("amplicon", "device", 3_000, 20_000, 150, 150, repeats="none", rate_hi=0.01),
        # short tags against a bacterial-sized reference: 100,000 x 25 bp on 1 Mbp
        _case("tags", "device", 1_000_000, 100_000, 25, 25, repeats="none", random=0.5, rate_hi=0.01),
        # an ordinary lane of fixed-length reads: 4,000,000 x 100 bp on 16 Mbp
        _case("lane_100", "device", 16_000_000, 4_000_000, 100, 100),
        # trimmed reads of uneven length, some with uncalled bases: 4,000,000 x 20-300 bp on 16 Mbp
        _case("ragged", "device", 16_000_000, 4_000_000, 20, 300, unknown=0.01),
        # the benchmark's step: 64,000,000 x 150 bp on 250 Mbp, tuned launch settings under a graph
        _case("chromosome", "device", 250_000_000, 64_000_000, 150, 150, repeats="interspersed", random=0.2,
              rate_lo=0.01, rate_hi=0.01, settings="graph"),
        # the paper's query shape: 1024-base queries on 10 Mbp
        _case("queries_1024", "device", 10_000_000, 65_536, 1024, 1024, random=0.5, rate_hi=0.01),
        # a run of long and short reads together: both sides of 320 bases in one batch
        _case("mixed_long", "device", 16_000_000, 50_001, 20, 1024, unknown=0.01),
        # reads that come from a file into host memory, with the results wanted there
        _case("from_host", "host", 16_000_000, 1_000_000, 150, 150),
        # positions of a mapped batch, at most 16 each
        _case("positions", "locate", 16_000_000, 1_000_000, 100, 100, cap=16),
        # a new reference: index it and map the first batch
        _case("new_reference", "build", 16_000_000, 200_000, 100, 100),
        # requests of 1-100,000 reads that arrive together at a server with two resident references
        _case("requests", "serve", 16_000_000, 0, 30, 300, requests=32),
    ]


def _log(rng, lo, hi):
    """An integer in [lo, hi], spread over its logarithm."""
    return int(min(hi, max(lo, round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    entry = rng.choice(["device"] * 5 + ["host", "locate", "build", "serve"])
    shape = rng.choice(["fixed", "fixed", "ragged", "ragged", "long", "any"])
    lo, hi = {"fixed": (20, 320), "ragged": (20, 320), "long": (321, 1024), "any": (20, 1024)}[shape]
    lo = rng.randint(lo, hi)
    hi = lo if shape in ("fixed", "long") else rng.randint(lo, hi)
    n = _log(rng, 2_000, 32_000_000)
    reads = _log(rng, 1, 4_000_000)
    requests = 0
    if entry == "build":
        n, reads = _log(rng, 2_000, 16_000_000), _log(rng, 1, 200_000)
    elif entry == "host":
        reads = _log(rng, 1, 1_000_000)
    elif entry == "serve":
        n, reads, requests = _log(rng, 100_000, 16_000_000), 0, rng.randint(1, 32)
        lo, hi = rng.randint(30, 100), rng.randint(100, 300)
    return _case(None, entry, n, min(reads, MAX_BASES // hi), lo, hi,
                 repeats=rng.choice(["none", "tandem", "interspersed"]), random=rng.choice([0.0, 0.2, 0.3, 0.5]),
                 rate_hi=rng.choice([0.0, 0.01, 0.02]), unknown=rng.choice([0.0, 0.01]),
                 cap=rng.choice([1, 4, 16, 100]) if entry == "locate" else 0, requests=requests)


# ------------------------------------------------------------------ inputs


def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _generator(*seed):
    g = torch.Generator(device=_device())
    g.manual_seed(zlib.crc32(repr(seed).encode()))
    return g


def _rand(g, *size):
    return torch.rand(size, generator=g, device=g.device)


def _randint(g, hi, *size):
    return torch.randint(0, hi, size, generator=g, device=g.device)


def _markov(n, g):
    """Codes 0..3 of an order-3 chain, as segments that run side by side."""
    w = torch.tensor([0.295, 0.205, 0.205, 0.295], device=g.device) * (0.8 + 0.4 * _rand(g, 64, 4))
    w[1::4, 2] *= 0.3  # few G after C
    cdf = torch.cumsum(w / w.sum(1, keepdim=True), 1)[:, :3].contiguous()
    length = min(n, 2048)
    chains = -(-n // length)
    state = _randint(g, 64, chains)
    out = torch.empty((length, chains), dtype=torch.uint8, device=g.device)
    for t in range(length):
        base = (_rand(g, chains, 1) > cdf[state]).sum(1)
        out[t] = base
        state = ((state << 2) | base) & 63
    return out.t().reshape(-1)[:n].contiguous()


def _add_repeats(codes, kind, g):
    """Overwrites 5 % of the text with tandem arrays (units of 2-6 bases, 10-50
    copies), or 10 % with copies of twenty 300-base elements at 10 % divergence,
    each in a slot of its own."""
    n, width = codes.numel(), 300
    share = {"none": 0.0, "tandem": 0.05 * 300 / 120, "interspersed": 0.10}[kind]
    count = int(share * n / width)
    if not count or n // count < width:
        return codes
    at = torch.arange(width, device=g.device)
    step = 1 << 18
    elements = _randint(g, 4, 20, width)
    for first in range(0, count, step):
        k = min(step, count - first)
        slot = n // count
        start = (torch.arange(first, first + k, device=g.device) * slot + _randint(g, slot - width + 1, k))[:, None]
        if kind == "tandem":
            unit = 2 + _randint(g, 5, k, 1)
            span = unit * (10 + _randint(g, 41, k, 1))
            bases = torch.gather(_randint(g, 4, k, 6), 1, at[None, :] % unit)
            keep = at[None, :] < span
        else:
            bases = elements[_randint(g, 20, k)]
            bases = torch.where(_rand(g, k, width) < 0.10, (bases + 1 + _randint(g, 3, k, width)) & 3, bases)
            keep = torch.ones_like(bases, dtype=torch.bool)
        where = (start + at[None, :])[keep]
        codes[where] = bases[keep].to(torch.uint8)
    return codes


def _reference(n, repeats, seed):
    """Text of n bases, as codes 0..3 on the device."""
    g = _generator(n, repeats, seed)
    return _add_repeats(_markov(n, g), repeats, g)


_LETTERS = torch.tensor(list(b"ACGTN"), dtype=torch.uint8)


def _reads(case, codes, count, g):
    """(ASCII bytes, int64 offsets) of `count` reads on the device."""
    n, dev = codes.numel(), g.device
    length = (case["lo"] + _randint(g, case["hi"] - case["lo"] + 1, count)).clamp(max=n)
    offs = torch.zeros(count + 1, dtype=torch.int64, device=dev)
    torch.cumsum(length, 0, out=offs[1:])
    data = torch.empty(int(offs[-1]), dtype=torch.uint8, device=dev)
    letters = _LETTERS.to(dev)
    source = (_rand(g, count).double() * (n - length + 1)).long().clamp(max=n - 1)
    rate = case["rate_lo"] + (case["rate_hi"] - case["rate_lo"]) * _rand(g, count)
    unrelated = _rand(g, count) < case["random"]
    uncalled = _rand(g, count) < case["unknown"]
    step = max(1, (1 << 26) // case["hi"])
    for r0 in range(0, count, step):
        r1 = min(count, r0 + step)
        a, b = int(offs[r0]), int(offs[r1])
        owner = torch.repeat_interleave(torch.arange(r0, r1, device=dev), length[r0:r1])
        base = codes[torch.arange(a, b, device=dev) - offs[owner] + source[owner]].long()
        new = _randint(g, 4, b - a)
        changed = _rand(g, b - a) < rate[owner]
        base = torch.where(unrelated[owner], new, torch.where(changed, (base + 1 + new % 3) & 3, base))
        if case["unknown"]:
            base = torch.where(uncalled[owner] & (_rand(g, b - a) < 0.02), 4, base)
        data[a:b] = letters[base]
    return data, offs


def _ascii(codes):
    return _LETTERS.to(codes.device)[codes.long()].cpu().numpy()


_kept = {}  # what a program keeps between calls, of one case at a time: texts, indexes, a stream, a server


def _keep(case, what, make):
    """What `make` returns, made once for the resident references of a case."""
    owner = (case["n"], case["repeats"], case["entry"] == "serve")
    if _kept.get("owner") != owner:
        _kept.clear()
        _kept["owner"] = owner
    if what not in _kept:
        _kept[what] = make()
    return _kept[what]


def _texts(case, seed):
    """The codes of the case's references; those of resident ones do not change with the seed."""
    if case["entry"] == "build":
        return [_reference(case["n"], case["repeats"], seed + 1)]
    lengths = [case["n"], case["n"] // 16] if case["entry"] == "serve" else [case["n"]]
    return _keep(case, "texts", lambda: [_reference(n, case["repeats"], -1) for n in lengths])


def _batches(case, codes, seed):
    """(reference, ASCII, offsets) of the case's batch, or of each of its requests."""
    g = _generator(case["n"], case["reads"], case["lo"], case["hi"], seed)
    if case["entry"] != "serve":
        return [(0, *_reads(case, codes[0], case["reads"], g))]
    return [(i % 2, *_reads(case, codes[i % 2], size, g)) for i, size in enumerate(_request_sizes(case))]


def _request_sizes(case):
    """Request sizes of 1 to 100,000 reads, spread over their logarithm, large and small in turn."""
    sizes = [int(100_000 ** ((i + 0.5) / case["requests"])) for i in range(case["requests"])]
    return [s for i in range(5) for s in sizes[i::5]]


def prepare(case, seed):
    entry, state = case["entry"], {"case": case}
    codes = _texts(case, seed)
    if entry != "build":
        indexes = _keep(case, "indexes", lambda: [S.sa_build_device(_ascii(c)) for c in codes])
        state["index"] = indexes[0]
    batches = _batches(case, codes, seed)
    _, data, offs = batches[0]
    if entry == "build":
        state["text"] = _ascii(codes[0])
    if entry == "host":
        state |= {"data": data.cpu().numpy(), "offs": offs.cpu().numpy()}
    elif entry == "serve":
        state["server"] = _keep(case, "server", lambda: S.Server(indexes))
        state["requests"] = [(r, d.cpu().numpy(), o.cpu().numpy()) for r, d, o in batches]
    else:
        state |= {"data": data, "offs": offs,
                  "out": torch.zeros((offs.numel() - 1, 4), dtype=torch.int32, device=data.device)}
    if entry == "device":
        state["stream"], state["config"] = None, None
        if case["settings"] == "graph":
            state["stream"] = _keep(case, "stream", torch.cuda.Stream)
            state["config"] = S.cfg(state["index"], tile_levels=8, block=512, blocks_per_cu=3, group=1, max_words=5,
                                    defer=2, use_graph=1)
    if entry == "locate":
        S.match_batch_dev(state["index"], data, offs, state["out"])
        state["start"] = torch.zeros_like(offs)
        state["pos"] = torch.zeros(case["reads"] * case["cap"], dtype=torch.int32, device=data.device)
    if torch.cuda.is_available():
        torch.cuda.synchronize()
    return state


def run(state):
    entry = state["case"]["entry"]
    if entry == "device":
        S.match_batch_dev(state["index"], state["data"], state["offs"], state["out"], stream=state["stream"],
                          config=state["config"])
        return state["out"]
    if entry == "host":
        return S.match_batch(state["index"], state["data"], state["offs"])
    if entry == "locate":
        total = S.locate_dev(state["index"], state["out"], state["case"]["cap"], 0, state["start"], state["pos"])
        return {"starts": state["start"], "positions": state["pos"], "total": total}
    if entry == "build":
        index = S.sa_build_device(state["text"])
        S.match_batch_dev(index, state["data"], state["offs"], state["out"])
        torch.cuda.synchronize()  # the index may not go while a batch is on it
        return state["out"]
    waiting = [state["server"].submit(*r) for r in state["requests"]]
    for ticket, _ in waiting:
        status, _ = state["server"].poll(ticket, timeout_us=-1)
        if status != S.SA_OK:
            raise RuntimeError(f"request failed with {status}")
    return [out for _, out in waiting]


def work(case):
    """Each read's bases and offset read once and its 16-byte result written
    once; of the index, the matched text at two bits a base."""
    mean = (case["lo"] + case["hi"]) / 2
    count, more = case["reads"], 0
    if case["entry"] == "serve":
        count = sum(_request_sizes(case))
    elif case["entry"] == "locate":  # results in, offsets and (at least) a position each out
        return {"bytes": float(count * (16 + 8 + 2 * 4 * (1 - case["random"]))), "flops": 0.0}
    elif case["entry"] == "build":  # the text in, the suffix array out
        more = 5 * case["n"]
    return {"bytes": float(count * (mean * 1.25 + 8 + 16) + more), "flops": 0.0}


# ------------------------------------------------------------------ exact results

_PER_WORD = 20  # bases in a word, three bits each: 0 past the end, then A C G T, 7 for what matches nothing


def _words(symbols):
    """Per position, the next _PER_WORD symbols as one integer."""
    padded = torch.cat([symbols.long(), torch.zeros(_PER_WORD, dtype=torch.int64, device=symbols.device)])
    w = torch.zeros(symbols.numel(), dtype=torch.int64, device=symbols.device)
    for j in range(_PER_WORD):
        w = (w << 3) | padded[j:j + symbols.numel()]
    return w


def _suffix_array(symbols):
    """Suffixes in ascending order, by prefix doubling."""
    n, dev = symbols.numel(), symbols.device
    key, h = _words(symbols), _PER_WORD
    while True:
        key, order = torch.sort(key)
        new = torch.ones(n, dtype=torch.int64, device=dev)
        new[1:] = key[1:] != key[:-1]
        rank = torch.empty(n, dtype=torch.int64, device=dev)
        rank[order] = torch.cumsum(new, 0)
        if int(rank.max()) == n:
            return order
        after = torch.zeros(n, dtype=torch.int64, device=dev)
        after[:max(0, n - h)] = rank[h:]
        key, h = rank * (n + 1) + after, 2 * h


def _exact_hits(text_words, sa, symbols, offs):
    """(lo, hi, len, exact) of each read, by binary searches over whole reads."""
    n, dev = sa.numel(), sa.device
    length, start = offs[1:] - offs[:-1], offs[:-1]
    read_words = _words(symbols)
    most = -(-int(length.max()) // _PER_WORD) if length.numel() else 0

    def word(k, size, fill):
        """Word k of each read's first `size` symbols; those past them are `fill`."""
        at = (start + k * _PER_WORD).clamp(max=max(0, symbols.numel() - 1))
        mask = (1 << (3 * (_PER_WORD - (size - k * _PER_WORD).clamp(0, _PER_WORD)))) - 1
        return (read_words[at] & ~mask) | (mask if fill else 0)

    def suffix_word(p, k):
        at = p + k * _PER_WORD
        return torch.where(at < n, text_words[at.clamp(max=n - 1)], 0)

    def bound(size, fill):
        """First row whose suffix is not below the read's first `size` symbols with `fill` after them."""
        left, right = torch.zeros_like(size), torch.full_like(size, n)
        for _ in range(int(n).bit_length()):
            mid = (left + right) // 2
            p = sa[mid.clamp(max=n - 1)]
            below, open_ = torch.zeros_like(size, dtype=torch.bool), left < right
            undecided = open_.clone()
            for k in range(most):
                x, y = suffix_word(p, k), word(k, size, fill)
                below |= undecided & (x < y)
                undecided &= (x == y)
            left, right = torch.where(open_ & below, mid + 1, left), torch.where(open_ & ~below, mid, right)
        return left

    def shared(row):
        """Symbols that each read shares with the suffix at its row."""
        p = sa[row.clamp(0, n - 1)]
        found, going = torch.zeros_like(length), (row >= 0) & (row < n)
        for j in range(int(length.max()) if length.numel() else 0):
            at = p + j
            t = torch.where(at < n, text_words[at.clamp(max=n - 1)] >> (3 * (_PER_WORD - 1)), 0)
            going &= (j < length) & (symbols[(start + j).clamp(max=max(0, symbols.numel() - 1))] == t)
            found += going
        return found

    row = bound(length, 0)
    size = torch.maximum(shared(row - 1), shared(row))
    return torch.stack([bound(size, 0), bound(size, 1), size, (size == length).long()], 1)


def exact(case, seed):
    """Results by plain torch in 64 bits; None for the chromosome-sized batch, where this takes too long."""
    if case["n"] > 32_000_000 or case["reads"] > 1_000_000:
        return None
    codes = _texts(case, seed)
    batches = _batches(case, codes, seed)
    texts = []
    for c in codes:
        symbols = c.long() + 1
        texts.append((_words(symbols), _suffix_array(symbols)))
    table = torch.full((256,), 7, dtype=torch.int64, device=codes[0].device)
    table[torch.tensor(list(b"ACGT"), device=table.device)] = torch.arange(1, 5, device=table.device)
    hits = [_exact_hits(*texts[ref], table[data.long()], offs) for ref, data, offs in batches]
    if case["entry"] == "serve":
        return hits
    if case["entry"] != "locate":
        return hits[0]
    h = hits[0]
    rows = (h[:, 1] - h[:, 0]).clamp(max=case["cap"]) * h[:, 3]
    starts = torch.zeros(rows.numel() + 1, dtype=torch.int64, device=h.device)
    torch.cumsum(rows, 0, out=starts[1:])
    total = int(starts[-1])
    owner = torch.repeat_interleave(torch.arange(rows.numel(), device=h.device), rows)
    pos = torch.zeros(case["reads"] * case["cap"], dtype=torch.int64, device=h.device)
    pos[:total] = texts[0][1][h[owner, 0] + torch.arange(total, device=h.device) - starts[owner]]
    return {"starts": starts, "positions": pos, "total": total}
