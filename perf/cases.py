"""Performance cases of the RotorMap path on one MI355X.

Each case is a call, or a short sequence of calls, that a program using the
package makes: building an index, encoding read heads, mapping reads
(product, top-k, FP32 rescore), mapping on a coarse index with refinement, one
batched step over reads of uneven length, the learned encoding's index,
mapping and training, the per-window thresholds and the threshold regime.

listed() are fixed cases, draw() makes one more of the same ranges, prepare()
makes on the GPU what a program holds before the call, run() is one pass, work()
the bytes and operations that a pass cannot do without, and exact() the same
outputs from 64-bit torch arithmetic.
"""
import math

import numpy as np
import torch

from paper_2603_22245_amd import learned, mapper

M = 32                      # factors of the letter encoding
CONTEXT = 9                 # letters of a token of the learned encoding
N_IN, N_HID, N_OUT = 32, 64, 128
TAU = 0.05                  # temperature of the ranking loss
BETA1, BETA2, EPS = 0.9, 0.999, 1e-8
ITEM = {"fp32": 4, "fp16": 2, "fp8": 1}

# name -> (letters per token, factors, classes, seeded map, schedule)
ENCODINGS = {
    "letters": (1, M, 4, False, "default"),
    "s2": (2, 8, 16, False, "default"),
    "s8c16": (8, 8, 16, True, "finetuned"),
    "s8c256": (8, 4, 256, True, "finetuned"),
}


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # a plasmid-sized reference and a few hundred reads in FP32: the smallest whole
        # call, where launches and latency count
        dict(name="map_plain", kind="map", encoding="letters", precision="fp32", ref_len=20_000,
             n_reads=200, read_len=150, error=0.02, k=8, k_fetch=16),
        # a handful of reads looked up in a bacterial-genome index: an interactive query,
        # which streams the whole index for little arithmetic
        dict(name="map_query", kind="map", encoding="letters", precision="fp16",
             ref_len=10_000_000, n_reads=8, read_len=150, error=0.02, k=8, k_fetch=16),
        # a sequencing run's reads against the same index: the largest call
        dict(name="map_precision", kind="map", encoding="letters", precision="fp16",
             ref_len=10_000_000, n_reads=100_000, read_len=150, error=0.02, k=8, k_fetch=16),
        # building that index: every window of a bacterial genome
        dict(name="index_letters", kind="index", encoding="letters", precision="fp16",
             ref_len=10_000_000, window=150, stride=1),
        # encoding the read heads of a run, the layer before the product
        dict(name="heads", kind="heads", encoding="letters", precision="fp16", n_reads=100_000,
             read_len=150),
        # reads of uneven length (100 bp to 10 kbp): seven strided indexes, one grouped
        # product, rescore per bucket
        dict(name="batch_uneven", kind="batch", precision="fp8", ref_len=16_000_000, n_reads=5_000,
             median=2000, k=8, k_fetch=16),
        # 8-mer tokens in 256 classes (1,024 components) on a coarse index, refined letter
        # by letter around the candidates
        dict(name="coarse_tokens", kind="coarse", encoding="s8c256", precision="fp8",
             ref_len=10_000_000, n_reads=20_000, read_len=150, error=0.02, stride=16, radius=15,
             k=8, k_fetch=32),
        # the learned encoding: offsets of the reference's tokens, then its index
        dict(name="index_learned", kind="index_learned", precision="fp16", ref_len=10_000_000,
             window=150, stride=1),
        # mapping reads with the learned encoding on a viral-to-small-bacterial reference
        dict(name="map_learned", kind="map_learned", precision="fp16", ref_len=1_000_000,
             n_reads=20_000, read_len=150, error=0.02, k=8, k_fetch=16),
        # training the offsets: edit-distance labels of new pairs, then Adam steps
        dict(name="train", kind="train", batch=1024, steps=8, length=150, max_edits=30),
        # cutting thresholds of every window at a target mutation rate
        dict(name="thresholds", kind="thresholds", precision="fp16", ref_len=1_000_000, window=150,
             stride=1, error=0.02, copies=16),
        # every location that passes its window's threshold, for a run's reads
        dict(name="regime", kind="regime", precision="fp16", ref_len=2_000_000, n_reads=20_000,
             read_len=150, error=0.02, floor=0.1),
    ]


def _spread(rng, lo, hi):
    """An integer spread over the logarithm of lo..hi."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["map", "map", "index", "heads", "batch", "coarse", "index_learned",
                       "map_learned", "train", "thresholds", "regime"])
    precision = rng.choice(["fp16", "fp16", "fp8", "fp32"])
    read_len = rng.choice([100, 150, 150, rng.randint(75, 300)])
    error = round(rng.uniform(0.005, 0.05), 4)
    k = rng.choice([1, 4, 8, 8, 10, 16])
    k_fetch = min(32, 2 * max(k, rng.choice([4, 8, 8])))
    if kind == "map":
        encoding = rng.choice(["letters", "letters", "letters", "s2", "s8c16"])
        ref_len = _spread(rng, 20_000, 10_000_000)
        most = 4e10 if precision == "fp32" else 5e11
        n_reads = _spread(rng, 1, min(100_000, most / ref_len))
        return dict(kind=kind, encoding=encoding, precision=precision, ref_len=ref_len,
                    n_reads=n_reads, read_len=read_len, error=error, k=k, k_fetch=k_fetch)
    if kind == "index":
        window = rng.choice([100, 150, 150, 200, 800, 1600, rng.randint(75, 3000)])
        stride = rng.choice([1, 1, max(1, window // 100), rng.randint(1, 16)])
        n_win = _spread(rng, 50_000, 10_000_000 if precision != "fp32" else 4_000_000)
        return dict(kind=kind, encoding=rng.choice(["letters", "letters", "s2", "s8c16"]),
                    precision=precision, ref_len=min(64_000_000, n_win * stride + window),
                    window=window, stride=stride)
    if kind == "heads":
        read_len = rng.choice([100, 150, 150, rng.randint(75, 1600)])
        return dict(kind=kind, encoding=rng.choice(["letters", "letters", "letters", "s2"]),
                    precision=precision, n_reads=_spread(rng, 1, 100_000 * 150 // max(150, read_len)),
                    read_len=read_len)
    if kind == "batch":
        return dict(kind=kind, precision=rng.choice(["fp16", "fp8"]),
                    ref_len=_spread(rng, 200_000, 16_000_000), n_reads=_spread(rng, 100, 5_000),
                    median=rng.choice([500, 1000, 2000]), k=8, k_fetch=16)
    if kind == "coarse":
        encoding = rng.choice(["letters", "s2", "s8c256", "s8c256"])
        if encoding == "s8c256":
            precision, stride = rng.choice(["fp16", "fp8"]), rng.choice([4, 8, 16])
        else:
            precision, stride = rng.choice(["fp16", "fp8"]), rng.choice([2, 3, 4])
        ref_len = _spread(rng, 100_000, 5_000_000 if precision == "fp16" else 10_000_000)
        n_reads = _spread(rng, 50, min(20_000, 1.2e10 * stride / ref_len))
        return dict(kind=kind, encoding=encoding, precision=precision, ref_len=ref_len,
                    n_reads=n_reads, read_len=read_len, error=error, stride=stride,
                    radius=max(stride - 1, 1), k=8, k_fetch=32)
    if kind == "index_learned":
        return dict(kind=kind, precision=precision,
                    ref_len=_spread(rng, 50_000, 10_000_000 if precision != "fp32" else 4_000_000),
                    window=rng.choice([100, 150, 150, rng.randint(75, 300)]),
                    stride=rng.choice([1, 1, 1, 2, 5]))
    if kind == "map_learned":
        return dict(kind=kind, precision=rng.choice(["fp16", "fp8"]),
                    ref_len=_spread(rng, 20_000, 1_000_000), n_reads=_spread(rng, 50, 20_000),
                    read_len=read_len, error=error, k=k, k_fetch=k_fetch)
    if kind == "train":
        return dict(kind=kind, batch=rng.choice([1024, 512, rng.randint(64, 1024)]),
                    steps=rng.randint(1, 8), length=rng.randint(100, 200),
                    max_edits=rng.randint(10, 40))
    if kind == "thresholds":
        window = rng.choice([100, 150, 150, rng.randint(75, 300)])
        return dict(kind=kind, precision=precision, ref_len=_spread(rng, 20_000, 1_000_000),
                    window=window, stride=rng.choice([1, 1, 2, 7]), error=error,
                    copies=rng.choice([8, 16, 16, rng.randint(4, 24)]))
    return dict(kind=kind, precision=rng.choice(["fp16", "fp8"]),
                ref_len=_spread(rng, 20_000, 2_000_000), n_reads=_spread(rng, 50, 20_000),
                read_len=read_len, error=error, floor=round(rng.uniform(0.1, 0.3), 3))


# ---------------------------------------------------------------- inputs

def _generator(seed, role):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * int(seed) + role)
    return g


def _reference(n, seed, gc=0.41, repeat_frac=0.05):
    """Letters of the stated GC with families of diverged repeats (unit 2 to 300 letters,
    2 to 50 copies, half of the families in tandem) over a part of it."""
    g = _generator(seed, 0)
    u = torch.rand(n, generator=g, device="cuda")
    other = torch.rand(n, generator=g, device="cuda") < 0.5
    is_gc = u < gc
    ref = torch.where(is_gc, torch.where(other, 1, 2), torch.where(other, 0, 3)).to(torch.uint8)
    rng = np.random.default_rng([int(seed), 7])
    covered, dst, val = 0, [], []
    family = 0
    while covered < repeat_frac * n:
        unit = int(round(math.exp(rng.uniform(math.log(2), math.log(300)))))
        copies = int(rng.integers(2, 51))
        if unit * copies > n // 4:
            break
        letters = np.tile(rng.integers(0, 4, unit), copies)
        changed = rng.random(letters.size) < 0.10
        letters[changed] = (letters[changed] + rng.integers(1, 4, int(changed.sum()))) % 4
        if family % 2 == 0:
            at = rng.integers(0, n - unit * copies) + np.arange(unit * copies)
        else:
            at = (rng.integers(0, n - unit, copies)[:, None] + np.arange(unit)).ravel()
        dst.append(at)
        val.append(letters)
        covered += unit * copies
        family += 1
    if dst:
        at, first = np.unique(np.concatenate(dst), return_index=True)
        letters = np.concatenate(val)[first].astype(np.uint8)
        ref[torch.from_numpy(at).cuda()] = torch.from_numpy(letters).cuda()
    return ref


def _reads(ref, lengths, error, seed, split=(1 / 3, 1 / 3, 1 / 3)):
    """Reads of the given lengths (a host array) from uniform starts: each step is a
    substitution, an insertion, a deletion (with `error` split between them) or a match.
    Returns letters and offsets as host arrays; error: a number or one per read."""
    g = _generator(seed, 1)
    n, total = len(lengths), int(ref.numel())
    offsets = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(lengths, out=offsets[1:])
    seq = torch.randint(0, 4, (int(offsets[-1]),), generator=g, device="cuda", dtype=torch.uint8)
    rate = torch.as_tensor(np.broadcast_to(np.asarray(error, dtype=np.float64), (n,)).copy(),
                           device="cuda")
    start = (torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
             * max(1, total - int(np.max(lengths)))).long()
    d_len = torch.from_numpy(np.asarray(lengths, dtype=np.int64)).cuda()
    d_off = torch.from_numpy(offsets).cuda()
    order = np.argsort(-lengths, kind="stable")
    done = 0
    while done < n:
        steps = int(1.3 * int(lengths[order[done]])) + 32
        ids = torch.from_numpy(order[done: done + max(1, (1 << 25) // steps)].copy()).cuda()
        done += ids.numel()
        shape = (ids.numel(), steps)
        u = torch.rand(shape, generator=g, device="cuda")
        e = rate[ids][:, None].float()
        sub = u < e * split[0]
        ins = (u >= e * split[0]) & (u < e * (split[0] + split[1]))
        dele = (u >= e * (split[0] + split[1])) & (u < e)
        shift = torch.randint(1, 4, shape, generator=g, device="cuda", dtype=torch.uint8)
        out = torch.cumsum((~dele).to(torch.int32), 1) - 1
        used = (~ins).to(torch.int32)
        pos = start[ids][:, None] + (torch.cumsum(used, 1) - used)
        letter = ref[pos.clamp_(max=total - 1)]
        letter = torch.where(sub, (letter + shift) % 4, letter)
        # an inserted letter is the random one that is there
        keep = ~dele & ~ins & (out < d_len[ids][:, None])
        seq[(d_off[ids][:, None] + out)[keep]] = letter[keep]
    return seq.cpu().numpy(), offsets


def _token_map(s, n_class):
    """A fixed balanced random table of 4^s s-mers to n_class classes."""
    codes = np.arange(4 ** s) % n_class
    return np.random.default_rng(17).permutation(codes).astype(np.uint8)


def _network(seed):
    """Parameters of a trained-like offset network (W1, b1, W2, b2)."""
    rng = np.random.default_rng([int(seed), 3])
    return np.concatenate([rng.uniform(-1, 1, N_HID * N_IN) / math.sqrt(N_IN),
                           rng.uniform(-1, 1, N_HID) / math.sqrt(N_IN),
                           rng.normal(0, 0.08, N_OUT * N_HID),
                           rng.normal(0, 0.05, N_OUT)]).astype(np.float32)


def _index_args(encoding):
    s, m, n_class, mapped, schedule = ENCODINGS[encoding]
    if encoding == "letters":
        return {}
    return dict(mer_len=s, n_freq=m, n_class=n_class, schedule=schedule,
                token_map=_token_map(s, n_class) if mapped else None)


def _pairs(case, seed):
    """Random strings and companions after 0..max_edits edits each (host arrays)."""
    n, length, most = case["batch"] * case["steps"], case["length"], case["max_edits"]
    g = _generator(seed, 2)
    a = torch.randint(0, 4, (n, length), generator=g, device="cuda", dtype=torch.uint8)
    edits = torch.randint(0, most + 1, (n,), generator=g, device="cuda")
    width = length + most
    b = torch.zeros((n, width), dtype=torch.uint8, device="cuda")
    b[:, :length] = a
    size = torch.full((n,), length, device="cuda", dtype=torch.int64)
    at = torch.arange(width, device="cuda")[None, :]
    for e in range(most):
        kind = torch.randint(0, 3, (n,), generator=g, device="cuda")
        where = (torch.rand(n, generator=g, device="cuda") * size).long().clamp_(max=width - 1)
        new = torch.randint(0, 4, (n,), generator=g, device="cuda", dtype=torch.uint8)
        live = edits > e
        # an insertion reads from one letter before past its place, a deletion from one after
        shift = torch.where(kind == 1, -1, torch.where(kind == 2, 1, 0))
        src = at + torch.where(at > where[:, None] - (kind == 2)[:, None].long(),
                               shift[:, None], 0)
        moved = torch.gather(b, 1, src.clamp_(0, width - 1))
        put = (at == where[:, None]) & (kind != 2)[:, None]
        moved = torch.where(put, new[:, None], moved)
        b = torch.where(live[:, None], moved, b)
        size = torch.where(live, size + (kind == 1).long() - (kind == 2).long(), size)
    keep = at < size[:, None]
    a_off = np.arange(n + 1, dtype=np.int64) * length
    b_off = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(size.cpu().numpy(), out=b_off[1:])
    return a.reshape(-1).cpu().numpy(), a_off, b[keep].cpu().numpy(), b_off


def _lengths(case, seed):
    """Log-normal read lengths: the same ones for every seed, in another order."""
    x = np.exp(np.random.default_rng(5).normal(math.log(case["median"]), 0.8, case["n_reads"]))
    x = np.clip(np.rint(x), 100, min(10_000, case["ref_len"] // 4)).astype(np.int64)
    return np.random.default_rng([int(seed), 5]).permutation(x)


def _mapping_inputs(case, seed):
    ref = _reference(case["ref_len"], seed)
    seq, off = _reads(ref, np.full(case["n_reads"], case["read_len"], dtype=np.int64),
                      case["error"], seed)
    return ref, seq, off


def _batch_inputs(case, seed):
    ref = _reference(case["ref_len"], seed, 0.45, 0.08)
    lengths = _lengths(case, seed)
    error = np.random.default_rng([int(seed), 6]).uniform(0.05, 0.10, len(lengths))
    seq, off = _reads(ref, lengths, error, seed, (0.2, 0.4, 0.4))
    return ref, seq, off


def _adam_state(seed):
    """Moments of a run under way (values, squares) and its step count."""
    rng = np.random.default_rng([int(seed), 4])
    n = learned.N_PARAMS
    return (rng.normal(0, 2e-4, n).astype(np.float32),
            np.square(1e-3 * rng.uniform(0.5, 2.0, n)).astype(np.float32), 200)


# ---------------------------------------------------------------- what a program holds, and a pass

def prepare(case, seed):
    kind, case = case["kind"], dict(case)
    if kind in ("map", "map_learned", "coarse", "regime"):
        ref, seq, off = _mapping_inputs(case, seed)
        args = _index_args(case.get("encoding", "letters"))
        index = mapper.build_index(ref, window_len=case["read_len"], stride=case.get("stride", 1),
                                   precision=case["precision"],
                                   learned=_network(seed) if kind == "map_learned" else None, **args)
        reads = mapper.upload_reads(index, seq, off)
        state = dict(case=case, index=index, reads=reads)
        if kind == "regime":
            state["thr"] = mapper.window_thresholds(index, case["error"], seed=int(seed) + 1)
            mapper.encode_reads(index, reads)
            return state
        state["bufs"] = mapper.map_buffers(index, case["n_reads"], case["k"], case["k_fetch"])
        if kind == "coarse":  # the refinement's workspace, kept between calls
            mapper.encode_reads(index, reads)
            state["bufs"].cand_idx.fill_(-1)
            state["ws"] = mapper.refine(index, reads, state["bufs"], case["radius"])
        return state
    if kind == "index":
        args = _index_args(case["encoding"])
        if args.get("token_map") is not None:
            args["token_map"] = torch.from_numpy(args["token_map"]).cuda()
        return dict(case=case, ref=_reference(case["ref_len"], seed), args=args)
    if kind == "index_learned":
        return dict(case=case, ref=_reference(case["ref_len"], seed),
                    learned=torch.from_numpy(_network(seed)).cuda())
    if kind == "heads":
        ref = _reference(max(100_000, 4 * case["read_len"]), seed)
        index = mapper.build_index(ref, window_len=case["read_len"], precision=case["precision"],
                                   **_index_args(case["encoding"]))
        seq, off = _reads(ref, np.full(case["n_reads"], case["read_len"], dtype=np.int64), 0.02, seed)
        return dict(case=case, index=index, reads=mapper.upload_reads(index, seq, off))
    if kind == "batch":
        ref, seq, off = _batch_inputs(case, seed)
        return dict(case=case, mapper=mapper.BatchMapper(ref.cpu().numpy(), seq, off, case["k"],
                                                         case["k_fetch"], case["precision"]))
    if kind == "train":
        a, a_off, b, b_off = _pairs(case, seed)
        trainer = learned.Trainer(_network(seed), nominal_len=case["length"], batch=case["batch"])
        m, v, step = _adam_state(seed)
        n = learned.N_PARAMS
        trainer.state[n:2 * n] = torch.from_numpy(m).cuda()
        trainer.state[2 * n:3 * n] = torch.from_numpy(v).cuda()
        trainer.state[3 * n] = step
        return dict(case=case, trainer=trainer, pairs=learned.upload_pairs(a, a_off, b, b_off))
    if kind == "thresholds":
        index = mapper.build_index(_reference(case["ref_len"], seed), window_len=case["window"],
                                   stride=case["stride"], precision=case["precision"])
        return dict(case=case, index=index, seed=int(seed) + 1)
    raise ValueError(f"unknown kind {kind!r}")


def _rows(values, precision):
    """Stored rows as numbers (FP8 codes as the e4m3 values they stand for)."""
    return values.view(torch.float8_e4m3fn) if precision == "fp8" else values


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("map", "map_learned"):
        mapper.map_reads(state["index"], state["reads"], state["bufs"])
        return dict(idx=state["bufs"].top_idx, score=state["bufs"].top_score)
    if kind == "coarse":
        mapper.map_reads_coarse(state["index"], state["reads"], state["bufs"], case["radius"],
                                state["ws"])
        return dict(idx=state["bufs"].top_idx, score=state["bufs"].top_score)
    if kind in ("index", "index_learned"):
        more = state["args"] if kind == "index" else dict(learned=state["learned"])
        index = mapper.build_index(state["ref"], window_len=case["window"], stride=case["stride"],
                                   precision=case["precision"], **more)
        return dict(rows=_rows(index.embeddings(), case["precision"]), norm2=index.norms2())
    if kind == "heads":
        index, reads = state["index"], state["reads"]
        mapper.encode_reads(index, reads)
        rows = reads.emb if case["precision"] == "fp8" else reads.emb.view(
            torch.float16 if case["precision"] == "fp16" else torch.float32)
        return dict(rows=_rows(rows, case["precision"]).view(case["n_reads"], 2, index.real_dim))
    if kind == "batch":
        bm = state["mapper"]
        bm.rebuild_indexes()
        bm.run()
        return dict(idx=[b.bufs.top_idx for b in bm.buckets],
                    score=[b.bufs.top_score for b in bm.buckets])
    if kind == "train":
        trainer, pairs = state["trainer"], state["pairs"]
        pairs.ld = learned.levenshtein(pairs)
        loss = trainer.epoch(pairs)
        n = learned.N_PARAMS
        return dict(ld=pairs.ld, loss=loss, params=trainer.params, m=trainer.state[n:2 * n],
                    v=trainer.state[2 * n:3 * n])
    if kind == "thresholds":
        return mapper.window_thresholds(state["index"], case["error"], case["copies"],
                                        seed=state["seed"])
    if kind == "regime":
        h = mapper.score_threshold(state["index"], state["reads"], state["thr"], case["floor"])
        return dict(off=h.hit_off, found=h.n_found, idx=h.hit_idx, score=h.hit_score)
    raise ValueError(f"unknown kind {kind!r}")


# ---------------------------------------------------------------- the least work of a pass

def _row_reals(case):
    """Reals that a stored row needs: letters with integer factors have 3 independent
    components per factor, of which the stored precisions other than FP16 keep 4."""
    if case["kind"] in ("index_learned", "map_learned"):
        return 256
    if case.get("encoding", "letters") == "letters":
        return 192 if case["precision"] == "fp16" else 256
    _, m, n_class, _, _ = ENCODINGS[case["encoding"]]
    return 2 * m * n_class


def work(case):
    kind = case["kind"]
    if kind in ("map", "map_learned", "coarse", "regime"):
        stride, N, R = case.get("stride", 1), case["read_len"], case["n_reads"]
        W, D = (case["ref_len"] - N) // stride + 1, _row_reals(case)
        flops = 4 * D * R * W
        moved = W * D * ITEM[case["precision"]] + R * N
        if kind == "regime":
            return dict(bytes=moved + 4 * W + 16 * R, flops=flops)
        per = case["k_fetch"] * (2 * case["radius"] + 1) if kind == "coarse" else case["k_fetch"]
        # each rescored window: its letters' phases summed, one inner product
        return dict(bytes=moved + 8 * R * case["k"], flops=flops + 2 * D * R * per)
    if kind in ("index", "index_learned"):
        W = (case["ref_len"] - case["window"]) // case["stride"] + 1
        # a slide: a term out, a term in, a turn and the norm per component
        flops = W * _row_reals(case) * 6
        if kind == "index_learned":
            flops += (case["ref_len"] - 8) * 2 * (8 * N_HID + N_HID * M)
        return dict(bytes=W * (_row_reals(case) * ITEM[case["precision"]] + 8) + case["ref_len"],
                    flops=flops)
    if kind == "heads":
        D = _row_reals(case)
        return dict(bytes=case["n_reads"] * (case["read_len"] + 2 * D * ITEM[case["precision"]]),
                    flops=case["n_reads"] * case["read_len"] * 2 * M)
    if kind == "batch":
        lengths = _lengths(case, 0)
        size, flops, moved = np.searchsorted(mapper.BUCKETS, lengths, side="right") - 1, 0, 0
        D = 192 if case["precision"] == "fp16" else 256
        for b, N in enumerate(mapper.BUCKETS):
            R = int((size == b).sum())
            W = (case["ref_len"] - N) // max(1, N // 100) + 1
            if R and W > 0:
                flops += 4 * D * R * W + W * D * 6
                moved += 2 * W * D * ITEM[case["precision"]] + R * (N + 8 * case["k"])
        return dict(bytes=moved, flops=flops)
    if kind == "train":
        strings = 2 * case["batch"] * case["steps"]
        tokens = strings * (case["length"] - CONTEXT + 1)
        # forward and backward of the network; the one-hot layer is 8 additions per unit,
        # and only the middle letter's 32 outputs are used
        flops = tokens * 2 * 3 * (8 * N_HID + N_HID * M) + tokens * 8 * M
        return dict(bytes=strings * case["length"] + case["steps"] * 24 * learned.N_PARAMS,
                    flops=flops)
    W = (case["ref_len"] - case["window"]) // case["stride"] + 1
    # per copy: a draw per letter (ten rounds of two products and four exclusive ors), the
    # letters' phases summed (2 reals per factor), one inner product
    return dict(bytes=case["ref_len"] + 4 * W,
                flops=W * case["copies"] * (case["window"] * (100 + 2 * M) + 1024))


# ---------------------------------------------------------------- 64-bit values

def _factors(m, schedule):
    f = torch.arange(1, m + 1, dtype=torch.float64, device="cuda")
    return f if schedule == "default" else 2 * (f - 1) / max(1, m - 1) + 1


def _turn(f, p, N):
    """omega^(f p) for positions p."""
    angle = torch.remainder(f[None, :] * p[:, None].double(), N) * (2 * math.pi / N)
    return torch.polar(torch.ones_like(angle), angle)


def _classes(seq, s, table):
    """Class of the s-mer at every location."""
    n = seq.shape[-1] - s + 1
    code = torch.zeros(seq.shape[:-1] + (n,), dtype=torch.int64, device="cuda")
    for i in range(s):
        code = code * 4 + seq[..., i: i + n].long()
    return code if table is None else table[code].long()


def _flanks(seq):
    """Middle letter of every 9-mer and its flanks' places in the one-hot input."""
    n = seq.shape[-1] - CONTEXT + 1
    at = [0, 1, 2, 3, 5, 6, 7, 8]
    x = torch.stack([4 * i + seq[..., o: o + n].long() for i, o in enumerate(at)], -1)
    return seq[..., 4: 4 + n].long(), x


def _unpack(p):
    a, b, c = N_HID * N_IN, N_HID * N_IN + N_HID, N_HID * N_IN + N_HID + N_OUT * N_HID
    return (p[:a].view(N_HID, N_IN), p[a:b], p[b:c].view(N_OUT, N_HID), p[c:])


def _offsets(params, seq):
    """Phase offsets of every token of a text: weights and hidden values are bfloat16."""
    W1, b1, W2, b2 = _unpack(torch.from_numpy(params).cuda())
    W1, W2 = W1.bfloat16().double(), W2.bfloat16().double()
    out = []
    for i in range(0, seq.numel() - CONTEXT + 1, 1 << 18):
        mid, x = _flanks(seq[i: i + (1 << 18) + CONTEXT - 1])
        h = torch.relu(W1.t()[x].sum(1) + b1.double()).float().bfloat16().double()
        o = (h @ W2.t() + b2.double()).view(-1, 4, M)
        out.append(torch.gather(o, 1, mid[:, None, None].expand(-1, 1, M))[:, 0])
    return torch.cat(out)


class _Encoder:
    """Windows and read heads of one encoding in complex128, [n, factors, classes]."""

    def __init__(self, encoding, N, params=None):
        self.s, self.m, self.C, mapped, schedule = ENCODINGS[encoding]
        self.N, self.params = N, params
        if params is not None:
            self.s = CONTEXT
        self.T = N - self.s + 1
        self.f = _factors(self.m, schedule)
        self.table = torch.from_numpy(_token_map(self.s, self.C)).cuda() if mapped else None
        # positions per block of the prefix sums, and windows per block
        self.block = max(1 << 14, (1 << 25) // (self.m * self.C))

    def tokens(self, seq):
        if self.params is None:
            return _classes(seq, self.s, self.table), None
        return seq[4: seq.numel() - 4].long(), _offsets(self.params, seq)

    def windows(self, ref, stride=1):
        """Blocks (first window, vectors) over every window of ref."""
        cls, delta = self.tokens(ref)
        W = (ref.numel() - self.N) // stride + 1
        step = max(1, self.block // stride)
        for a in range(0, W, step):
            b = min(W, a + step)
            lo, hi = a * stride, (b - 1) * stride + self.T
            local = torch.arange(hi - lo, device="cuda")
            g = _turn(self.f, local, self.N)
            if delta is not None:
                g = g * torch.polar(torch.ones_like(delta[lo:hi]), delta[lo:hi])
            sums = torch.zeros((hi - lo + 1, self.C, self.m), dtype=torch.complex128, device="cuda")
            sums[local + 1, cls[lo:hi]] = g
            sums = torch.cumsum(sums, 0)
            at = torch.arange(0, (b - a - 1) * stride + 1, stride, device="cuda")
            v = (sums[at + self.T] - sums[at]) * _turn(self.f, at, self.N).conj()[:, None, :]
            yield a, v.transpose(1, 2)

    def heads(self, seq, off):
        """Vectors of the reads' first N letters (reads shorter than N do not occur)."""
        seq, off = torch.from_numpy(seq).cuda(), torch.from_numpy(off).cuda()
        cls, delta = self.tokens(seq)
        out, p = [], torch.arange(self.T, device="cuda")
        turn = _turn(self.f, p, self.N)
        rows = max(1, (1 << 24) // (self.T * self.m))
        for a in range(0, off.numel() - 1, rows):
            at = off[a: min(off.numel() - 1, a + rows), None] + p
            g = turn[None].expand(at.shape[0], -1, -1)
            if delta is not None:
                g = g * torch.polar(torch.ones_like(delta[at]), delta[at])
            v = torch.zeros((at.shape[0] * self.C, 2 * self.m), dtype=torch.float64, device="cuda")
            row = torch.arange(at.shape[0], device="cuda")[:, None] * self.C + cls[at]
            v.index_add_(0, row.reshape(-1), torch.view_as_real(g).reshape(-1, 2 * self.m))
            out.append(torch.view_as_complex(v.view(-1, self.C, self.m, 2)).transpose(1, 2))
        return torch.cat(out)

    def unit(self, v):
        """Normalised rows [n, factors * classes] and squared norms."""
        flat = v.reshape(v.shape[0], -1)
        norm2 = torch.view_as_real(flat).square().sum((1, 2))
        scale = torch.where(norm2 < 1e-4 * self.N, 0.0, norm2.clamp(min=1e-30).rsqrt())
        return flat * scale[:, None], norm2


def _reduced(v):
    """Coordinates of [n, factors * 4] rows on the letter weights that sum to zero."""
    h = torch.tensor([[1, 1, -1, -1], [1, -1, 1, -1], [1, -1, -1, 1]], device="cuda",
                     dtype=torch.float64) / 2
    return (v.view(v.shape[0], -1, 4) @ h.t().to(torch.complex128)).reshape(v.shape[0], -1)


def _reals(v, precision, reduced):
    v = torch.view_as_real(_reduced(v) if reduced else v.contiguous()).reshape(v.shape[0], -1)
    return v * 256 if precision == "fp8" else v


def _fidelities(heads, rows):
    x, c = torch.view_as_real(heads).flatten(1), torch.view_as_real(rows.contiguous()).flatten(1)
    y = torch.view_as_real(1j * heads).flatten(1)
    return (x @ c.t()).square_() + (y @ c.t()).square_()


def _best(enc, ref, heads, k, stride=1):
    """The k best fidelities of every head over all windows, and their ids."""
    score = torch.full((heads.shape[0], k), -1.0, dtype=torch.float64, device="cuda")
    ids = torch.full((heads.shape[0], k), -1, dtype=torch.int64, device="cuda")
    for a, v in enc.windows(ref, stride):
        rows, _ = enc.unit(v)
        part = max(1, (1 << 27) // rows.shape[0])
        for r in range(0, heads.shape[0], part):
            F = _fidelities(heads[r: r + part], rows)
            s, i = torch.topk(F, min(k, F.shape[1]), dim=1)
            s, i = torch.cat([score[r: r + part], s], 1), torch.cat([ids[r: r + part], i + a], 1)
            s, at = torch.topk(s, k, dim=1)
            score[r: r + part], ids[r: r + part] = s, torch.gather(i, 1, at)
    return score, ids


def _exact_map(case, seed):
    if case["n_reads"] * case["ref_len"] > 5e10:
        return None
    ref, seq, off = _mapping_inputs(case, seed)
    learned_ = _network(seed) if case["kind"] == "map_learned" else None
    enc = _Encoder(case.get("encoding", "letters"), case["read_len"], learned_)
    heads, _ = enc.unit(enc.heads(seq, off))
    return dict(idx=None, score=_best(enc, ref, heads, case["k"])[0].clamp(min=0))


def _exact_batch(case, seed):
    ref, seq, off = _batch_inputs(case, seed)
    size = np.searchsorted(mapper.BUCKETS, np.diff(off), side="right") - 1
    score = []
    for b, N in enumerate(mapper.BUCKETS):
        ids = np.nonzero(size == b)[0]
        if not ids.size:
            continue
        enc = _Encoder("letters", N)
        at = (off[ids][:, None] + np.arange(N)).ravel()
        heads, _ = enc.unit(enc.heads(seq[at], np.arange(ids.size + 1, dtype=np.int64) * N))
        score.append(_best(enc, ref, heads, case["k"], max(1, N // 100))[0].clamp(min=0))
    return dict(idx=[None] * len(score), score=score)


def _exact_coarse(case, seed):
    if case["n_reads"] * (case["ref_len"] // case["stride"]) > 2e10:
        return None
    ref, seq, off = _mapping_inputs(case, seed)
    N, radius, stride = case["read_len"], case["radius"], case["stride"]
    enc = _Encoder(case["encoding"], N)
    heads, _ = enc.unit(enc.heads(seq, off))
    _, ids = _best(enc, ref, heads, case["k_fetch"], stride)
    starts = ref.numel() - N + 1
    norm2 = torch.cat([enc.unit(v)[1] for _, v in enc.windows(ref)])
    near = torch.arange(-radius, radius + 1, device="cuda")
    cls, _ = enc.tokens(ref)
    p = torch.arange(enc.T, device="cuda")
    turn = _turn(enc.f, p, N)
    x = heads.view(-1, enc.m, enc.C).conj().transpose(1, 2).contiguous()  # [R, C, m]
    score = []
    pool = ids.shape[1] * near.numel()
    rows = max(1, (1 << 25) // (pool * enc.T))
    for r in range(0, ids.shape[0], rows):
        j = (ids[r: r + rows, :, None] * stride + near).flatten(1)
        ok = (ids[r: r + rows, :, None] >= 0).expand(-1, -1, near.numel()).flatten(1)
        ok = ok & (j >= 0) & (j < starts)
        j = torch.where(ok, j, -1)
        j, _ = torch.sort(j, 1)
        ok = (j >= 0) & torch.cat([torch.ones_like(j[:, :1]).bool(), j[:, 1:] != j[:, :-1]], 1)
        j = j.clamp(min=0)
        c = cls[j[..., None] + p]                              # [r, pool, T]
        n = c.shape[0]
        xr = torch.view_as_real(x[r: r + n]).reshape(n * enc.C, -1)
        xr = xr[c + torch.arange(n, device="cuda")[:, None, None] * enc.C]
        z = (torch.view_as_complex(xr.view(*c.shape, enc.m, 2)) * turn).sum((-1, -2))
        F = torch.where(ok, (z.real.square() + z.imag.square()) / norm2[j], 0.0)
        score.append(torch.topk(F, case["k"], dim=1)[0])
    return dict(idx=None, score=torch.cat(score))


def _exact_index(case, seed):
    ref = _reference(case["ref_len"], seed)
    learned_ = _network(seed) if case["kind"] == "index_learned" else None
    enc = _Encoder(case.get("encoding", "letters"), case["window"], learned_)
    reduced = _row_reals(case) == 192
    W = (case["ref_len"] - case["window"]) // case["stride"] + 1
    rows = torch.empty((W, _row_reals(case)), dtype=torch.float64, device="cuda")
    norm2 = torch.empty(W, dtype=torch.float64, device="cuda")
    for a, v in enc.windows(ref, case["stride"]):
        unit, n2 = enc.unit(v)
        norm2[a: a + n2.numel()] = n2
        rows[a: a + n2.numel()] = _reals(unit, case["precision"], reduced)
    return dict(rows=rows, norm2=norm2)


def _exact_heads(case, seed):
    ref = _reference(max(100_000, 4 * case["read_len"]), seed)
    seq, off = _reads(ref, np.full(case["n_reads"], case["read_len"], dtype=np.int64), 0.02, seed)
    enc = _Encoder(case["encoding"], case["read_len"])
    x, _ = enc.unit(enc.heads(seq, off))
    x = _reduced(x) if _row_reals(case) == 192 else x
    rows = torch.stack([torch.view_as_real(v.contiguous()).flatten(1) for v in (x, 1j * x)], 1)
    if case["precision"] == "fp8":  # codes of v / 2^e, e the least with all of a read in range
        most = rows.abs().amax((1, 2), keepdim=True)
        rows = rows * torch.exp2(-torch.ceil(torch.log2(most / 448)))
    return dict(rows=rows)


def _edit_distances(a, a_off, b, b_off):
    """Levenshtein distances, all pairs at once, by anti-diagonal-free row updates."""
    n, width = len(a_off) - 1, int(np.diff(b_off).max())
    A = torch.from_numpy(a).cuda().view(n, -1).long()
    size = torch.from_numpy(np.diff(b_off)).cuda()
    at = torch.from_numpy(b_off[:-1]).cuda()[:, None] + torch.arange(width, device="cuda")
    B = torch.from_numpy(b).cuda()[at.clamp(max=len(b) - 1)].long()
    j = torch.arange(width + 1, device="cuda")
    row = j.expand(n, -1).clone()
    for i in range(A.shape[1]):
        best = torch.cat([row[:, :1] + 1, torch.minimum(row[:, 1:] + 1,
                                                        row[:, :-1] + (B != A[:, i: i + 1]))], 1)
        row = torch.cummin(best - j, 1)[0] + j  # the cheapest run of insertions before each place
    return torch.gather(row, 1, size[:, None])[:, 0]


def _encode_pairs(params, seq, off, N):
    """Learned encodings [n, 4, M] (complex) of strings of up to 256 letters."""
    W1, b1, W2, b2 = _unpack(params)
    T = int(np.diff(off).max()) - CONTEXT + 1
    start, size = torch.from_numpy(off[:-1]).cuda(), torch.from_numpy(np.diff(off)).cuda()
    at = start[:, None] + torch.arange(T + CONTEXT - 1, device="cuda")
    mid, x = _flanks(torch.from_numpy(seq).cuda()[at.clamp(max=len(seq) - 1)])
    live = torch.arange(T, device="cuda") < (size - CONTEXT + 1)[:, None]
    h = torch.relu(sum(W1.t()[x[..., i]] for i in range(8)) + b1)
    o = (h @ W2.t() + b2).view(*mid.shape, 4, M)
    o = torch.gather(o, 2, mid[..., None, None].expand(-1, -1, 1, M))[:, :, 0]
    theta = torch.arange(T, device="cuda").double()[:, None] * _factors(M, "default") * (2 * math.pi / N)
    u = torch.polar(live[..., None].double().expand_as(o), theta + o)
    hot = torch.nn.functional.one_hot(mid, 4).double().transpose(1, 2)
    return torch.complex(hot @ u.real, hot @ u.imag)


def _exact_train(case, seed):
    a, a_off, b, b_off = _pairs(case, seed)
    ld = _edit_distances(a, a_off, b, b_off)
    params = torch.from_numpy(_network(seed)).cuda().double()
    m, v, step = _adam_state(seed)
    m, v = torch.from_numpy(m).cuda().double(), torch.from_numpy(v).cuda().double()
    B, losses = case["batch"], []

    def strings(seq, off, i):
        return seq[off[i]: off[i + B]], off[i: i + B + 1] - off[i]

    for s in range(case["steps"]):
        p = params.clone().requires_grad_()
        ca = _encode_pairs(p, *strings(a, a_off, s * B), case["length"])
        cb = _encode_pairs(p, *strings(b, b_off, s * B), case["length"])
        z = (ca.conj() * cb).sum((1, 2))
        norm = [c.real.square().sum((1, 2)) + c.imag.square().sum((1, 2)) for c in (ca, cb)]
        F = (z.real.square() + z.imag.square()) / (norm[0] * norm[1])
        y = ld[s * B: (s + 1) * B]
        ranked = y[:, None] < y[None, :]
        soft = torch.nn.functional.softplus(-(F[:, None] - F[None, :]) / TAU, threshold=1e9)
        loss = (soft * ranked).sum() / ranked.sum().clamp(min=1)
        grad, = torch.autograd.grad(loss, p)
        losses.append(loss.detach())
        step += 1
        m, v = BETA1 * m + (1 - BETA1) * grad, BETA2 * v + (1 - BETA2) * grad * grad
        params = params - 3e-3 * (m / (1 - BETA1 ** step)) / ((v / (1 - BETA2 ** step)).sqrt() + EPS)
    return dict(ld=None, loss=torch.stack(losses), params=params, m=m, v=v)


def _philox(c0, c1, c2, c3, key):
    """Four 32-bit words of Philox4x32-10 (Salmon, Moraes, Dror and Shaw, SC 2011)."""
    mask, k0, k1 = 0xFFFFFFFF, key & 0xFFFFFFFF, 0

    def product(a, x):
        return (a * (x >> 16) + ((a * (x & 0xFFFF)) >> 16)) >> 16, (a * x) & mask

    for _ in range(10):
        hi0, lo0 = product(0xD2511F53, c0)
        hi1, lo1 = product(0xCD9E8D57, c2)
        c0, c1, c2, c3 = hi1 ^ c1 ^ k0, lo1, hi0 ^ c3 ^ k1, lo0
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c0, c1, c2, c3


def _exact_thresholds(case, seed):
    ref = _reference(case["ref_len"], seed)
    N, stride, G = case["window"], case["stride"], case["ref_len"]
    enc = _Encoder("letters", N)
    W = (G - N) // stride + 1
    cut = int(math.floor(float(np.float32(case["error"])) / 3 * 4294967296.0))
    turn = torch.view_as_real(_turn(enc.f, torch.arange(N, device="cuda"), N)).reshape(N, 2 * M)

    def encode(letters):
        v = torch.stack([(letters == c).double() @ turn for c in range(4)], 1)
        return enc.unit(torch.view_as_complex(v.view(-1, 4, M, 2)).transpose(1, 2))[0]

    out = []
    for a in range(0, W, 1 << 17):
        j = torch.arange(a, min(W, a + (1 << 17)), device="cuda")
        own = encode(ref[j[:, None] * stride + torch.arange(N, device="cuda")])
        F = []
        for copy in range(case["copies"]):
            letters = torch.full((j.numel(), N + 1), 4, dtype=torch.uint8, device="cuda")
            pos, n = j * stride, torch.zeros_like(j)
            for t in range(8 * N + 64):
                if t >= N and t % 8 == 0 and bool((n == N).all()):
                    break
                w0, w1, w2, _ = _philox(j, torch.zeros_like(j), torch.full_like(j, copy),
                                        torch.full_like(j, t), seed + 1)
                ins = (w0 < cut) | (pos >= G)
                dele, sub = ~ins & (w0 < 2 * cut), ~ins & (w0 >= 2 * cut) & (w0 < 3 * cut)
                old = ref[pos.clamp(max=G - 1)].long()
                new = torch.where(ins, w1 & 3, torch.where(sub, (old + 1 + w2 % 3) & 3, old))
                # a finished copy writes to the spare last place
                letters.scatter_(1, torch.where(dele, N, n)[:, None], new.to(torch.uint8)[:, None])
                n = torch.where(dele, n, n + 1).clamp_(max=N)
                pos = torch.where(ins, pos, pos + 1)
            z = (own.conj() * encode(letters[:, :N])).sum(1)
            F.append(z.real.square() + z.imag.square())
        out.append(torch.sort(torch.stack(F, 1), 1)[0][:, min(1, case["copies"] - 1)])
    return torch.cat(out)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("map", "map_learned"):
        return _exact_map(case, seed)
    if kind in ("index", "index_learned"):
        return _exact_index(case, seed)
    by_kind = dict(heads=_exact_heads, batch=_exact_batch, coarse=_exact_coarse, train=_exact_train,
                   thresholds=_exact_thresholds)
    # the regime's spans follow the product's proposals, which 64 bits do not have
    return by_kind[kind](case, seed) if kind in by_kind else None
