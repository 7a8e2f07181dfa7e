"""The work that users of this library have it do, as cases that can be timed and compared.

Three kinds of user stand behind the list:
  - a data-parallel training job on real GPUs calls the codec on ONE worker's chunk at a time: the leaf's
    compress, the fused decompress-accumulate-recompress hop, the sink's decompress-accumulate (with or
    without the restore fused in) and an all-gather receiver's decompress;
  - the same job prepares every bucket: statistics, their combination, the bit allocation, the means and
    origins in reordered order;
  - a study of compressed collectives replays whole schedules of N simulated workers inside one GPU, for
    this codec and for the MX formats it is compared with, or asks for the whole simulated all-reduce.

Inputs are synthetic gradients (workloads.py's distributions).  Every result of the library is a pure
function of its arguments, bit for bit, so every case is compared exactly.
"""
import math

import torch

from paper_2602_08923_amd import allreduce, prep, workloads
from paper_2602_08923_amd import binding as B

TOPOLOGY = {"ring": B.DQ_RING, "butterfly": B.DQ_BUTTERFLY, "chain": B.DQ_CHAIN}
CODEC = {"dynamiq": B.DQ_DYNAMIQ, "mxfp8": B.DQ_MXFP8_E4M3, "mxfp6": B.DQ_MXFP6_E3M2, "mxfp4": B.DQ_MXFP4_E2M1}
CALLS = ("compress", "hop", "sink", "receive", "restore")


def _call(op, dtype, workers, n2, n4, n8, n16, means, gather):
    """One worker's call on one chunk of n2 + n4 + n8 + n16 super-groups (2, 4, 8 and 16 bits)."""
    return {"op": op, "dtype": dtype, "workers": workers, "n2": n2, "n4": n4, "n8": n8, "n16": n16, "means": means, "gather": gather}


def _replay(topology, codec, dtype, workers, super_groups, buckets, bits, max_width, means, original, all_gather):
    """One replay of a schedule; super_groups per bucket (chain: of the one chunk), bits per coordinate."""
    return {"op": "replay", "topology": topology, "codec": codec, "dtype": dtype, "workers": workers,
            "super_groups": super_groups, "buckets": buckets, "bits": bits, "max_width": max_width, "means": means,
            "original": original, "all_gather": all_gather}


def _prepare_bucket(dtype, workers, super_groups, buckets, bits, max_width):
    return {"op": "statistics", "dtype": dtype, "workers": workers, "super_groups": super_groups, "buckets": buckets,
            "bits": bits, "max_width": max_width}


def _allreduce(topology, workers, super_groups, bits, max_width, all_gather):
    return {"op": "allreduce", "topology": topology, "workers": workers, "super_groups": super_groups, "bits": bits,
            "max_width": max_width, "all_gather": all_gather}


def listed():
    return [
        # the smallest call: a hop of a few super-groups in fp32 (a short tensor of its own bucket, four workers)
        dict(_call("hop", "f32", 4, 5, 8, 3, 0, False, False), name="hop_16sg_f32"),
        # the leaf of an 8-worker ring over one 25 MB bf16 DDP bucket: one chunk, about 4 bits per coordinate
        dict(_call("compress", "bf16", 8, 2201, 4198, 1, 0, True, False), name="leaf_6400sg_bf16"),
        # a ragged chunk of an odd worker count with all four widths, read from the original tensor through the index
        dict(_call("hop", "bf16", 5, 701, 1502, 851, 133, True, True), name="hop_3187sg_gather"),
        # a hop of a 125 M entry chunk (64 workers, 5 bits): the largest single launches of the benchmark
        dict(_call("hop", "bf16", 64, 32411, 364018, 91853, 0, True, False), name="hop_488282sg_bf16"),
        # the sink of that chunk, gathered on the way in, restored to the original order on the way out
        dict(_call("restore", "bf16", 64, 32411, 364018, 91853, 0, True, True), name="restore_488282sg_bf16"),
        # the benchmark's headline: reduce-scatter of one 25 MB bf16 bucket over a ring of 8
        dict(_replay("ring", "dynamiq", "bf16", 8, 51200, 1, 4.0, 8, True, False, False), name="ring8_25mb_bf16"),
        # a small fp32 all-reduce: ring of 4, 2^20 entries, all-gather included, on the original tensors
        dict(_replay("ring", "dynamiq", "f32", 4, 4096, 1, 5.0, 8, True, True, True), name="ring4_1m_f32_allgather"),
        # recursive halving over 16 workers, several buckets of a large model per call, 3 bits
        dict(_replay("butterfly", "dynamiq", "bf16", 16, 51200, 8, 3.0, 8, True, False, False), name="butterfly16_8buckets"),
        # the large-scale simulation: hundreds of workers, a few super-groups per chunk, W = {2, 4, 8, 16}
        dict(_replay("ring", "dynamiq", "bf16", 256, 4096, 1, 8.5, 16, True, True, True), name="ring256_4096sg_w16"),
        # the comparison codec on the headline's bucket
        dict(_replay("ring", "mxfp8", "bf16", 8, 51200, 1, 8.25, 8, False, False, False), name="ring8_25mb_mxfp8"),
        # what precedes the main stage, for the headline's bucket
        dict(_prepare_bucket("bf16", 8, 51200, 1, 4.0, 8), name="statistics8_25mb"),
        # the whole simulated all-reduce, as the studies of accuracy call it
        dict(_allreduce("ring", 8, 8192, 4.6875, 8, True), name="allreduce8_8192sg"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["call", "call", "call", "replay", "replay", "replay", "replay", "statistics", "allreduce"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    max_width = rng.choice([8, 8, 16])
    if kind == "call":
        n = _log(rng, 8, 488282)
        cut = sorted(rng.randint(0, n) for _ in range(3))
        n2, n4, n8, n16 = cut[0], cut[1] - cut[0], cut[2] - cut[1], n - cut[2]
        if max_width == 8:
            n4, n16 = n4 + n16, 0
        op = rng.choice(CALLS)
        return _call(op, dtype, _log(rng, 2, 64), n2, n4, n8, n16, rng.random() < 0.7 and op != "receive",
                     rng.random() < 0.4 and op != "receive")
    bits = round(rng.uniform(3.0, 6.0) if max_width == 8 else rng.uniform(5.0, 8.5), 2)
    if kind == "statistics":
        workers, buckets = _log(rng, 2, 16), rng.choice([1, 1, 2, 5])
        return _prepare_bucket(dtype, workers, _log(rng, 64, min(60000, 1200000 // (workers * buckets))), buckets, bits, max_width)
    topology = rng.choice(["ring", "ring", "butterfly", "butterfly", "chain"] if kind == "replay" else ["ring", "butterfly"])
    if kind == "allreduce":
        workers = 1 << rng.randint(1, 5) if topology == "butterfly" else _log(rng, 2, 32)
        chunk = _log(rng, 4, max(8, 400000 // (workers * workers)))
        return _allreduce(topology, workers, chunk * workers, bits, max_width, rng.random() < 0.7)
    codec = rng.choice(["dynamiq", "dynamiq", "dynamiq", "mxfp8", "mxfp6", "mxfp4"])
    workers = 1 << rng.randint(1, 7) if topology == "butterfly" else _log(rng, 2, 256)
    buckets = 1 if topology == "chain" else rng.choice([1, 1, 1, 3, 8])
    most = 2500000 // (workers * buckets)  # super-groups per bucket: at most a third of the largest listed replay
    chunks = 1 if topology == "chain" else workers
    super_groups = chunks * max(1, round(_log(rng, 64, max(128, min(60000, most))) / chunks))
    mx = codec != "dynamiq"
    return _replay(topology, codec, dtype, workers, super_groups, buckets, bits, max_width, not mx and rng.random() < 0.8,
                   not mx and topology != "chain" and rng.random() < 0.5, rng.random() < 0.5)


# ---------------------------------------------------------------------------------------- inputs
def _torch_dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _gradients(case, seed, count, super_groups):
    """`count` workers' gradients: norms that differ from super-group to super-group by the fitted mixture's
    law, Gaussian entries with 0.1 % of them 100 times as large."""
    dev = torch.device("cuda:0")
    magnitudes = workloads.mixture_magnitudes(super_groups, seed=seed % 100003, device=dev).clamp_(1e-12, 1e3)
    gen = torch.Generator(device=dev)
    grads = []
    for w in range(count):
        gen.manual_seed(1000003 * (seed % 1000003) + w)
        x = torch.randn(super_groups, 256, generator=gen, device=dev)
        x *= (magnitudes / 16.0).unsqueeze(1)
        x = x.reshape(-1)
        at = torch.randint(0, x.numel(), (max(1, x.numel() // 1000),), generator=gen, device=dev)
        x[at] = x[at] * 100.0
        grads.append(x.to(_torch_dtype(case)))
    return grads


def _allocation(case, grads):
    """Statistics, allocation and the reordered means of a bucket set, by the library."""
    n, J = len(grads), case["super_groups"]
    total = grads[0].numel() // 256
    mu_all = torch.empty((n, total), dtype=torch.float32, device=grads[0].device)
    F_all = torch.empty_like(mu_all)
    for w, g in enumerate(grads):
        B.dq_sg_stats(g, mu_all[w], F_all[w])
    mu, F = B.dq_stats_combine(mu_all, F_all)
    budget = int(math.floor(prep.code_bits(case["bits"]) * J))
    _, pos, counts = B.dq_allocate(F, J, budget, max_width=case["max_width"])
    mu_main, origin = B.dq_reorder_mean(mu, pos, J, counts, with_origin=True)
    return pos, [[int(v) for v in row[:4]] for row in counts.cpu().tolist()], mu_main, origin


def _prepare_call(case, seed):
    counts = [case["n2"], case["n4"], case["n8"], case["n16"]]
    n_sg, n = sum(counts), case["workers"]
    ctx = B.Context(n, seed=seed)
    chunk = B.make_chunk(seed % 1000 * 7919, counts)
    mine, other = _gradients(case, seed, 2, n_sg)
    dev = mine.device
    s = {"op": case["op"], "ctx": ctx, "chunk": chunk, "rank": 1 % n, "local": mine, "mu": None, "index": None}
    if case["means"]:
        s["mu"] = B.dq_sg_stats(mine)[0]
        if case["n16"]:
            s["mu"][n_sg - case["n16"]:] = 0.0  # raw bf16 super-groups keep their mean
    if case["gather"]:
        gen = torch.Generator(device=dev)
        gen.manual_seed(seed + 17)
        s["index"] = torch.randperm(n_sg, generator=gen, device=dev).to(torch.int32)
    if case["op"] != "compress":  # the message of the worker before
        s["message"] = ctx.dq_compress(other, chunk, 0)
    if case["op"] in ("compress", "hop"):
        s["out"] = torch.zeros(B.dq_packed_bytes(chunk), dtype=torch.uint8, device=dev)
    else:
        s["out"] = torch.empty(n_sg * 256, dtype=torch.float32, device=dev)
    if case["op"] == "restore":
        s["origin"] = s["index"]
        if s["origin"] is None:
            s["origin"] = torch.arange(n_sg - 1, -1, -1, dtype=torch.int32, device=dev)
    return s


def prepare(case, seed):
    if case["op"] in CALLS:
        return _prepare_call(case, seed)
    workers, J, buckets = case["workers"], case["super_groups"], case.get("buckets", 1)
    grads = _gradients(case, seed, workers, J * buckets)
    s = {"op": case["op"], "grads": grads, "case": case, "seed": seed}
    if case["op"] == "statistics":
        s["mu_all"] = torch.empty((workers, J * buckets), dtype=torch.float32, device=grads[0].device)
        s["F_all"] = torch.empty_like(s["mu_all"])
        s["budget"] = int(math.floor(prep.code_bits(case["bits"]) * J))
    elif case["op"] == "replay":
        ctx = B.Context(workers, seed=seed)
        topology, codec = TOPOLOGY[case["topology"]], CODEC[case["codec"]]
        if case["codec"] != "dynamiq":
            s["replay"] = B.Replay(ctx, topology, codec, grads, J, n_buckets=buckets, all_gather=case["all_gather"])
        else:
            pos, widths, mu_main, origin = _allocation(case, grads)
            if not case["original"]:
                grads = [B.dq_reorder(g, pos, J) for g in grads]
            s["replay"] = B.Replay(ctx, topology, codec, grads, J, widths, n_buckets=buckets, all_gather=case["all_gather"],
                                   mu=mu_main if case["means"] else None, origin=origin if case["original"] else None,
                                   inputs_in_original_order=case["original"])
        s["grads"] = None  # the replay holds them
    return s


# ---------------------------------------------------------------------------------------- one pass
def run(s):
    op = s["op"]
    if op == "compress":
        return s["ctx"].dq_compress(s["local"], s["chunk"], s["rank"], packed_out=s["out"], mu=s["mu"], sg_index=s["index"])
    if op == "hop":
        return s["ctx"].dq_dar_hop(s["message"], s["local"], s["chunk"], s["rank"], packed_out=s["out"], mu=s["mu"], sg_index=s["index"])
    if op == "sink":
        return s["ctx"].dq_decompress(s["message"], s["chunk"], local=s["local"], out=s["out"], mu=s["mu"], sg_index=s["index"])
    if op == "receive":
        return s["ctx"].dq_decompress(s["message"], s["chunk"], out=s["out"])
    if op == "restore":
        return s["ctx"].dq_decompress_restore(s["message"], s["chunk"], s["origin"], s["out"], local=s["local"], mu=s["mu"],
                                              mu_back=s["mu"], sg_index=s["index"])
    if op == "replay":
        s["replay"].run()
        return s["replay"].out
    case, grads = s["case"], s["grads"]
    if op == "statistics":
        J = case["super_groups"]
        for w, g in enumerate(grads):
            B.dq_sg_stats(g, s["mu_all"][w], s["F_all"][w])
        mu, F = B.dq_stats_combine(s["mu_all"], s["F_all"])
        widths, pos, counts = B.dq_allocate(F, J, s["budget"], max_width=case["max_width"])
        mu_main, origin = B.dq_reorder_mean(mu, pos, J, counts, with_origin=True)
        return {"mu": mu, "F": F, "widths": widths, "pos": pos, "counts": counts, "mu_main": mu_main, "origin": origin}
    total, _ = allreduce.simulated_allreduce(grads, case["bits"], topology=TOPOLOGY[case["topology"]], seed=s["seed"],
                                             all_gather=case["all_gather"], max_width=case["max_width"])
    return total


# ---------------------------------------------------------------------------------------- what a pass must do
def work(case):
    """Inputs read once, outputs written once.  Operations per entry and worker, in fp32: 1 to take the mean off, 2 to
    decode and add, 1 for the maximum, 1 to normalise, 2 for the random number, 3 for the level and the rounding."""
    size = 4 if case.get("dtype", "bf16") == "f32" else 2
    if case["op"] in CALLS:
        n2, n4, n8, n16 = case["n2"], case["n4"], case["n8"], case["n16"]
        sg = n2 + n4 + n8 + n16
        packed = 64 * n2 + 128 * n4 + 256 * n8 + 512 * n16 + 18 * (n2 + n4 + n8)
        op = case["op"]
        b = 0 if op == "receive" else sg * 256 * size + (4 * sg if case["means"] else 0) + (4 * sg if case["gather"] else 0)
        b += packed * (2 if op == "hop" else 1)
        b += 0 if op in ("compress", "hop") else sg * 1024
        b += 4 * sg * (2 if case["means"] else 1) if op == "restore" else 0
        return {"bytes": b, "flops": sg * 256 * {"compress": 8, "hop": 10, "sink": 3, "receive": 1, "restore": 4}[op]}
    entries = case["workers"] * case["super_groups"] * case.get("buckets", 1) * 256
    if case["op"] == "statistics":
        sg = entries // 256 // case["workers"]
        return {"bytes": entries * size + sg * (case["workers"] * 8 + 21), "flops": entries * 3}
    out = entries // case["workers"] * 4
    return {"bytes": entries * size + out, "flops": entries * 10}


def tolerance(case):
    return "exact"
