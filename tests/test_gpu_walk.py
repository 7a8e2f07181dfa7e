"""A replay run whole (one launch, every tile carried through all its hops) against the same replay run step
by step, whose steps the parity tests hold against the oracle: same result, same messages of the last two
steps -- at the edges of tiles, of the draws' batches and of the split over waves.  And the bounds
check of super-group indices in front of a call."""
import threading
import time

import pytest
import torch

from paper_2602_08923_amd import allreduce
from paper_2602_08923_amd import binding as B

pytestmark = pytest.mark.gpu

TOPO = {"ring": B.DQ_RING, "butterfly": B.DQ_BUTTERFLY, "chain": B.DQ_CHAIN}


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def gradients(n, n_sg, dtype, dev, seed):
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    scale = torch.exp(2.0 * torch.randn(n_sg, 1, generator=gen, device=dev)) * 1e-3
    grads = []
    for _ in range(n):
        x = torch.randn(n_sg, 256, generator=gen, device=dev) * scale
        x[::7, :32] = 0.0
        x[::5, 16:48] *= -0.0
        grads.append(x.reshape(-1).to(dtype))
    return grads


def whole_against_steps(rp, chunks):
    for t in range(rp.n_steps):
        rp.run_steps(t, 1)
    torch.cuda.synchronize()
    want = rp.out.clone()
    msgs = {}
    if chunks:
        n = rp.ctx.n_workers
        kept = [t for t in (n - 3, n - 2) if t >= 0]
        msgs = {(t, b, c): rp.message(t, b, c) for t in kept for b in range(rp.desc.n_buckets) for c in range(chunks)}
        saved = {k: v.clone() for k, v in msgs.items()}
        for v in msgs.values():
            v.fill_(0xA5)
    rp.out.fill_(float("nan"))
    rp.run()
    torch.cuda.synchronize()
    assert torch.equal(rp.out.view(torch.int32), want.view(torch.int32))
    for k, v in msgs.items():
        same = v == saved[k]
        same[-15:] |= v[-15:] == 0xA5                      # padding bytes are never written
        assert bool(same.all()), f"message of step, bucket, chunk {k}"


CASES = [
    # topology, workers, widths of the bucket(s), all_gather
    ("ring", 2, [[1, 1, 0, 0]], False), ("ring", 3, [[3, 5, 4, 3]], True), ("ring", 5, [[20, 10, 4, 1], [0, 0, 0, 35]], False),
    ("ring", 17, [[17, 40, 20, 8]], True), ("ring", 16, [[16, 60, 30, 6]], False), ("ring", 9, [[9, 9, 9, 0]], True),
    ("chain", 2, [[0, 5, 0, 0]], True), ("chain", 4, [[6, 7, 9, 3]], False), ("chain", 33, [[5, 5, 5, 5]], True),
    ("butterfly", 2, [[3, 2, 2, 1]], True), ("butterfly", 4, [[4, 12, 8, 0], [24, 0, 0, 0]], False),
    ("butterfly", 8, [[10, 30, 20, 4]], True), ("butterfly", 32, [[32, 96, 30, 2]], False), ("butterfly", 64, [[0, 64, 64, 0]], True),
]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("means", [False, True])
@pytest.mark.parametrize("topology,n,widths,all_gather", CASES)
def test_whole_replay_equals_its_steps(dev, topology, n, widths, all_gather, means, dtype):
    J, nb = sum(widths[0]), len(widths)
    grads = gradients(n, J * nb, dtype, dev, 100 * n + J)
    ctx = B.Context(n, seed=n)
    mu = None
    if means:
        mu = torch.stack([g.float().reshape(-1, 256).mean(dim=1) for g in grads]).mean(dim=0).contiguous()
    rp = B.Replay(ctx, TOPO[topology], B.DQ_DYNAMIQ, grads, J, widths, n_buckets=nb, first_sg=2 ** 33 + 5, all_gather=all_gather, mu=mu)
    whole_against_steps(rp, {"ring": n, "chain": 1, "butterfly": 0}[topology])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("topology,n,widths,all_gather", [
    # tiles of two super-groups, and of four, of a wave: chunks with remainders in every width
    ("ring", 17, [[1001, 2002, 1503, 594]], True), ("chain", 33, [[1501, 2003, 1707, 302]], False),
    ("butterfly", 64, [[1601, 3203, 1500, 608]], True), ("butterfly", 32, [[2049, 2047, 640, 0]], False),
    ("ring", 5, [[1601, 3002, 1603, 304]], False), ("ring", 17, [[1501, 3002, 1503, 352]], True), ("chain", 33, [[0, 7003, 3300, 6]], True),
    ("butterfly", 8, [[1601, 3002, 1693, 104]], True), ("butterfly", 64, [[3201, 6003, 1300, 56]], False),
])
def test_whole_replay_of_many_super_groups_equals_its_steps(dev, topology, n, widths, all_gather, dtype):
    test_whole_replay_equals_its_steps(dev, topology, n, widths, all_gather, True, dtype)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("topology,n,widths", [
    # between one and three tiles of four per wave, several buckets, the last row of blocks on the CUs not full: waves hold 0 to 5 tiles of a width
    ("butterfly", 8, [[2401, 3202, 1501, 96]] * 3), ("butterfly", 2, [[9001, 6002, 5001, 0], [0, 4, 20000, 0]]), ("butterfly", 16, [[23001, 9, 1230, 0]]),
    # CUs with a block more, which take the 16-bit tiles
    ("butterfly", 16, [[385, 376, 4981, 3570]]), ("butterfly", 8, [[289, 1687, 55, 1161]] * 3), ("butterfly", 8, [[1, 9, 0, 8790]]),
    ("butterfly", 4, [[7433, 0, 15439, 0]]), ("butterfly", 4, [[5601, 3002, 1502, 207]] * 2), ("butterfly", 2, [[21001, 13802, 2, 1001]]),
    ("ring", 6, [[9001, 602, 501, 96]] * 3), ("ring", 3, [[20000, 31000, 1, 8]]), ("ring", 9, [[2, 16000, 8001, 0]]),
])
def test_whole_replay_of_few_tiles_per_wave_equals_its_steps(dev, topology, n, widths, dtype):
    test_whole_replay_equals_its_steps(dev, topology, n, widths, False, True, dtype)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("all_gather", [False, True])
@pytest.mark.parametrize("topology,n,J", [("ring", 2, 3072), ("ring", 2, 3074), ("ring", 2, 4096), ("ring", 2, 4098), ("butterfly", 2, 3074), ("butterfly", 2, 4098),
                                          ("butterfly", 2, 5120), ("butterfly", 2, 5122), ("butterfly", 4, 4100), ("butterfly", 4, 5376), ("butterfly", 4, 5380), ("butterfly", 4, 5632), ("butterfly", 4, 5636), ("ring", 11, 5368),
                                          ("ring", 16, 5376), ("ring", 16, 5392)])
def test_whole_replay_of_few_super_groups_per_cu_equals_its_steps(dev, topology, n, J, all_gather, dtype):
    """Both sides of the sizes from which tiles of two and of four super-groups are taken; the all-gather moves some."""
    test_whole_replay_equals_its_steps(dev, topology, n, [[J // 3, J - J // 3 - 901, 701, 200]], all_gather, True, dtype)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("all_gather", [False, True])
@pytest.mark.parametrize("topology,n,J", [("ring", 4, 2044), ("ring", 4, 2048), ("ring", 4, 2052), ("chain", 5, 2049), ("ring", 12, 5160), ("butterfly", 16, 2048),
                                          ("butterfly", 16, 5632), ("butterfly", 32, 4096)])
def test_whole_replay_with_short_and_long_level_entries_equals_its_steps(dev, topology, n, J, all_gather, dtype):
    """Rings and chains on both sides of two waves per SIMD, tiles of one and of two, all four widths."""
    test_whole_replay_equals_its_steps(dev, topology, n, [[J // 4, J // 4, J - J // 4 * 2 - 77, 77]], all_gather, True, dtype)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("topology,n,J", [("ring", 8, 2056), ("ring", 9, 2043), ("ring", 9, 2052), ("chain", 8, 2100), ("chain", 9, 2100)])
def test_whole_replay_on_both_sides_of_eight_workers_equals_its_steps(dev, topology, n, J, dtype):
    """Level entries of 16 bytes up to eight workers, of 8 from nine on where SIMDs have more than two waves, in fp32 always."""
    test_whole_replay_equals_its_steps(dev, topology, n, [[J // 4, J // 4, J - J // 4 * 2 - 77, 77]], True, True, dtype)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("topology,J", [("ring", 64), ("butterfly", 64), ("ring", 8192), ("butterfly", 8192)])   # one and four super-groups per tile
def test_whole_replay_of_extreme_magnitudes_equals_its_steps(dev, topology, J, dtype):
    """Groups whose maximum's reciprocal is denormal, groups too small for a scale beside ones that are not, super-groups encoded as zero."""
    grads = gradients(8, J, dtype, dev, J)
    for w, g in enumerate(grads):
        x = g.view(J, 16, 16)
        x[::3, ::2] *= 2.0 ** -124
        x[1::6] *= 0.0 if w % 2 else 2.0 ** -118
        x[2::6, w] = torch.sign(x[2::6, w]) * 1.5e38
    ctx = B.Context(8, seed=5)
    whole_against_steps(B.Replay(ctx, TOPO[topology], B.DQ_DYNAMIQ, grads, J, [[J // 4, J // 2, J // 4, 0]]), 8 if topology == "ring" else 0)


@pytest.mark.parametrize("topology", ["ring", "butterfly"])
@pytest.mark.parametrize("J", [8192, 66000])                # one tile per wave, and several waves' shares per chunk
def test_whole_replay_on_original_tensors_over_the_whole_grid(dev, topology, J):
    n = 4
    grads = gradients(n, J, torch.bfloat16, dev, J)
    widths = [[J // 4, J // 2, J // 4 - 600, 600]]
    gen = torch.Generator(device=dev)
    gen.manual_seed(3)
    origin = torch.randperm(J, generator=gen, device=dev).to(torch.int32)
    mu = torch.randn(J, generator=gen, device=dev) * 1e-4
    rp = B.Replay(B.Context(n, seed=2), TOPO[topology], B.DQ_DYNAMIQ, grads, J, widths, mu=mu, origin=origin, inputs_in_original_order=True)
    whole_against_steps(rp, 0)


@pytest.mark.parametrize("fmt", [B.DQ_MXFP8_E4M3, B.DQ_MXFP6_E3M2, B.DQ_MXFP4_E2M1])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("topology,n,J,nb,all_gather", [("ring", 2, 2, 1, False), ("ring", 5, 45, 2, True), ("chain", 7, 9, 1, False),
                                                        ("chain", 3, 8, 1, True), ("butterfly", 2, 2, 3, True),
                                                        ("butterfly", 16, 16 * 9, 2, False), ("ring", 4, 36000, 1, False),
                                                        # groups of eight leaves; both sides of the sizes at which the split changes
                                                        ("ring", 8, 24, 1, False), ("ring", 15, 45, 1, True), ("chain", 16, 7, 1, False),
                                                        ("ring", 17, 17, 1, False), ("chain", 24, 3, 1, True), ("butterfly", 32, 96, 1, True),
                                                        ("chain", 3, 4096, 1, False), ("chain", 2, 5121, 1, False), ("ring", 4, 6144, 1, False),
                                                        ("ring", 4, 6148, 1, False), ("ring", 8, 32768, 1, False), ("butterfly", 8, 32760, 1, False),
                                                        ("ring", 8, 131072, 1, False), ("ring", 8, 8200, 1, False), ("ring", 4, 10244, 1, False),
                                                        ("butterfly", 8, 16392, 1, False), ("ring", 64, 8256, 1, False),
                                                        ("chain", 14, 5120, 1, True), ("chain", 14, 5121, 1, False), ("ring", 16, 14400, 1, True),
                                                        ("ring", 8, 21840, 1, False), ("ring", 8, 21856, 1, False), ("chain", 99, 9216, 1, False)])
def test_whole_mx_replay_equals_its_steps(dev, fmt, dtype, topology, n, J, nb, all_gather):
    grads = gradients(n, J * nb, dtype, dev, J + n)
    rp = B.Replay(B.Context(n), TOPO[topology], fmt, grads, J, n_buckets=nb, all_gather=all_gather)
    whole_against_steps(rp, {"ring": n, "chain": 1, "butterfly": 0}[topology])


@pytest.mark.parametrize("fmt", [B.DQ_MXFP8_E4M3, B.DQ_MXFP6_E3M2, B.DQ_MXFP4_E2M1])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("topology,n,J", [("ring", 4, 18428), ("ring", 4, 18432), ("ring", 8, 20480), ("ring", 16, 23040), ("ring", 8, 25592), ("ring", 8, 25600),
                                          ("butterfly", 8, 33272), ("butterfly", 8, 33280), ("ring", 48, 51216), ("butterfly", 4, 84480), ("chain", 2, 24577)])
def test_a_large_whole_mx_replay_equals_its_steps(dev, fmt, dtype, topology, n, J):
    """Both sides of the sizes, by tiles per CU, from which inputs that come from memory go four lanes to a block, and of the blocks per CU of the others."""
    rp = B.Replay(B.Context(n), TOPO[topology], fmt, gradients(n, J, dtype, dev, J + n), J)
    whole_against_steps(rp, {"ring": n, "chain": 1, "butterfly": 0}[topology])


@pytest.mark.parametrize("fmt", [B.DQ_MXFP8_E4M3, B.DQ_MXFP6_E3M2, B.DQ_MXFP4_E2M1])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("topology,n,J", [("ring", 5, 45), ("ring", 17, 17), ("butterfly", 16, 48)])
def test_whole_mx_replay_of_any_pattern_equals_its_steps(dev, fmt, dtype, topology, n, J):
    """Infinities, quiet and signalling NaN, denormals: every bit pattern may come from a worker."""
    gen = torch.Generator(device=dev)
    gen.manual_seed(n)
    word = torch.int32 if dtype == torch.float32 else torch.int16
    info = torch.iinfo(word)
    grads = [torch.randint(info.min, info.max, (J * 256,), dtype=word, device=dev, generator=gen).view(dtype) for _ in range(n)]
    rp = B.Replay(B.Context(n), TOPO[topology], fmt, grads, J)
    for t in range(rp.n_steps):
        rp.run_steps(t, 1)
    torch.cuda.synchronize()
    want = rp.out.clone()
    rp.run()
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(rp.out), torch.isnan(want))
    assert torch.equal(torch.nan_to_num(rp.out, nan=7.0).view(torch.int32), torch.nan_to_num(want, nan=7.0).view(torch.int32))


@pytest.mark.parametrize("at", [0, 3, 4, 4095, 8190, 8191, 8192, 10238, 10239, 14334, 14335])
def test_a_call_of_few_super_groups_checks_every_index_itself(dev, at):
    """Rounds of 8,192 indices per block, fours and the rest of the array; beyond 12,288 (decompress: of one array 16,384, of two
    10,240) the check is a launch of its own again.  Two arrays: the same one within two tensors of different length, and two."""
    ctx = B.Context(4, seed=1)
    for n_sg in {at + 1, at + 2, at + 5}:
        ch = B.make_chunk(0, [0, n_sg, 0])
        x = gradients(1, n_sg, torch.bfloat16, dev, n_sg)[0]
        message = ctx.dq_compress(x, ch, 1)
        bad = torch.arange(n_sg, dtype=torch.int32, device=dev)
        good = bad.clone()
        bad[at] = n_sg
        longer = torch.cat([x, x[:256]])
        def restored(local, index, origin, out_sgs):
            out = torch.full((out_sgs * 256,), 7.0, device=dev)
            try:
                ctx.dq_decompress_restore(message, ch, origin, out, local=local, sg_index=index)
                return "written"
            except B.DqError as e:
                torch.cuda.synchronize()
                assert bool((out == 7.0).all())
                return str(e)[:8]
        assert restored(x, good, good, n_sg) == "written"
        assert restored(x, bad, bad, n_sg + 1) == "sg_index"[:8]
        assert restored(longer, bad, bad, n_sg) == "out_base"[:8]
        assert restored(longer, bad, good, n_sg) == "written"
        assert restored(longer, good, bad, n_sg) == "out_base"[:8]
        assert restored(x, bad[:n_sg].clone(), good, n_sg) == "sg_index"[:8]
        hop = torch.full_like(message, 9)
        with pytest.raises(B.DqError, match="sg_index"):
            ctx.dq_dar_hop(message, x, ch, 2, packed_out=hop, sg_index=bad)
        torch.cuda.synchronize()
        assert bool((hop == 9).all())


@pytest.mark.parametrize("at", [12286, 12287, 12288, 16382, 16383, 16384])
def test_a_call_at_the_edge_of_its_own_check(dev, at):
    test_a_call_of_few_super_groups_checks_every_index_itself(dev, at)


def test_a_result_smaller_than_a_super_group_is_refused(dev):
    """No destination is good, and none may be written to before the check has spoken."""
    ctx, n_sg = B.Context(4, seed=1), 9
    ch = B.make_chunk(0, [2, n_sg - 2, 0])
    x = gradients(1, n_sg, torch.bfloat16, dev, 1)[0]
    index = torch.arange(n_sg, dtype=torch.int32, device=dev)
    message = ctx.dq_compress(x, ch, 1)
    out = torch.full((n_sg * 256,), 7.0, device=dev)
    for kw in ({}, {"local": x}, {"local": x, "sg_index": index}):
        with pytest.raises(B.DqError, match="out_base"):
            ctx.dq_decompress_restore(message, ch, index, out[:255], **kw)
    with pytest.raises(B.DqError):
        ctx.dq_dar_hop(message, x[:0], ch, 2, sg_index=index)
    torch.cuda.synchronize()
    assert bool((out == 7.0).all())


@pytest.mark.parametrize("n_sg", [1, 4, 2049, 70001])
def test_indices_out_of_bounds_are_refused_and_nothing_is_written(dev, n_sg):
    ctx = B.Context(4, seed=1)
    ch = B.make_chunk(0, [0, n_sg, 0])
    x = gradients(1, n_sg, torch.bfloat16, dev, n_sg)[0]
    good = torch.arange(n_sg - 1, -1, -1, dtype=torch.int32, device=dev)
    want = ctx.dq_compress(x.reshape(-1, 256).flip(0).reshape(-1).contiguous(), ch, 1)
    for at, value in ((0, n_sg), (n_sg - 1, -1)):
        bad = good.clone()
        bad[at] = value
        out = torch.full_like(want, 7)
        with pytest.raises(B.DqError, match="sg_index points outside"):
            ctx.dq_compress(x, ch, 1, packed_out=out, sg_index=bad)
        total = torch.full((n_sg * 256,), 7.0, device=dev)
        with pytest.raises(B.DqError, match="holds every destination"):
            ctx.dq_decompress_restore(want, ch, bad, total)
        torch.cuda.synchronize()
        assert bool((out == 7).all()) and bool((total == 7.0).all())
    for _ in range(300):
        got = ctx.dq_compress(x, ch, 1, sg_index=good)
    assert torch.equal(got, want)


def test_checks_of_several_threads_and_streams_do_not_mix(dev):
    """Workspaces pass from call to call, over streams, without a reset: good and refused calls, two indices and one, side by side."""
    n_sg, ctx = 5000, B.Context(4, seed=1)                  # three blocks of the check
    ch = B.make_chunk(0, [0, n_sg, 0])
    x = gradients(1, n_sg, torch.bfloat16, dev, 5)[0]
    good = torch.arange(n_sg - 1, -1, -1, dtype=torch.int32, device=dev)
    bad = good.clone()
    bad[::1111] = n_sg
    message = ctx.dq_compress(x, ch, 1, sg_index=good)
    restored = ctx.dq_decompress_restore(message, ch, good, torch.empty(n_sg * 256, device=dev), local=x, sg_index=good)
    torch.cuda.synchronize()
    errors = []

    def work(k):
        try:
            side = torch.cuda.Stream()
            with torch.cuda.stream(side):
                kept = torch.full_like(restored, 7.0)
                for i in range(40):
                    assert torch.equal(ctx.dq_compress(x, ch, 1, sg_index=good), message)
                    for index, origin, text in ((bad, good, "sg_index"), (good, bad, "every destination")):
                        if (i + k) % 3 == 0:
                            with pytest.raises(B.DqError, match=text):
                                ctx.dq_decompress_restore(message, ch, origin, kept, local=x, sg_index=index)
                    out = ctx.dq_decompress_restore(message, ch, good, torch.empty_like(restored), local=x, sg_index=good)
                    assert torch.equal(out.view(torch.int32), restored.view(torch.int32))
                assert bool((kept == 7.0).all())
        except BaseException as e:                          # noqa: BLE001 -- shown below
            errors.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_a_check_under_capture_is_refused_and_leaves_the_next_one_whole(dev):
    n_sg, ctx = 100, B.Context(4, seed=1)
    ch = B.make_chunk(0, [0, n_sg, 0])
    x = gradients(1, n_sg, torch.bfloat16, dev, 6)[0]
    index = torch.arange(n_sg - 1, -1, -1, dtype=torch.int32, device=dev)
    want = ctx.dq_compress(x, ch, 1, sg_index=index)
    counts = torch.arange(10, dtype=torch.int32, device=dev).reshape(2, 5)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        with pytest.raises(B.DqError, match="captur"):
            ctx.dq_compress(x, ch, 1, packed_out=want, sg_index=index)
        with pytest.raises(B.DqError, match="captur"):
            B.widths_of_buckets(counts)
        plain = ctx.dq_compress(x, ch, 1)                   # without indices there is nothing to check
    for _ in range(3):
        graph.replay()
        assert torch.equal(ctx.dq_compress(x, ch, 1, sg_index=index), want)
        assert torch.equal(ctx.dq_compress(x, ch, 1), plain)
        assert B.widths_of_buckets(counts) == [[0, 1, 2, 3], [5, 6, 7, 8]]


# ---- plans and streams: a plan's tables lie in memory that the stream's earlier work may still be using
ALLREDUCE = [dict(codec=B.DQ_MXFP8_E4M3), dict(codec=B.DQ_MXFP4_E2M1), dict(uniform_width=4), dict(uniform_width=8, topology=B.DQ_BUTTERFLY),
             dict(), dict(max_width=16, topology=B.DQ_BUTTERFLY)]


def allreduce_inputs(dev, calls, n=8, n_sg=2048):
    return [gradients(n, n_sg, torch.bfloat16, dev, 900 + k) for k in range(calls)]


@pytest.mark.parametrize("options", ALLREDUCE)
def test_allreduces_back_to_back_on_a_side_stream_keep_their_own_tables(dev, options):
    calls = allreduce_inputs(dev, 6)
    want = [allreduce.simulated_allreduce(g, 6.0, seed=k, **options)[0].clone() for k, g in enumerate(calls)]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    got = []
    with torch.cuda.stream(side):
        for k, g in enumerate(calls):                       # each call's scratch is the one before's
            got.append(allreduce.simulated_allreduce(g, 6.0, seed=k, **options)[0])
    side.synchronize()
    for k, (x, y) in enumerate(zip(got, want)):
        assert torch.equal(x.view(torch.int32), y.view(torch.int32)), f"call {k}"


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("topology,n,J,nb,bits,max_width", [
    ("ring", 2, 2, 1, 4.0, 8), ("ring", 3, 1023, 2, 5.0, 16), ("ring", 5, 1025, 1, 3.3, 8), ("ring", 8, 8192, 1, 4.6875, 8), ("ring", 61, 61, 3, 8.0, 16),
    ("ring", 7, 16387, 1, 5.0, 8), ("ring", 6, 20004, 2, 6.0, 16), ("ring", 64, 128, 16, 4.0, 8), ("ring", 64, 128, 17, 4.0, 8), ("ring", 256, 512, 1, 4.5, 8),
    ("ring", 257, 514, 1, 4.5, 8), ("ring", 4, 65536, 1, 3.0, 8), ("ring", 4, 65540, 1, 3.0, 8), ("ring", 2, 4, 500, 4.0, 8), ("ring", 2, 4, 512, 4.0, 8),
    ("butterfly", 2, 4096, 3, 5.5, 8), ("butterfly", 4, 4, 1, 3.0, 8), ("butterfly", 8, 8200, 1, 6.5, 16), ("butterfly", 16, 20656, 1, 4.3, 8),
    ("butterfly", 64, 4096, 2, 4.0, 16), ("butterfly", 128, 640, 1, 3.5, 8),
])
def test_an_allreduce_enqueued_whole_equals_its_steps(dev, monkeypatch, topology, n, J, nb, bits, max_width, dtype):
    """Rows of 1,024 and their remainders, one path to 1,024 (and the first sizes that go step by step: 1,025 paths, 257 tensors, 65,537 super-groups,
    512 buckets); all gathered or not, with means or without, norms alike and masses of equal ones."""
    J = J // n * n
    whole, enqueued = B.allreduce_whole, []

    def spy(*args):
        got = whole(*args)
        enqueued.append(got is not None)
        return got

    monkeypatch.setattr(B, "allreduce_whole", spy)
    for seed, spread in ((1, 3.0), (2, 0.0)):
        grads = gradients(n, J * nb, dtype, dev, seed + J)
        scale = torch.exp(spread * torch.randn(J * nb, 1, device=dev, generator=torch.Generator(dev).manual_seed(seed)))
        grads = [(g.reshape(-1, 256).float() * scale).to(dtype).reshape(-1).contiguous() for g in grads]
        if seed == 2:
            grads = [g.reshape(-1, 256)[:1].repeat(J * nb, 1).reshape(-1).contiguous() for g in grads]
        for options in ({"all_gather": True}, {"all_gather": False, "subtract_mean": False}):
            kw = dict(topology=TOPO[topology], seed=seed, n_sg_bucket=J, max_width=max_width, **options)
            got, info = allreduce.simulated_allreduce(grads, bits, **kw)
            want, parts = allreduce.simulated_allreduce(grads, bits, fused_reorder=False, **kw)
            assert info == parts
            assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    assert enqueued == [n <= 256 and n * nb <= 1024 and J <= 65536 and nb <= 511] * 4


@pytest.mark.parametrize("topology,n,J", [("ring", 8, 42664), ("ring", 3, 45057), ("butterfly", 2, 40960), ("ring", 7, 65534)])
def test_an_allreduce_of_listed_norms_enqueued_whole_equals_its_steps(dev, monkeypatch, topology, n, J):
    """Every block goes on from the rows' lists: a last row of one, of many and none behind the last list; norms alike and all equal."""
    test_an_allreduce_enqueued_whole_equals_its_steps(dev, monkeypatch, topology, n, J, 1, 4.2, 8, torch.bfloat16)


class Miscounted(list):
    """A list that another thread makes longer or shorter once its length has been asked for."""
    def __init__(self, items, count):
        super().__init__(items)
        self.count = count

    def __len__(self):
        return self.count


@pytest.mark.parametrize("topology", ["ring", "butterfly"])
@pytest.mark.parametrize("held,workers", [(2, 4), (3, 4), (5, 4), (8, 4), (4, 2), (7, 8)])
def test_a_whole_allreduce_takes_one_tensor_per_worker(dev, topology, held, workers):
    """Refused before anything is enqueued, as the steps refuse it."""
    J = 64
    grads = gradients(held, J, torch.bfloat16, dev, 5)
    assert B.allreduce_whole(B.Context(workers), grads, J, TOPO[topology], 4 * J, 8, True, True) is None
    with pytest.raises(B.DqError, match=f"{held} worker gradients for a context of {workers}"):
        allreduce.simulated_allreduce(Miscounted(grads, workers), 4.6875, topology=TOPO[topology])


def test_allreduces_of_several_threads_on_their_own_streams(dev):
    calls = allreduce_inputs(dev, len(ALLREDUCE))
    want = [allreduce.simulated_allreduce(g, 6.0, seed=k, **o)[0].clone() for k, (g, o) in enumerate(zip(calls, ALLREDUCE))]
    torch.cuda.synchronize()
    got, errors = [None] * len(calls), []

    def work(k):
        try:
            side = torch.cuda.Stream()
            with torch.cuda.stream(side):
                for _ in range(10):
                    got[k] = allreduce.simulated_allreduce(calls[k], 6.0, seed=k, **ALLREDUCE[k])[0]
            side.synchronize()
        except Exception as e:                              # noqa: BLE001 -- shown below
            errors.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(calls))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for k, (x, y) in enumerate(zip(got, want)):
        assert torch.equal(x.view(torch.int32), y.view(torch.int32)), f"thread {k}"


@pytest.mark.parametrize("codec,n,J", [(B.DQ_DYNAMIQ, 8, 64), (B.DQ_MXFP6_E3M2, 8, 64), (B.DQ_DYNAMIQ, 64, 192)])   # the last: 360 KB of tables
def test_a_plan_made_on_one_stream_runs_on_another_and_in_a_graph(dev, codec, n, J):
    grads = gradients(n, J, torch.bfloat16, dev, 7)
    ctx, widths = B.Context(n, seed=3), [[J // 4, J // 2, J // 4 - 8, 8]]
    ref = B.Replay(ctx, B.DQ_RING, codec, grads, J, widths)
    ref.run()
    torch.cuda.synchronize()
    want = ref.out.view(torch.int32).clone()
    side, busy = torch.cuda.Stream(), torch.randn(4096, 4096, device=dev)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(8):
            busy = busy @ busy * 1e-3                       # the upload has to wait for this
        rp = B.Replay(ctx, B.DQ_RING, codec, grads, J, widths)
        rp.out.zero_()
    torch.cuda.current_stream().wait_stream(side)           # for the zeros; the library sees to its tables itself
    rp.run()
    torch.cuda.synchronize()
    assert torch.equal(rp.out.view(torch.int32), want)

    with torch.cuda.stream(side):
        rp2 = B.Replay(ctx, B.DQ_RING, codec, grads, J, widths)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rp2.run()
    for _ in range(4):
        rp2.out.fill_(3.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(rp2.out.view(torch.int32), want)
        ref.run()                                           # eager work between the replays
        torch.cuda.synchronize()
        assert torch.equal(ref.out.view(torch.int32), want)


@pytest.mark.parametrize("how", ["run", "run_steps", "run_launch"])
def test_a_plan_dropped_while_another_stream_runs_it_keeps_its_scratch(dev, how):
    n, J = 8, 512
    inputs = [gradients(n, J, torch.bfloat16, dev, seed) for seed in (1, 2)]
    ctx = B.Context(n, seed=3)
    make = lambda k: B.Replay(ctx, B.DQ_RING, B.DQ_MXFP8_E4M3, inputs[k], J)   # noqa: E731
    ref = make(0)
    ref.run()
    torch.cuda.synchronize()
    want = ref.out.clone()
    side, busy = torch.cuda.Stream(), torch.randn(4096, 4096, device=dev)
    rp = make(0)
    out, scratch = rp.out, rp.scratch.data_ptr()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(8):
            busy = busy @ busy * 1e-3                       # the replay has to wait for this
        if how == "run":
            rp.run()
        elif how == "run_steps":
            rp.run_steps(0, rp.n_steps - 1)
            rp.run_steps(rp.n_steps - 1, 1)
        else:
            for t in range(rp.n_steps):
                rp.run_launch(t, 0)
    rp.close()
    del rp
    others = [make(1) for _ in range(3)]
    assert all(x.scratch.data_ptr() != scratch for x in others)
    for x in others:
        x.run()
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int32), want.view(torch.int32))


def test_a_plan_is_not_made_under_capture(dev):
    grads = gradients(4, 16, torch.bfloat16, dev, 1)
    ctx = B.Context(4)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        with pytest.raises(B.DqError, match="captur"):
            B.Replay(ctx, B.DQ_RING, B.DQ_DYNAMIQ, grads, 16, [[4, 8, 4, 0]])
        grads[0].zero_()                                    # a graph with something in it
    graph.replay()
    torch.cuda.synchronize()


def test_other_threads_run_while_a_call_enqueues(dev):
    """Thousands of launches in one call: they wait for the queue, and the interpreter is free meanwhile."""
    n = 6000
    g = gradients(1, 4, torch.bfloat16, dev, 1)[0]
    rp = B.Replay(B.Context(n), B.DQ_CHAIN, B.DQ_DYNAMIQ, [g] * n, 4, [[1, 2, 1, 0]])
    rp.run_steps(0, 2)
    torch.cuda.synchronize()
    ticks, stop = [], threading.Event()

    def tick():
        while not stop.is_set():
            ticks.append(time.perf_counter())
            time.sleep(0.0002)

    t = threading.Thread(target=tick)
    t.start()
    time.sleep(0.01)
    begin = time.perf_counter()
    rp.run_steps(0, n - 1)                                  # not the whole schedule: step by step
    end = time.perf_counter()
    stop.set()
    t.join()
    torch.cuda.synchronize()
    assert end - begin > 0.005 and sum(begin < x < end for x in ticks) >= 5, (end - begin, len(ticks))


@pytest.mark.parametrize("codec", [B.DQ_DYNAMIQ, B.DQ_MXFP8_E4M3])
@pytest.mark.parametrize("topology,n,all_gather", [("ring", 5, False), ("ring", 4, True), ("chain", 6, True), ("butterfly", 8, False),
                                                   ("butterfly", 16, True), ("butterfly", 2, True)])
def test_steps_continue_from_a_whole_replay(dev, topology, n, all_gather, codec):
    """Steps, and launches of a step, after a whole replay meet the state that the same replay run step by step leaves:
    not messages and keep-buffers of an older run on other inputs."""
    J = 3 * n
    inputs = [gradients(n, J, torch.bfloat16, dev, seed) for seed in (1, 2)]
    widths = [[J // 3, J // 3, J // 3, 0]]

    def play(whole, continue_with):
        grads = [g.clone() for g in inputs[0]]
        rp = B.Replay(B.Context(n, seed=3), TOPO[topology], codec, grads, J, widths, all_gather=all_gather)

        def steps():
            for t in range(rp.n_steps):
                rp.run_steps(t, 1)
        steps()
        for g, x in zip(grads, inputs[1]):
            g.copy_(x)
        rp.run() if whole else steps()
        if continue_with == "launches":
            kinds = [rp.step_info(t)[0] for t in range(rp.n_steps)]
            for t in range(1, rp.n_steps):
                for launch in range(2 if kinds[t] == 3 else 1):
                    rp.run_launch(t, launch)
        else:
            for first, count in continue_with:
                rp.run_steps(first, count)
        torch.cuda.synchronize()
        return rp.out.view(torch.int32).clone()

    ns = {"ring": n, "chain": n, "butterfly": n.bit_length()}[topology] + (2 if all_gather else 0)
    plays = [[(k, ns - k)] for k in range(1, ns)] + [[(0, 1), (ns - 1, 1)], [(0, 2), (2, ns - 2)], [(ns - 1, 1), (ns - 1, 1)], "launches"]
    if all_gather:
        plays += [[(ns - 2, 1), (ns - 1, 1)], [(1, 1), (ns - 1, 1)]]
    for continue_with in plays:
        if continue_with != "launches" and any(c < 1 or f < 1 and c == ns for f, c in continue_with):
            continue
        assert torch.equal(play(True, continue_with), play(False, continue_with)), continue_with


@pytest.mark.parametrize("topology,n,widths,dtype", [
    # wide trees, whose tile size follows an estimate: each size of tile, several rounds of tiles per wave
    ("butterfly", 32, [[300, 2500, 900, 396]], torch.bfloat16), ("butterfly", 128, [[201, 1500, 300, 47]], torch.float32),
    ("butterfly", 128, [[1001, 5002, 2003, 186]], torch.bfloat16), ("butterfly", 256, [[511, 1025, 400, 112]], torch.bfloat16),
    ("butterfly", 256, [[0, 5000, 2900, 292]], torch.float32), ("butterfly", 64, [[3201, 9003, 900, 80]], torch.bfloat16),
    ("ring", 256, [[257, 513, 200, 54]], torch.float32), ("ring", 256, [[1025, 4097, 1900, 146]], torch.bfloat16),
    ("chain", 200, [[1501, 4003, 2707, 302]], torch.bfloat16),
    # raw chunks of so many workers that the stacks of eight waves do not fit a CU
    ("butterfly", 1024, [[4000, 4000, 4000, 1312]], torch.bfloat16),
])
def test_whole_replay_of_many_workers_equals_its_steps(dev, topology, n, widths, dtype):
    J = sum(widths[0])
    assert topology == "chain" or J % n == 0
    grads = gradients(8, J, dtype, dev, n + J)
    rp = B.Replay(B.Context(n, seed=n), TOPO[topology], B.DQ_DYNAMIQ, [grads[(3 * w + w // 8) % 8] for w in range(n)], J, widths, all_gather=True,
                  mu=torch.randn(J, device=dev) * 1e-4)
    whole_against_steps(rp, {"ring": n, "chain": 1, "butterfly": 0}[topology])


def test_calls_on_the_default_stream_while_another_thread_captures(dev):
    n_sg, ctx = 300, B.Context(4, seed=1)
    ch = B.make_chunk(0, [0, n_sg, 0])
    x = gradients(1, n_sg, torch.bfloat16, dev, 8)[0]
    index = torch.arange(n_sg - 1, -1, -1, dtype=torch.int32, device=dev)
    want, plain = ctx.dq_compress(x, ch, 1, sg_index=index), ctx.dq_compress(x, ch, 1)
    out, errors = torch.zeros_like(want), []
    torch.cuda.synchronize()

    def work():
        try:
            for _ in range(5):
                ctx.dq_compress(x, ch, 1, packed_out=out, sg_index=index)
        except Exception as e:                              # noqa: BLE001 -- shown below
            errors.append(e)

    graph = torch.cuda.CUDAGraph()
    got = torch.zeros_like(plain)
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        ctx.dq_compress(x, ch, 1, packed_out=got)
        t = threading.Thread(target=work)
        t.start()
        t.join()
        ctx.dq_compress(x, ch, 1, packed_out=got)
    assert not errors, errors
    assert torch.equal(out, want)
    for _ in range(3):
        got.zero_()
        graph.replay()
        assert torch.equal(got, plain)


def test_a_pipelined_hop_orders_and_keeps_the_buffers_it_makes(dev):
    n_sg = [300, 411, 200, 90]
    ctx, ch = B.Context(8, seed=21), B.make_chunk(5000, n_sg)
    x = gradients(1, sum(n_sg), torch.bfloat16, dev, 4)[0]
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    want = B.dq_dar_hop_pipelined(ctx, None, x, ch, 0, 96, s1, s2)
    torch.cuda.synchronize()
    want, busy = want.clone(), torch.randn(4096, 4096, device=dev)
    torch.cuda.synchronize()
    for _ in range(8):
        busy = busy @ busy * 1e-3                           # the zeros of stage and wire wait behind this
    got = B.dq_dar_hop_pipelined(ctx, None, x, ch, 0, 96, s1, s2)
    spoil = [torch.full((B.dq_pipelined_stage_bytes(ch, 96),), 255, dtype=torch.uint8, device=dev) for _ in range(4)]
    torch.cuda.synchronize()
    assert torch.equal(got, want) and len(spoil) == 4
