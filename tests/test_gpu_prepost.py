"""HIP path of the steps before and after the main stage against the CPU oracle
(oracle/pp_oracle.c), through the C ABI.  Each stage gets the oracle's output of the stage
before it (never the other way round): statistics within the tolerance of fp32 accumulation
against the float64 definition, everything that is an integer decision or a single rounded
operation bit-exactly."""
import ctypes
import math

import numpy as np
import pytest
import torch

from oracle import pp_oracle as P
from paper_2602_08923_amd import binding as B
from paper_2602_08923_amd import prep, workloads

pytestmark = pytest.mark.gpu
f32 = np.float32


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def host(t):
    return t.detach().cpu().numpy()


def draw(cfg, worker, entries, bucket=0):
    return workloads.draw(workloads.CONFIGS[cfg], worker, bucket, device="cpu", entries=entries)


def as_np(t):
    return workloads.to_numpy(t)


def lognormal_F(seed, J, zeros=0, ties=0):
    rng = np.random.default_rng(seed)
    F = np.exp(rng.normal(-14, 2.5, J)).astype(f32)
    if zeros:
        F[rng.integers(0, J, zeros)] = 0
    if ties:
        F[rng.integers(0, J, ties)] = F[0]
    return F


# ---------------------------------------------------------------- statistics
@pytest.mark.parametrize("cfg,n_sg", [(1, 1), (1, 5), (2, 1027), (4, 4096), (5, 2049)])
def test_sg_stats(dev, cfg, n_sg):
    x = draw(cfg, 3, n_sg * 256)
    mu64, F64 = P.sg_stats(as_np(x))
    mu, F = B.dq_sg_stats(x.to(dev))
    mu, F = host(mu).astype(np.float64), host(F).astype(np.float64)
    # 16 sequential + 4 tree additions in fp32: relative error below 20 * 2^-24 of the sum of magnitudes
    tol = 20 * 2.0 ** -24
    assert np.all(np.abs(F - F64) <= tol * F64 + 1e-45)
    mean_abs = np.abs(x.double().numpy().reshape(n_sg, 256)).sum(axis=1) / 256
    assert np.all(np.abs(mu - mu64) <= tol * mean_abs + 1e-45)
    assert np.all(F64 > 0)


def test_sg_stats_exact_cases(dev):
    c = 0.375
    x = np.concatenate([np.full(256, c), np.tile([0.5, -0.5], 128), np.arange(256) * 2.0 ** -10, np.zeros(256)]).astype(f32)
    for t in (torch.from_numpy(x), torch.from_numpy(x).to(torch.bfloat16)):      # all values are bf16-exact
        mu, F = B.dq_sg_stats(t.to(dev))
        assert host(mu).tolist() == [c, 0.0, 127.5 * 2.0 ** -10, 0.0]
        assert host(F).tolist() == [256 * c * c, 64.0, 5559680 * 2.0 ** -20, 0.0]
    mu, F = B.dq_sg_stats(torch.empty(0, dtype=torch.float32, device=dev))       # empty input
    assert mu.numel() == 0 and F.numel() == 0


@pytest.mark.parametrize("dtype,n,J", [("bf16", 5, 1), ("bf16", 6, 3), ("bf16", 16, 4093), ("bf16", 17, 1027), ("bf16", 21, 2815), ("bf16", 256, 6),
                                       ("bf16", 40, 5633), ("f32", 5, 1789), ("f32", 19, 3585), ("f32", 33, 18), ("f32", 3, 500)])
def test_stats_of_workers_is_stats_and_combination(dev, dtype, n, J):
    """A wave per worker and tile, per several workers, or per tile: the same bits as every worker's statistics, then their combination."""
    gen = torch.Generator(device=dev)
    gen.manual_seed(n * 10007 + J)
    x = torch.randn(n, J * 256, generator=gen, device=dev).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    want = B.dq_stats_combine(*(torch.stack(t) for t in zip(*(B.dq_sg_stats(w) for w in x))))
    for g, w in zip(B.stats_of_workers(x.unbind(0)), want):
        assert torch.equal(g, w)


def test_stats_combine(dev):
    n, J = 8, 3001
    xs = [draw(2, w, J * 256) for w in range(n)]
    st = [P.sg_stats(as_np(x)) for x in xs]
    mu_all = np.array([s[0] for s in st], f32)
    F_all = np.array([s[1] for s in st], f32)
    want_mu, want_F = P.stats_combine(mu_all, F_all)
    mu, F = B.dq_stats_combine(torch.from_numpy(mu_all).to(dev), torch.from_numpy(F_all).to(dev))
    assert np.array_equal(host(mu).view(np.uint32), want_mu.view(np.uint32))
    assert np.array_equal(host(F).view(np.uint32), want_F.view(np.uint32))
    # n = 1 and a worker count that is not a power of two (the division is rounded, not a shift)
    for k in (1, 3):
        want_mu, want_F = P.stats_combine(mu_all[:k], F_all[:k])
        mu, F = B.dq_stats_combine(torch.from_numpy(mu_all[:k].copy()).to(dev), torch.from_numpy(F_all[:k].copy()).to(dev))
        assert np.array_equal(host(mu).view(np.uint32), want_mu.view(np.uint32))
        assert np.array_equal(host(F).view(np.uint32), want_F.view(np.uint32))


# ---------------------------------------------------------------- allocation
def check_allocate(dev, F, J, budget, max_width=8):
    nb = F.size // J
    widths, pos, counts = B.dq_allocate(torch.from_numpy(F).to(dev), J, budget, max_width=max_width)
    widths, pos, counts = host(widths), host(pos).view(np.uint32), host(counts).view(np.uint32)
    for b in range(nb):
        w, tbits = P.allocate(F[b * J:(b + 1) * J], budget, max_width=max_width)
        p, c = P.positions(w)
        assert np.array_equal(widths[b * J:(b + 1) * J], w), f"bucket {b}"
        assert np.array_equal(pos[b * J:(b + 1) * J], p), f"bucket {b}"
        assert counts[b].tolist() == c + [tbits], f"bucket {b}"
    return counts


@pytest.mark.parametrize("J", [1, 7, 64, 1000, 1024, 1025, 51200, 65536])
@pytest.mark.parametrize("bits", [3.0, 5.0])
def test_allocate_sizes(dev, J, bits):
    F = lognormal_F(J, J, zeros=min(J // 10, 50), ties=min(J // 7, 40))
    check_allocate(dev, F, J, int(math.floor(prep.code_bits(bits) * J)))


@pytest.mark.parametrize("J", [1, 64, 1025, 51200, 70000])
@pytest.mark.parametrize("bits", [5.0, 8.5, 12.0])
def test_allocate_with_sixteen_bit_class(dev, J, bits):
    F = lognormal_F(J + 1, J, zeros=min(J // 10, 50), ties=min(J // 7, 40))
    c = check_allocate(dev, F, J, int(math.floor(prep.code_bits(bits) * J)), max_width=16)
    if J >= 1025 and bits >= 8.5:
        assert c[0][3] > 0                       # some super-groups do get 16 bits


def test_allocate_many_buckets_full_size(dev):
    """config 4's shape: 100 buckets of 51,200 super-groups, one block per bucket."""
    J, nb = 51200, 100
    rng = np.random.default_rng(4)
    F = np.concatenate([np.exp(rng.normal(rng.uniform(-20, -8), rng.uniform(0.5, 3.0), J)) for _ in range(nb)]).astype(f32)
    counts = check_allocate(dev, F, J, int(math.floor(prep.code_bits(3.0) * J)))
    assert len({tuple(c[:3]) for c in counts.tolist()}) > 50


def test_allocate_beyond_register_capacity(dev):
    J = 65536 + 4321                                   # runs no longer fit 64 registers per thread
    F = lognormal_F(99, 2 * J, zeros=100, ties=100)
    check_allocate(dev, F, J, int(math.floor(prep.code_bits(4.0) * J)))


@pytest.mark.parametrize("bits", [2.8, 4.0, 6.0, 8.5])
def test_allocate_masses_of_equal_values(dev, bits):
    """More equal norms than the kernel keeps as candidates of its narrowed search: it must fall
    back to counting everything and still agree."""
    J = 51200
    F = lognormal_F(21, J)
    F[5000:35000] = F[7]                      # 30,000 equal values
    F[40000:46000] = np.float32(F[7] * np.float32(17.0 / 512.0))   # and 6,000 at the tied lower threshold
    check_allocate(dev, F, J, int(math.floor(prep.code_bits(bits) * J)))
    check_allocate(dev, np.full(J, 3.25e-7, f32), J, int(math.floor(prep.code_bits(bits) * J)))


def test_allocate_narrow_value_ranges(dev):
    """Norms one bit pattern apart around the threshold, two distinct values tied by the threshold
    ratio, several small buckets per call."""
    J = 20000
    base = np.float32(1.5e-3)
    pat = base.view(np.uint32) + np.arange(J, dtype=np.uint32) % 300          # 300 neighbouring patterns
    F = pat.view(f32).copy()
    for bits in (2.8, 4.0, 7.0):
        check_allocate(dev, F, J, int(math.floor(prep.code_bits(bits) * J)))
    F2 = np.where(np.arange(J) % 3 == 0, np.float32(2.0), np.float32(2.0 * 17.0 / 512.0)).astype(f32)
    for bits in (2.8, 3.5, 4.0, 6.0):
        check_allocate(dev, F2, J, int(math.floor(prep.code_bits(bits) * J)))
        check_allocate(dev, F2, J, int(math.floor(prep.code_bits(bits) * J)), max_width=16)
    F3 = lognormal_F(8, 3 * 4097)
    check_allocate(dev, F3, 4097, int(math.floor(prep.code_bits(4.0) * 4097)))   # 3 buckets, 5 rows each, ragged


@pytest.mark.parametrize("J,nb", [(1, 3), (1024, 300), (1025, 128), (1025, 129), (16384, 16), (16384, 17), (15361, 2), (40000, 6), (65536, 4)])
@pytest.mark.parametrize("max_width", [8, 16])
def test_allocate_where_every_row_searches(dev, J, nb, max_width):
    """One launch for two rows and more while there is a CU for every row of every bucket; a search and its positions for one row, and beyond; at 40,960 and more
    and up to 8 bits lists (which launches these are: test_allocation_launches.py)."""
    F = np.concatenate([lognormal_F(J + b, J, ties=min(J // 7, 40)) for b in range(nb)])
    check_allocate(dev, F, J, int(math.floor(prep.code_bits(4.0 if max_width == 8 else 7.0) * J)), max_width=max_width)


@pytest.mark.parametrize("J", [16384, 16385, 51200, 65536])       # from 16,385 on the search sets norms aside, up to 15 per thread
@pytest.mark.parametrize("max_width", [8, 16])
def test_allocate_at_the_edges_of_what_is_set_aside(dev, J, max_width):
    """Few norms around the threshold, but one thread (norms 4096 g + 4 t + 0..3) has 13 to 16 of its own there."""
    rng = np.random.default_rng(J)
    spread = np.exp(rng.normal(-14, 6, J)).astype(f32)
    budget = int(math.floor(prep.code_bits(4.0) * J))
    T = P.allocate(spread, budget, max_width=max_width)[1]
    for t in (0, 1, 1023):
        own = [j for j in range(J) if j % 4096 // 4 == t]
        for m in (13, 14, 15, 16):
            F = spread.copy()
            F[own[:m]] = (T + 3 * np.arange(m, dtype=np.uint32)).astype(np.uint32).view(f32)
            check_allocate(dev, F, J, budget, max_width=max_width)


@pytest.mark.parametrize("J", [3, 63, 1025, 8192, 16385, 65536])
@pytest.mark.parametrize("max_width", [8, 16])
@pytest.mark.parametrize("kind", ["patterns", "denormals", "infinities", "steps", "narrow"])
def test_allocate_any_patterns(dev, J, max_width, kind):
    """Thresholds in every range of the format: where the tied ones are denormal or infinite, many patterns to one, a bin apart or in one bin."""
    rng = np.random.default_rng(J)
    if kind == "patterns":        # the whole range, evenly over the patterns
        pat = rng.integers(0, 0x7F800000, J, dtype=np.uint32)
    elif kind == "denormals":     # on both sides of the smallest normal, and its 512/17 and 257/131072
        pat = rng.integers(0, 0x00800000 << rng.integers(0, 4), J, dtype=np.uint32) >> rng.integers(0, 24, J, dtype=np.uint32)
    elif kind == "infinities":
        pat = np.where(rng.random(J) < 0.3, 0x7F800000, rng.integers(0x7A000000, 0x7F800000, J)).astype(np.uint32)
    elif kind == "narrow":        # masses a few thousand patterns wide, tied by the ratios
        values = np.float32(0.7) * np.float32([1.0, 17 / 512, 131072 / 257])
        pat = rng.choice(values.view(np.uint32), J) + rng.integers(0, 1 << rng.integers(0, 13), J, dtype=np.uint32)
    else:                         # a few values tied by the ratios, one pattern below, at and above
        values = np.float32(1e-4) * np.float32([1.0, 512 / 17, 17 / 512, 257 / 131072, (17 / 512) ** 2])
        pat = rng.choice(values.view(np.uint32), J) + rng.integers(0, 3, J, dtype=np.uint32) - 1
    F = pat.astype(np.uint32).view(f32)
    for bits in (2, 3, 4, 6, 8, 15):
        for budget in (bits * J, bits * J + 1):
            if kind == "infinities" and budget < 2 * J + (6 if max_width == 8 else 14) * int(np.isinf(F).sum()):
                counts = host(B.dq_allocate(torch.from_numpy(F).to(dev), J, budget, max_width=max_width)[2]).view(np.uint32)
                assert counts[0][4] == 0x7F800000      # not even +infinity fits: the allocation is that of +infinity
            else:
                check_allocate(dev, F, J, budget, max_width=max_width)


@pytest.mark.parametrize("J", [3, 100, 9000, 16385, 65536])
@pytest.mark.parametrize("max_width", [8, 16])
@pytest.mark.parametrize("share", [0.02, 0.5, 0.999])
def test_allocate_when_not_even_infinity_fits(dev, J, max_width, share):
    """Infinite norms are all above any threshold: the allocation is that of +infinity, whatever it costs."""
    rng = np.random.default_rng(J)
    pat = np.where(np.arange(J) < max(1, int(share * J)), 0x7F800000, rng.integers(0x7F000000, 0x7F800000, J)).astype(np.uint32)
    F = rng.permutation(pat).view(f32)
    for budget in (2 * J, 2 * J + 1, 2 * J + 5):
        widths, pos, counts = B.dq_allocate(torch.from_numpy(F).to(dev), J, budget, max_width=max_width)
        w = np.where(np.isinf(F), max_width, 2).astype(np.uint8)
        p, c = P.positions(w)
        assert np.array_equal(host(widths), w) and np.array_equal(host(pos).view(np.uint32), p)
        assert host(counts).view(np.uint32)[0].tolist() == c + [0x7F800000]


@pytest.mark.parametrize("J", [1, 2, 5, 8, 9, 11, 100, 8191, 8192, 8193, 16383, 16384])
@pytest.mark.parametrize("max_width", [8, 16])
def test_allocate_norms_close_together(dev, J, max_width):
    """Up to 8,192 norms around the threshold the levels take as they are, more the search halves away first: equal ones, and ones within a tenth and a factor of two."""
    rng = np.random.default_rng(J)
    for F in (np.full(J, 3.0), 1.0 + 0.1 * rng.random(J), 1.0 + rng.random(J)):
        for bits in (2.0, 3.3, 4.7, 7.9, 13.0):
            check_allocate(dev, F.astype(f32), J, int(bits * J), max_width=max_width)


@pytest.mark.parametrize("J", [32767, 32768, 33791, 40959, 40960, 41983, 65535, 65536])   # below and from where rows list their norms; whole rows and a rest
@pytest.mark.parametrize("kind", ["random", "sorted", "dense_end", "clustered", "aliased", "equal", "half"])
def test_allocate_from_lists(dev, J, kind):
    """Rows list the norms around a threshold that a sample brackets: lists longer than what is asked for ahead, longer than their place (in the last row
    with what follows it, too), too many of those, and samples that are beside the mark."""
    rng = np.random.default_rng(J)
    F = np.exp(rng.normal(-14, 2.5, 2 * J)).astype(f32)
    if kind == "sorted":
        F = np.sort(F)
    elif kind == "dense_end":         # the norms around the threshold in the last row and behind it
        F = F.reshape(2, J)
        F[:, J - 1800:] = np.exp(rng.normal(-12.5, 0.2, (2, 1800)))
        F = F.reshape(-1)
    elif kind == "clustered":         # a few rows each hold most of what is near the threshold
        F = (np.exp(rng.normal(-14, 2.5, 2 * J // 512 + 1)).repeat(512)[:2 * J] * np.exp(rng.normal(0, 0.05, 2 * J))).astype(f32)
    elif kind == "aliased":           # the sampled norms are unlike the others
        at = np.arange(8192, dtype=np.int64) * J // 8192
        F[at] *= f32(1e-6)
        F[J + at] *= f32(1e6)
    elif kind == "equal":
        F = np.full(2 * J, 3.25e-7, f32)
    elif kind == "half":
        F[::2] = 0
    for bits in (2.1, 4.0, 7.5):
        check_allocate(dev, F, J, int(bits * J))


@pytest.mark.parametrize("J,nb", [(40960, 1), (41983, 2), (65536, 4)])
def test_allocate_without_memory_for_lists(dev, J, nb):
    """The C entry, whose rows list their norms where the positions go: the same as the binding's, whose lists have memory of their own."""
    F = torch.from_numpy(lognormal_F(J, J * nb, ties=40)).to(dev)
    want = B.dq_allocate(F, J, 4 * J)
    got = [torch.empty_like(w) for w in want]
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert B.lib().dq_allocate(F.data_ptr(), J, nb, 4 * J, 8, *(g.data_ptr() for g in got), stream) == 0
    for g, w in zip(got, want):
        assert torch.equal(g, w)


@pytest.mark.parametrize("J,nb,max_width", [(1, 1, 8), (1025, 2, 8), (16385, 3, 16), (30000, 1, 8), (41983, 2, 8), (65537, 1, 8)])
def test_allocate_beside_other_work(dev, J, nb, max_width):
    """Fewer blocks, the same bits; the counts that are sent ahead, too."""
    F = torch.from_numpy(lognormal_F(J, J * nb, ties=min(J // 7, 40))).to(dev)
    want = B.dq_allocate(F, J, 4 * J, max_width=max_width)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        plain = B.dq_allocate(F, J, 4 * J, max_width=max_width, beside=True)
        *ahead, by_width = B.allocate_ahead(F, J, 4 * J, max_width=max_width, beside=True)
        assert by_width() == [row[:4] for row in want[2].cpu().tolist()]
    side.synchronize()
    for got in (plain, ahead):
        for g, w in zip(got, want):
            assert torch.equal(g, w)


def test_allocate_from_lists_in_a_graph(dev):
    """The lists' memory is free again within the capture, and what is captured next takes it: every replay, with the program's own work in between, is as the call itself."""
    J, nb = 41983, 2
    F = torch.from_numpy(lognormal_F(J, J * nb, ties=40)).to(dev)
    B.dq_allocate(F, J, 4 * J)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = B.dq_allocate(F, J, 4 * J)
        filled = torch.full((J * nb,), -1, dtype=torch.int32, device=dev)
        beside = B.dq_allocate(F, J, 4 * J, beside=True)
    for replay in range(3):
        F.copy_(torch.from_numpy(lognormal_F(J + replay, J * nb, ties=7)))
        graph.replay()
        want = B.dq_allocate(F, J, 4 * J)
        torch.cuda.synchronize()
        assert bool((filled == -1).all())
        for g, b, w in zip(got, beside, want):
            assert torch.equal(g, w) and torch.equal(b, w)


def test_allocate_more_buckets_than_a_grid_dimension(dev):
    """70,000 buckets of 5 super-groups: the positions launch is cut at 65,535 buckets (the grid's second
    dimension); buckets on both sides of the cut must come out right."""
    J, nb = 5, 70000
    F = lognormal_F(17, J * nb)
    budget = 4 * J + 2
    widths, pos, counts = B.dq_allocate(torch.from_numpy(F).to(dev), J, budget)
    widths, pos, counts = host(widths), host(pos).view(np.uint32), host(counts).view(np.uint32)
    for b in list(range(0, nb, 997)) + [65534, 65535, 65536, nb - 1]:
        w, tbits = P.allocate(F[b * J:(b + 1) * J], budget)
        p, c = P.positions(w)
        assert np.array_equal(widths[b * J:(b + 1) * J], w), f"bucket {b}"
        assert np.array_equal(pos[b * J:(b + 1) * J], p), f"bucket {b}"
        assert counts[b].tolist() == c + [tbits], f"bucket {b}"


def test_allocate_budget_edges(dev):
    F = lognormal_F(5, 2000)
    c = check_allocate(dev, F, 2000, 2 * 2000)                       # exactly 2 bits each
    assert c[0][:3].tolist() == [2000, 0, 0]
    c = check_allocate(dev, F, 2000, 8 * 2000 + 5)                   # everything fits
    assert c[0][:3].tolist() == [0, 0, 2000] and c[0][4] == 1
    c = check_allocate(dev, np.zeros(512, f32), 512, 3 * 512)        # an all-zero bucket
    assert c[0][:3].tolist() == [512, 0, 0]
    with pytest.raises(B.DqError):
        B.dq_allocate(torch.from_numpy(F).to(dev), 2000, 3999)       # below 2 bits per coordinate


# ---------------------------------------------------------------- reorder / restore
@pytest.mark.parametrize("J,nb,max_width", [(1, 1, 8), (1000, 3, 16), (65536, 1, 8), (65536, 2, 16), (65537, 1, 8), (4, 511, 16), (4, 512, 8)])
def test_counts_ahead_of_the_allocation_are_its_counts(dev, J, nb, max_width):
    """The largest counts that fit 17 bits and one beyond, the most buckets that a workspace holds and one beyond; asked for once, twice,
    late and never, on one workspace after the other."""
    F = torch.from_numpy(np.concatenate([lognormal_F(7 * b + 1, J) for b in range(nb)])).to(dev)
    for bits in (2, 3, 16) if max_width == 16 else (2, 3, 8):   # all of the narrowest, some of each, all of the widest
        want = [[int(v) for v in row[:4]] for row in B.dq_allocate(F, J, bits * J, max_width=max_width)[2].cpu().tolist()]
        widths, pos, counts, by_width = B.allocate_ahead(F, J, bits * J, max_width=max_width)
        B.allocate_ahead(F, J, bits * J, max_width=max_width)
        late = B.allocate_ahead(F, J, 2 * J, max_width=max_width)[3]
        assert by_width() == want and by_width() == want
        torch.cuda.synchronize()
        assert late() == [[J, 0, 0, 0]] * nb
        assert [[int(v) for v in row[:4]] for row in counts.cpu().tolist()] == want
    with pytest.raises(B.DqError):
        B.allocate_ahead(F, J, 2 * J - 1, max_width=max_width)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("J,nb", [(1, 1), (37, 3), (1030, 2)])
def test_reorder_and_restore(dev, dtype, J, nb):
    n_sg = J * nb
    x = draw(2 if dtype == "bf16" else 1, 1, n_sg * 256)
    rng = np.random.default_rng(J)
    widths = rng.choice(np.array([2, 4, 8, 16], np.uint8), n_sg, p=[0.4, 0.3, 0.2, 0.1])
    pc = [P.positions(widths[b * J:(b + 1) * J]) for b in range(nb)]
    pos = np.concatenate([p for p, _ in pc])
    counts = np.array([c + [0] for _, c in pc], np.int32)                  # [nb, 5] as dq_allocate writes it
    mu = (rng.standard_normal(n_sg) * 1e-4).astype(f32)
    xn = as_np(x)
    pos_t = torch.from_numpy(pos.view(np.int32)).to(dev)
    want = np.concatenate([P.reorder(xn[b * J * 256:(b + 1) * J * 256], pos[b * J:(b + 1) * J]) for b in range(nb)])
    got = B.dq_reorder(x.to(dev), pos_t, J)
    assert np.array_equal(as_np(got.cpu()), want)
    # the means of the main stage: reordered, zero for the 16-bit super-groups; without counts: all kept
    for cnt in (counts, None):
        want_mm = np.concatenate([P.reorder_mean(mu[b * J:(b + 1) * J], pos[b * J:(b + 1) * J],
                                                 0 if cnt is None else cnt[b][3]) for b in range(nb)])
        got_mm = B.dq_reorder_mean(torch.from_numpy(mu).to(dev), pos_t, J,
                                   None if cnt is None else torch.from_numpy(cnt).to(dev))
        assert np.array_equal(host(got_mm).view(np.uint32), want_mm.view(np.uint32))
    # the inverse of the positions, alone and together with the means
    inv = np.concatenate([np.argsort(pos[b * J:(b + 1) * J]) for b in range(nb)]).astype(np.int32)
    _, origin = B.dq_reorder_mean(None, pos_t, J, with_origin=True)
    assert np.array_equal(host(origin), inv)
    mm2, origin2 = B.dq_reorder_mean(torch.from_numpy(mu).to(dev), pos_t, J, with_origin=True)
    assert np.array_equal(host(origin2), inv) and np.array_equal(host(mm2).view(np.uint32), want_mm.view(np.uint32))
    total = (rng.standard_normal(n_sg * 256) * 1e-2).astype(f32)
    for m in (want_mm, None):
        want = np.concatenate([P.restore(total[b * J * 256:(b + 1) * J * 256], pos[b * J:(b + 1) * J],
                                         None if m is None else m[b * J:(b + 1) * J], 8) for b in range(nb)])
        got = B.dq_restore(torch.from_numpy(total).to(dev), pos_t, J, 8,
                           mu_main=None if m is None else torch.from_numpy(m).to(dev))
        assert np.array_equal(host(got).view(np.uint32), want.view(np.uint32))


def test_reorder_full_bucket(dev):
    """One worker's whole config-2 bucket (13,107,200 bf16 entries), allocation from the oracle."""
    wl = workloads.CONFIGS[2]
    J = wl.entries // 256
    x = workloads.draw(wl, 0, 0, device="cpu")
    mu64, F64 = P.sg_stats(as_np(x))
    mu, F = P.stats_combine(mu64.astype(f32)[None], (8 * F64).astype(f32)[None])
    w, _ = P.allocate(F, int(math.floor(prep.code_bits(wl.budget_bits) * J)))
    pos, counts = P.positions(w)
    assert counts[0] > 0 and counts[1] > 0
    pos_t = torch.from_numpy(pos.view(np.int32)).to(dev)
    got = B.dq_reorder(x.to(dev), pos_t, J)
    assert np.array_equal(as_np(got.cpu()), P.reorder(as_np(x), pos))
    mm = P.reorder_mean(mu, pos, 0)
    got_mm = B.dq_reorder_mean(torch.from_numpy(mu).to(dev), pos_t, J)
    assert np.array_equal(host(got_mm).view(np.uint32), mm.view(np.uint32))
    total = got.float()
    back = B.dq_restore(total, pos_t, J, 1, mu_main=got_mm)
    assert np.array_equal(host(back).view(np.uint32), P.restore(host(total), pos, mm, 1).view(np.uint32))
    # the permutation alone is undone exactly
    assert torch.equal(B.dq_restore(total, pos_t, J, 1).cpu(), x.float())


def test_rejects_bad_arguments(dev):
    x = torch.zeros(512, dtype=torch.float32, device=dev)
    pos = torch.zeros(2, dtype=torch.int32, device=dev)
    L = B.lib()
    st = L.dq_reorder(B._ptr(x), 0, B._ptr(pos), 2, 1, B._ptr(x), None)               # in place
    assert st == B.DQ_EINVAL
    st = L.dq_reorder(x.data_ptr() + 4, 0, B._ptr(pos), 2, 1, B._ptr(torch.empty_like(x)), None)
    assert st == B.DQ_EALIGN
    mu = torch.zeros(2, dtype=torch.float32, device=dev)
    st = L.dq_reorder_mean(B._ptr(mu), B._ptr(pos), None, 2, 1, B._ptr(mu), None, None)     # in place
    assert st == B.DQ_EINVAL
    st = L.dq_reorder_mean(B._ptr(mu), B._ptr(pos), None, 2, 1, None, None, None)           # no output asked for
    assert st == B.DQ_EINVAL
    st = L.dq_restore(B._ptr(x), B._ptr(pos), None, 0, 2, 1, B._ptr(torch.empty_like(x)), None)   # n = 0
    assert st == B.DQ_EINVAL
    st = L.dq_sg_stats(B._ptr(x), 7, 2, B._ptr(x), B._ptr(x), None)                  # unknown dtype
    assert st == B.DQ_EINVAL


def test_whole_pipeline_is_consistent(dev):
    """statistics -> combine -> allocate -> reorder -> ring reduce-scatter -> restore, all on the GPU:
    the allocation meets its budget with larger norms never getting fewer bits, and the restored
    result estimates the true sum."""
    wl = workloads.CONFIGS[2]
    n, J = 8, 4096
    xs = [workloads.draw(wl, w, 0, device=dev, entries=J * 256) for w in range(n)]
    xs[3][:256] += 0.5                                                   # a super-group with a large mean
    st = [B.dq_sg_stats(x) for x in xs]
    mu, F = B.dq_stats_combine(torch.stack([s[0] for s in st]), torch.stack([s[1] for s in st]))
    budget = int(math.floor(prep.code_bits(5.0) * J))
    widths, pos, counts = B.dq_allocate(F, J, budget)
    c = counts.cpu().numpy()[0]
    w = host(widths).astype(int)
    assert sum(c[:4]) == J and budget - 6 < int(w.sum()) <= budget
    order = np.argsort(host(F), kind="stable")
    assert np.all(np.diff(w[order]) >= 0)
    re = [B.dq_reorder(x, pos, J) for x in xs]
    mu_main = B.dq_reorder_mean(mu, pos, J, counts)
    ctx = B.Context(n, seed=11)
    rp = B.Replay(ctx, B.DQ_RING, B.DQ_DYNAMIQ, re, J, [[int(v) for v in c[:3]]], mu=mu_main)
    rp.run()
    out = B.dq_restore(rp.out, pos, J, n, mu_main=mu_main)
    true = sum(x.double() for x in xs)
    est = out.double()
    assert float(((est - true) ** 2).sum() / (true ** 2).sum()) < 0.05
    # the shifted super-group: without the mean handling its 0.5 offset would dominate the error
    assert float((est[:256] - true[:256]).abs().max()) < 0.02
