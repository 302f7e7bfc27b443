"""The decoder's registers-held window and its workgroup sizes: stretches of codewords beyond the table (of up to 38
bits, drawn at random) in runs that otherwise hit it, at one to eight wavefronts a workgroup; codewords of up to 52
bits in every order around hits; stored tables of a shorter prefix; and the average with the values of a tensor in
LDS against an anchor per run or element.  Everything is defined bit for bit."""
import numpy as np
import pytest

import oracle
import co3_inputs as inp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def co3():
    import paper_2203_09044_amd as pkg
    return pkg


@pytest.mark.parametrize("E,M", [(2, 0), (1, 2), (3, 1), (4, 3)])
@pytest.mark.parametrize("n,C,U", [(1, 256, 1), (15, 64, 1), (17, 64, 1), (64 * 64, 64, 1), (64 * 64 + 1, 64, 3), (1_048_577, 64, 1),
                                   (700_001, 64, 3), (4_194_304 - 31, 64, 1), (3_000_013, 64, 3), (9_000_001, 128, 1)])
def test_stretches_of_long_codewords(co3, E, M, n, C, U):
    fmt = co3.Fmt(E, M)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + U)
    # probabilities fall by a factor 0.6 a symbol, with a floor, so the lengths run from 1 to far beyond the table
    # (where the alphabet is large enough); stretches of 8 to 40 symbols come from the rarest ones
    K = fmt.K
    p = 0.6 ** np.arange(K)
    p = np.maximum(p, 1e-12)
    w = np.maximum((p / p.sum() * 3e9), 1).astype(np.uint64).astype(np.uint32)
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=C, codes="user", cap_words=2 * (n // 4 + 64))
    s = torch.multinomial(torch.tensor(p, device="cuda"), U * n, replacement=True, generator=gen).reshape(U, n)
    rare = torch.randint(max(K - 8, 0), K, (U, n), device="cuda", generator=gen)
    at = torch.rand(U, (n + 39) // 40, device="cuda", generator=gen).repeat_interleave(40, dim=1)[:, :n] < 0.01
    s = torch.where(at, rare, s).to(torch.uint8)
    pipe.sym[:, :n] = s
    weights = torch.from_numpy(np.tile(w.view(np.int32), (U, 1))).cuda()
    pipe.build(weights)
    pipe.encode()
    pipe.decode()
    assert pipe.poll() == 0
    assert torch.equal(pipe.sym_dec[:, :n], s)


# more chunks than 20 wavefronts a compute unit hold: the stream is requested 64 aligned bytes at a time; every user's
# begins at another place within these, and ends where the buffer does
@pytest.mark.parametrize("E,M", [(4, 3), (3, 1)])
@pytest.mark.parametrize("n,C,U", [(2_199_999, 256, 40), (24_000_257, 512, 7)])
def test_requests_of_64_bytes(co3, E, M, n, C, U):
    fmt = co3.Fmt(E, M)
    K = fmt.K
    p = np.maximum(0.9 ** np.arange(K), 1e-9)
    w = np.maximum((p / p.sum() * 3e9), 1).astype(np.uint64).astype(np.uint32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    edges = torch.tensor(np.cumsum(p / p.sum()), device="cuda", dtype=torch.float32)
    s = torch.empty((U, n), dtype=torch.uint8, device="cuda")
    for u in range(U):
        x = torch.bucketize(torch.rand(n, device="cuda", generator=gen), edges).clamp_(max=K - 1)
        rare = torch.randint(K - 8, K, (n,), device="cuda", generator=gen)
        at = (torch.rand((n + 39) // 40, device="cuda", generator=gen) < 0.01).repeat_interleave(40)[:n]
        s[u] = torch.where(at, rare, x).to(torch.uint8)
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=C, cap_words=(n // 6) // 8 * 8 + 2)
    pipe.sym[:, :n] = s
    pipe.build(torch.from_numpy(np.tile(w.view(np.int32), (U, 1))).cuda())
    pipe.encode()
    longest = (int(pipe.total_bits.max()) + 127) // 128 * 2          # as little room as the streams leave
    pipe.words = pipe.words[:, :longest + (6 if longest % 8 == 0 else 0)].contiguous()
    pipe.decode()
    assert pipe.poll() == 0
    assert torch.equal(pipe.sym_dec[:, :n], s)


# Shared codes of few long tensors on at least eight wavefronts a compute unit: 64 bytes a request, tables from tensor to
# tensor.  All users hold the same symbols, as many as a power of two: their average is one user's values.
@pytest.mark.parametrize("n,C,U", [(1_100_001, 128, 16), (2_199_999, 256, 16), (2_199_999, 512, 32)])
def test_requests_of_64_bytes_under_shared_codes(co3, n, C, U):
    fmt, f = co3.Fmt(4, 3), oracle.Fmt(4, 3)
    r = np.random.default_rng(C)
    seg = [0, n // 5 + 3, n // 2 - 77, n // 2 - 77, n - 70_000, n]
    p = np.maximum(0.9 ** np.arange(fmt.K), 1e-9)
    w = np.stack([np.roll(np.maximum(p / p.sum() * 3e9, 1).astype(np.uint32), 5 * k) for k in range(5)])
    s = np.minimum(np.searchsorted(np.cumsum(p / p.sum()), r.random(n)), fmt.K - 1)
    at = np.repeat(r.random((n + 39) // 40) < 0.01, 40)[:n]
    s[at] = r.integers(fmt.K - 8, fmt.K, int(at.sum()))
    for k in range(5):
        s[seg[k]:seg[k + 1]] = (s[seg[k]:seg[k + 1]] + 5 * k) % fmt.K
    s = s.astype(np.uint8)
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=C, cap_words=(n // 6) // 8 * 8 + 2, codes="layer", code_seg_off=seg)
    row = torch.from_numpy(s).cuda()
    pipe.sym[:, :n] = row
    pipe.build(torch.from_numpy(w.view(np.int32)).cuda())
    pipe.encode()
    pipe.decode()
    pipe.anchor.fill_(2)
    pipe.aggregate()
    assert pipe.poll() == 0
    assert torch.equal(pipe.sym_dec[:, :n], row.expand(U, n))
    want = oracle.aggregate(s[None], np.array([[2]], np.int32), f)
    assert np.array_equal(pipe.avg[:n].cpu().numpy().view(np.uint32), want.view(np.uint32))


def fibonacci(k):
    w = [1, 1]
    while len(w) < k:
        w.append(w[-1] + w[-2])
    return w[:k]


# codes whose longest codewords (43 and 52 bits) do not fit what a window of 64 bits holds after two hits of the
# 14-bit table (36 bits), the second one not even what it holds after one (50)
DEEP = {"43 bits": fibonacci(44), "52 bits": fibonacci(47) + [2**32 - 1] * 200}


def runs_around_misses(lengths, quiet):
    """Runs of 16 symbols: every group of four drawn from the longest codeword, two that the table misses, two hits
    at and below its width and the shortest, at each of the run's four places, shortest codewords around it and in
    `quiet` further runs."""
    by_length = [int(np.flatnonzero(lengths == k)[-1]) for k in (lengths.max(), 37, 20, 14, 13, lengths[lengths > 0].min())]
    groups = np.stack(np.meshgrid(*[by_length] * 4, indexing="ij"), axis=-1).reshape(-1, 4)
    runs = np.full((len(groups), 4, 16 * (1 + quiet)), by_length[-1], np.uint8)
    for q in range(4):
        runs[:, q, 4 * q:4 * q + 4] = groups
    return runs.reshape(-1)


# without quiet runs some chunks take more than eight bits a symbol, where the decoder tests for misses symbol by
# symbol; with these no chunk does, and it tests after every four
@pytest.mark.parametrize("code,C,quiet", [("43 bits", 64, 0), ("43 bits", 64, 1), ("43 bits", 256, 0), ("43 bits", 256, 3),
                                          ("52 bits", 64, 0), ("52 bits", 256, 15)])
def test_misses_around_hits(co3, code, C, quiet):
    fmt, f = co3.Fmt(4, 3), oracle.Fmt(4, 3)
    w = np.zeros(256, np.uint32)
    w[:len(DEEP[code])] = DEEP[code]
    lengths = np.asarray(oracle.huffman_lengths(w))
    s = runs_around_misses(lengths, quiet)
    n, U = len(s), 2
    words, off, total = oracle.encode(s, lengths, oracle.canonical_codes(lengths), C)
    assert (int(np.diff(off.astype(np.int64)).max()) > 8 * C) == (quiet == 0)
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=C, cap_words=len(words) + 2)
    pipe.sym[:, :n] = torch.from_numpy(s).cuda()
    pipe.build(torch.from_numpy(np.tile(w.view(np.int32), (U, 1))).cuda())
    pipe.encode()
    assert np.array_equal(pipe.words[1, :(total + 63) // 64].cpu().numpy().view(np.uint64), words[:(total + 63) // 64])
    pipe.decode()
    got = pipe.sym_dec[:, :n].cpu().numpy()
    assert np.array_equal(got, np.tile(s, (U, 1)))
    pipe.anchor[:] = torch.tensor([[3], [-2]], dtype=torch.int32)
    pipe.aggregate()
    want = oracle.aggregate(np.tile(s, (U, 1)), np.array([[3], [-2]], np.int32), f)
    assert np.array_equal(pipe.avg[:n].cpu().numpy().view(np.uint32), want.view(np.uint32))
    assert pipe.poll() == 0


@pytest.mark.parametrize("bits", [0, 1, 2, 3, 7, 11])
@pytest.mark.parametrize("longest", [13, 14, 15, 19])
def test_stored_table_of_a_shorter_prefix(co3, bits, longest):
    """A code blob whose decoder table resolves fewer leading bits than the library's own (which takes 12; 0 is read
    as 1): what it leaves out is entered from the canonical lengths, nothing is written beyond the widened table."""
    fmt = co3.Fmt(4, 3)
    w = np.zeros(256, np.uint32)
    w[:longest + 1] = fibonacci(longest + 1)
    lengths = np.asarray(oracle.huffman_lengths(w))
    assert lengths.max() == longest
    codewords = oracle.canonical_codes(lengths)
    n = 64 * 256 + 5
    s = np.random.default_rng(bits).integers(0, longest + 1, n).astype(np.uint8)
    pipe = co3.Co3Pipeline(1, n, fmt, cap_words=n // 2)
    pipe.sym[0, :n] = torch.from_numpy(s).cuda()
    pipe.build(torch.from_numpy(w.view(np.int32)).cuda().reshape(1, 256))
    pipe.encode()
    assert pipe.poll() == 0
    blob = pipe.codes[0].cpu().numpy().copy()
    lut_bits = blob[3352:3356].view(np.uint32)       # behind len, enc, first_code, count, base, sorted, nact, maxlen
    lut = blob[3360:3360 + 2 * 4096].view(np.uint16)
    assert int(lut_bits[0]) == 12 and int(lut[0]) == (1 << 8 | longest)
    stored = max(bits, 1)
    lut[:] = 0
    for k in np.flatnonzero((lengths > 0) & (lengths <= stored)):
        span = 1 << (stored - int(lengths[k]))
        lut[int(codewords[k]) * span:(int(codewords[k]) + 1) * span] = (int(lengths[k]) << 8) | k
    lut_bits[0] = bits
    pipe.codes[0] = torch.from_numpy(blob).cuda()
    pipe.decode()
    assert pipe.poll() == 0
    assert np.array_equal(pipe.sym_dec[0, :n].cpu().numpy(), s)


# users are taken four (or two) at a time; a division by a power of two is a multiplication: results down to the
# smallest subnormal numbers, which both round once
@pytest.mark.parametrize("E,M", [(3, 0), (3, 1), (4, 3)])
@pytest.mark.parametrize("U", [1, 2, 4, 5, 8, 9, 63])
@pytest.mark.parametrize("alpha", [1e-3, 1e-36, 1e-38, 1e-41])
def test_average_of_users_taken_together(co3, E, M, U, alpha):
    n = 2_501
    fmt, f = co3.Fmt(E, M), oracle.Fmt(E, M)
    r = np.random.default_rng(U * 11 + E)
    g = (r.standard_normal((U, n)) * alpha).astype(np.float32)
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=64)
    buf = pipe.new_gradient_buffer()
    buf[:, :n] = torch.from_numpy(g).cuda()
    pipe.step(buf)
    assert pipe.poll() == 0
    A = np.array([[oracle.anchor(g[u], f)] for u in range(U)], np.int32).reshape(U, 1)
    sym = np.stack([oracle.convert_ef(g[u], np.zeros(n, np.float32), int(A[u, 0]), 1.0, f)[0] for u in range(U)])
    want = oracle.aggregate(sym, A, f)
    assert np.array_equal(pipe.avg[:n].cpu().numpy().view(np.uint32), want.view(np.uint32))


LAYOUTS = {
    "one tile and less": [5000, 3, 0, 900],
    "steps inside tensors": [100_000, 60_001, 7],
    "tile edges": [16_384, 16_384, 1, 16_383, 64],
    "many small": [37] * 700 + [40_000] + [1] * 65,
}


@pytest.mark.parametrize("layout", list(LAYOUTS))
@pytest.mark.parametrize("E,M", [(3, 0), (3, 1), (4, 3)])
@pytest.mark.parametrize("U", [1, 2, 3, 5])
def test_average_of_several_tensors(co3, layout, E, M, U):
    sizes = LAYOUTS[layout]
    seg = inp.seg_offsets(sizes)
    n = int(seg[-1])
    fmt, f = co3.Fmt(E, M), oracle.Fmt(E, M)
    r = np.random.default_rng(U * 7 + E)
    scale = np.repeat(10.0 ** r.uniform(-30, 20, len(sizes)), sizes)
    g = (r.standard_normal((U, n)) * scale).astype(np.float32)
    pipe = co3.Co3Pipeline(U, n, fmt, seg_off=seg)
    buf = pipe.new_gradient_buffer()
    buf[:, :n] = torch.from_numpy(g).cuda()
    pipe.step(buf)
    assert pipe.poll() == 0
    A = np.stack([oracle.anchor(g[u], f, seg) for u in range(U)])
    sym = np.stack([oracle.convert_ef(g[u], np.zeros(n, np.float32), A[u], 1.0, f, seg)[0] for u in range(U)])
    want = oracle.aggregate(sym, A, f, seg)
    assert np.array_equal(pipe.avg[:n].cpu().numpy().view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("scaled", [False, True])
@pytest.mark.parametrize("E,M", [(3, 0), (4, 3)])
@pytest.mark.parametrize("U", [1, 2, 4])
def test_average_over_empty_and_single_element_tensors(co3, E, M, U, scaled):
    """Runs that hold many tensors, several beginning at the same element, beside runs inside one."""
    r = np.random.default_rng(U)
    sizes = np.concatenate([r.choice([0, 0, 1, 2, 40], 2000), [0] * 300, [20_000, 0, 1, 0], r.choice([0, 1], 700)])
    seg = inp.seg_offsets(sizes)
    n, fmt, f = int(seg[-1]), co3.Fmt(E, M), oracle.Fmt(E, M)
    pipe = co3.Co3Pipeline(U, n, fmt, seg_off=seg)
    s = r.integers(0, fmt.K, (U, n)).astype(np.uint8)
    pipe.sym[:, :n] = torch.from_numpy(s).cuda()
    co3.binding.histogram(pipe.sym, n, fmt, pipe.counts)
    pipe.build()
    pipe.encode()
    anchor = r.integers(-20, 20, (U, len(sizes))).astype(np.int32)
    scale = r.uniform(0.5, 40.0, (U, len(sizes))).astype(np.float32) if scaled else None
    pipe.anchor[:] = torch.from_numpy(anchor)
    if scaled:
        co3.binding.ps_aggregate_scaled(pipe.words, pipe.chunk_bitoff, pipe.chunk_syms, pipe.codes, fmt, n, U, pipe.anchor,
                                        torch.from_numpy(scale).cuda(), pipe.avg, pipe.agg_ws, pipe.status, seg_off=pipe.seg_off)
    else:
        pipe.aggregate()
    assert pipe.poll() == 0
    want = oracle.aggregate(s, anchor, f, seg, scale)
    assert np.array_equal(pipe.avg[:n].cpu().numpy().view(np.uint32), want.view(np.uint32))


def encoded(co3, fmt, s, seg, C=256):
    """A pipeline that holds the streams of the users' symbols s."""
    U, n = s.shape
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=C, seg_off=seg)
    pipe.sym[:, :n] = torch.from_numpy(s).cuda()
    co3.binding.histogram(pipe.sym, n, fmt, pipe.counts)
    pipe.build()
    pipe.encode()
    return pipe


# tensors whose values are kept in LDS: from 65,536 elements each on average and three users (six in 7- and 8-bit formats),
# from 32,768 and ten; one of too few users and one of too short tensors beside them
@pytest.mark.parametrize("E,M,U", [(3, 0, 3), (3, 1, 4), (4, 3, 6), (5, 2, 7), (3, 0, 10), (3, 1, 10), (4, 3, 5)])
@pytest.mark.parametrize("way", ["plain", "multipliers", "continued sum"])
def test_average_with_a_tensors_values_in_lds(co3, E, M, U, way):
    fmt, f, B = co3.Fmt(E, M), oracle.Fmt(E, M), co3.binding
    r = np.random.default_rng(U * 3 + E)
    sizes = [150_001, 90_000, 7, 120_000, 64] if U < 10 else [60_001, 40_000, 3, 64_000]
    seg = inp.seg_offsets(sizes)
    n = int(seg[-1])
    s = r.integers(0, fmt.K, (U, n)).astype(np.uint8)
    pipe = encoded(co3, fmt, s, seg)
    anchor = r.integers(-20, 20, (U, len(sizes))).astype(np.int32)
    pipe.anchor[:] = torch.from_numpy(anchor)
    if way == "continued sum":
        start = r.standard_normal(n).astype(np.float32)
        acc = torch.nn.functional.pad(torch.from_numpy(start), (0, pipe.stride - n)).cuda()
        B.ps_aggregate_partial(pipe.words, pipe.chunk_bitoff, 256, pipe.codes, fmt, n, U, pipe.anchor, acc, U + 3, acc, pipe.agg_ws,
                               pipe.status, seg_off=pipe.seg_off)
        want = start
        for u in range(U):
            want = want + oracle.aggregate(s[u:u + 1], anchor[u:u + 1], f, seg)
        got, want = acc, want / np.float32(U + 3)
    elif way == "multipliers":
        scale = (r.uniform(0.5, 40.0, anchor.shape) * r.choice([-1.0, 1.0], anchor.shape)).astype(np.float32)
        B.ps_aggregate_scaled(pipe.words, pipe.chunk_bitoff, 256, pipe.codes, fmt, n, U, pipe.anchor, torch.from_numpy(scale).cuda(),
                              pipe.avg, pipe.agg_ws, pipe.status, seg_off=pipe.seg_off)
        got, want = pipe.avg, oracle.aggregate(s, anchor, f, seg, scale)
    else:
        pipe.aggregate()
        got, want = pipe.avg, oracle.aggregate(s, anchor, f, seg)
    assert pipe.poll() == 0
    assert np.array_equal(got[:n].cpu().numpy().view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("E,M,U", [(3, 0, 1), (3, 0, 5), (3, 1, 4), (4, 3, 1), (4, 3, 4), (4, 3, 5), (4, 3, 9)])
def test_average_with_negative_multipliers(co3, E, M, U):
    """One tensor: a value is the level divided by the multiplier, sign and all, in every form of the table."""
    fmt, f = co3.Fmt(E, M), oracle.Fmt(E, M)
    r = np.random.default_rng(U + E)
    n = 20_003
    s = r.integers(0, fmt.K, (U, n)).astype(np.uint8)
    pipe = encoded(co3, fmt, s, None)
    anchor = r.integers(-20, 20, (U, 1)).astype(np.int32)
    scale = (r.uniform(0.5, 40.0, (U, 1)) * np.where(np.arange(U) % 2, 1.0, -1.0)[:, None]).astype(np.float32)
    pipe.anchor[:] = torch.from_numpy(anchor)
    co3.binding.ps_aggregate_scaled(pipe.words, pipe.chunk_bitoff, 256, pipe.codes, fmt, n, U, pipe.anchor,
                                    torch.from_numpy(scale).cuda(), pipe.avg, pipe.agg_ws, pipe.status)
    assert pipe.poll() == 0
    want = oracle.aggregate(s, anchor, f, None, scale)
    assert np.array_equal(pipe.avg[:n].cpu().numpy().view(np.uint32), want.view(np.uint32))


# runs inside a tensor take a value as the code's bits times a power of two where that is exact, from the conversion's lowest
# anchor to its highest; one below it they do not
@pytest.mark.parametrize("E,M", [(1, 2), (3, 0), (3, 1), (4, 3), (5, 2), (7, 0)])
@pytest.mark.parametrize("U", [1, 2, 5])
def test_average_at_the_ends_of_the_anchors(co3, E, M, U):
    fmt, f = co3.Fmt(E, M), oracle.Fmt(E, M)
    r = np.random.default_rng(U)
    low = (1 << E) - 1 - 126
    ends = [low - 1, low, low + 1, 0, 125, 126, 127]
    seg = inp.seg_offsets([2000] * len(ends))
    n = int(seg[-1])
    s = r.integers(0, fmt.K, (U, n)).astype(np.uint8)
    s[1:, int(seg[4]):] = 0                       # sums of the largest levels stay finite
    s[:, :64] = 1                                 # the smallest level
    s[0, -64:] = fmt.K // 2 - 1                   # the largest
    pipe = encoded(co3, fmt, s, seg)
    anchor = np.tile(np.array(ends, np.int32), (U, 1))
    pipe.anchor[:] = torch.from_numpy(anchor)
    pipe.aggregate()
    assert pipe.poll() == 0
    want = oracle.aggregate(s, anchor, f, seg)
    assert np.isfinite(want).all() and np.abs(want).max() >= 2.0 ** 127 / U and np.abs(want[want != 0]).min() <= 2.0 ** -126
    assert np.array_equal(pipe.avg[:n].cpu().numpy().view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("E,M", [(3, 0), (4, 3)])
@pytest.mark.parametrize("U", [1, 2, 5])
def test_average_of_extreme_tensors(co3, E, M, U):
    """Tensors of zeros, of subnormal numbers and of one user's values near the largest float, through a whole iteration."""
    fmt, f = co3.Fmt(E, M), oracle.Fmt(E, M)
    r = np.random.default_rng(U)
    sizes = [3000, 2001, 5, 4096, 900]
    seg = inp.seg_offsets(sizes)
    n = int(seg[-1])
    g = (r.standard_normal((U, n)) * np.repeat([0.0, 1e-41, 1e-38, 1.0, 0.0], sizes)).astype(np.float32)
    g[0, int(seg[4]):] = (r.uniform(-1.0, 1.0, sizes[4]) * 3.3e38).astype(np.float32)
    pipe = co3.Co3Pipeline(U, n, fmt, seg_off=seg)
    buf = pipe.new_gradient_buffer()
    buf[:, :n] = torch.from_numpy(g).cuda()
    pipe.step(buf)
    assert pipe.poll() == 0
    A = np.stack([oracle.anchor(g[u], f, seg) for u in range(U)])
    assert A.min() == (1 << E) - 1 - 126 and A.max() == 127
    sym = np.stack([oracle.convert_ef(g[u], np.zeros(n, np.float32), A[u], 1.0, f, seg)[0] for u in range(U)])
    want = oracle.aggregate(sym, A, f, seg)
    assert np.array_equal(pipe.avg[:n].cpu().numpy().view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("E,M", [(3, 0), (4, 3)])
@pytest.mark.parametrize("n", [1, 1024, 16_384, 16_385, 64 * 16_384 - 1, 64 * 16_384, 64 * 16_384 + 1])
def test_group_offsets_in_the_packer(co3, n, E, M):
    """Up to 64 groups of tiles the packer scans the group sizes itself; the stream, its index and its length are
    the oracle's on both sides of the line, and a stream beyond its capacity is reported on both."""
    fmt, f = co3.Fmt(E, M), oracle.Fmt(E, M)
    g = (np.random.default_rng(n).standard_normal(n) * 1e-3).astype(np.float32)
    A = oracle.anchor(g, f)
    s, _ = oracle.convert_ef(g, np.zeros(n, np.float32), A, 1.0, f)
    lengths = oracle.huffman_lengths(oracle.histogram(s, f))
    words, off, total = oracle.encode(s, lengths, oracle.canonical_codes(lengths), 256)
    need = (total + 63) // 64
    need += need & 1
    for cap, want in ((need, 0), (need - 2, co3.binding.ECAP)):
        if cap == 0:
            continue
        pipe = co3.Co3Pipeline(1, n, fmt, cap_words=need)
        pipe.convert(torch.nn.functional.pad(torch.from_numpy(g), (0, pipe.stride - n)).reshape(1, -1).cuda())
        pipe.build()
        w = torch.zeros((1, cap), dtype=torch.int64, device="cuda")
        co3.binding.encode(pipe.sym, n, fmt, pipe.codes, w, 256, pipe.chunk_bitoff, pipe.total_bits, pipe.enc_ws, pipe.status)
        assert pipe.poll() == want
        assert int(pipe.total_bits[0].item()) == total
        assert np.array_equal(pipe.chunk_bitoff[0].cpu().numpy().view(np.uint64), off)
        if want == 0:
            assert np.array_equal(w[0, :(total + 63) // 64].cpu().numpy().view(np.uint64), words[:(total + 63) // 64])
