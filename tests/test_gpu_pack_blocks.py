"""The packer in batches of at least 4,096 blocks of four tiles, where a workgroup takes groups of four blocks if the users'
vectors hold whole ones, and a tile per wavefront if not: ends on, before and behind a block, codewords and pairs of
codewords beyond its 32-bit table entries, blocks beyond its window, streams beyond their capacity, codes per user and per
group of tensors, symbols a byte and two per byte.  Every word is defined; the oracle packs some of the users, and the
others are equal to them."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BLOCK = 4096


@pytest.fixture(scope="module")
def co3():
    import paper_2203_09044_amd as pkg
    return pkg


def draw(n, K, seed, dense):
    """Symbols of geometric probabilities; stretches of the rarest ones; `dense`: a whole block of these."""
    rng = np.random.default_rng(seed)
    s = np.minimum(np.floor(np.log(rng.random(n)) / np.log(0.6)), K - 1).astype(np.uint8)
    rare = rng.integers(max(K - 8, 0), K, n).astype(np.uint8)
    at = np.repeat(rng.random((n + 39) // 40) < 0.01, 40)[:n]
    s[at] = rare[at]
    if dense:
        s[BLOCK // 2:BLOCK + BLOCK // 2] = rare[BLOCK // 2:BLOCK + BLOCK // 2][:max(n - BLOCK // 2, 0)]
    return s


def geometric_weights(K):
    p = np.maximum(0.6 ** np.arange(K), 1e-12)
    return np.maximum(p / p.sum() * 3e9, 1).astype(np.uint64).astype(np.uint32)


def fill(pipe, rows, n):
    """Rows of symbols to all users in turn."""
    for r, s in enumerate(rows):
        pipe.sym[r::len(rows), :n] = torch.from_numpy(s).cuda()


def check(pipe, rows, want, n):
    for r, (words, off, total) in enumerate(want):
        nw = (total + 63) // 64
        got = pipe.words[r::len(rows), :nw]
        assert torch.equal(got, torch.from_numpy(words[:nw].view(np.int64)).cuda().expand_as(got))
        assert bool((pipe.total_bits[r::len(rows)] == total).all())
        got = pipe.chunk_bitoff[r::len(rows)]
        assert torch.equal(got, torch.from_numpy(off.view(np.int64)).cuda().expand_as(got))


# users of few blocks (those of a group and a little more take a tile per wavefront); the last two with more than 64
# groups of tiles
SIZES = [(2050, 2 * BLOCK), (2050, 2 * BLOCK - 1), (1400, 2 * BLOCK + 1), (1100, 4 * BLOCK - 1025), (900, 4 * BLOCK + 62),
         (4100, 4 * BLOCK), (3300, 4 * BLOCK + 1), (2800, 6 * BLOCK - 63), (17, 262 * BLOCK + 1023), (64, 257 * BLOCK)]


@pytest.mark.parametrize("E,M", [(3, 1), (4, 3)])
@pytest.mark.parametrize("U,n", SIZES)
def test_codes_per_user(co3, E, M, U, n):
    fmt = co3.Fmt(E, M)
    C = 64 if n < 10 * BLOCK else 4096
    w = geometric_weights(fmt.K)
    lengths = np.asarray(oracle.huffman_lengths(w))
    codes = oracle.canonical_codes(lengths)
    rows = [draw(n, fmt.K, 1, False), draw(n, fmt.K, 2, True), np.zeros(n, np.uint8)]
    want = [oracle.encode(s, lengths, codes, C) for s in rows]
    cap = max((t + 63) // 64 for _, _, t in want) + 2
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=C, cap_words=cap)
    fill(pipe, rows, n)
    pipe.build(torch.from_numpy(np.tile(w.view(np.int32), (U, 1))).cuda())
    pipe.encode()
    check(pipe, rows, want, n)
    assert pipe.poll() == 0


@pytest.mark.parametrize("U,n", [(1400, 2 * BLOCK + 1), (900, 4 * BLOCK + 62), (2800, 6 * BLOCK - 63), (17, 262 * BLOCK + 1023)])
def test_codes_per_group_of_tensors(co3, U, n):
    fmt, C = co3.Fmt(4, 3), 128
    # boundaries on a block, just behind one (within its look-ahead), inside a tile, and an empty group
    seg = [0, BLOCK, 2 * BLOCK - 70 if n < 3 * BLOCK else 3 * BLOCK + 30, 2 * BLOCK - 70 if n < 3 * BLOCK else 3 * BLOCK + 30, n - 30, n]
    w = np.stack([np.roll(geometric_weights(fmt.K), 3 * k) for k in range(len(seg) - 1)])
    lengths = np.stack([np.asarray(oracle.huffman_lengths(x)) for x in w])
    codes = np.stack([oracle.canonical_codes(x) for x in lengths])
    rows = [draw(n, fmt.K, 3, False), draw(n, fmt.K, 4, True)]
    want = [oracle.encode_layers(s, lengths, codes, seg, C) for s in rows]
    cap = max((t + 63) // 64 for _, _, t in want) + 2
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=C, cap_words=cap, codes="layer", code_seg_off=seg)
    fill(pipe, rows, n)
    pipe.build(torch.from_numpy(w.view(np.int32)).cuda())
    pipe.encode()
    check(pipe, rows, want, n)
    assert pipe.poll() == 0


@pytest.mark.parametrize("U,n", [(2050, 2 * BLOCK), (900, 4 * BLOCK + 62), (2800, 6 * BLOCK - 63), (17, 262 * BLOCK + 1023)])
def test_two_symbols_per_byte(co3, U, n):
    """co3_user_encode keeps the symbols two per byte unless the caller asks for them; the streams are the same.  The
    counts fall by half from symbol to symbol; in a stretch of the rarest ones eight symbols take more than 64 bits (and in
    the longest vector a pair of them more than 24)."""
    fmt = co3.Fmt(3, 0)
    rng = np.random.default_rng(n)
    mags = np.concatenate([[0.0], 2.0 ** np.arange(-6, 1)]).astype(np.float32)           # levels under the anchor 0
    rank = np.minimum(np.floor(-np.log2(rng.random(n))), 14).astype(int)
    rank[BLOCK // 2:BLOCK // 2 + 48] = rng.integers(11, 15, 48)
    rank[:15] = np.arange(15)
    g_host = np.concatenate([mags, -mags[1:]])[rank]
    out = []
    for keep in (True, False):
        pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=64, one_call=True, keep_symbols=keep)
        g = pipe.new_gradient_buffer()
        g[:, :n] = torch.from_numpy(g_host).cuda()
        pipe.user_encode(g)
        assert pipe.poll() == 0
        out.append(pipe)
    s = out[0].sym[0, :n].cpu().numpy()
    lengths = out[0].codes[0, :fmt.K].cpu().numpy()
    assert lengths[s[BLOCK // 2:BLOCK // 2 + 8]].sum() > 64 and (n < 100 * BLOCK or lengths.max() >= 13)
    want = oracle.encode(s, lengths, oracle.canonical_codes(lengths), 64)
    for pipe in out:
        check(pipe, [s], [want], n)


@pytest.mark.parametrize("short", [1, 65, 200])
def test_beyond_the_capacity(co3, short):
    """A tile is written if its end lies within the capacity; nothing is written behind the last such tile."""
    fmt, U, n, C = co3.Fmt(4, 3), 900, 4 * BLOCK + 62, 64
    w = geometric_weights(fmt.K)
    lengths = np.asarray(oracle.huffman_lengths(w))
    long_row, rows = draw(n, fmt.K, 5, False), [np.zeros(n, np.uint8), (np.arange(n) % 2).astype(np.uint8)]
    codes = oracle.canonical_codes(lengths)
    words, off, total = oracle.encode(long_row, lengths, codes, C)
    cap = ((total + 63) // 64 - short) // 2 * 2
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=C, cap_words=cap)
    fill(pipe, rows, n)
    pipe.sym[1, :n] = torch.from_numpy(long_row).cuda()
    pipe.words.fill_(-1)
    pipe.build(torch.from_numpy(np.tile(w.view(np.int32), (U, 1))).cuda())
    pipe.encode()
    assert pipe.poll() == -2                                # CO3_ECAP
    ends = off[16::16].astype(np.int64)                     # of the whole tiles of 1,024
    last = int((((ends + 63) // 64) <= cap).sum())
    nw = (int(ends[last - 1]) + 63) // 64
    got = pipe.words[1].cpu().numpy().view(np.uint64)
    assert np.array_equal(got[:nw], words[:nw]) and bool((got[nw:] == np.uint64(2**64 - 1)).all())
    for u, r in ((0, 0), (2, 0), (3, 1), (U - 1, 1)):
        ww, _, t = oracle.encode(rows[r], lengths, codes, C)
        assert np.array_equal(pipe.words[u, :(t + 63) // 64].cpu().numpy().view(np.uint64), ww[:(t + 63) // 64])


# Groups of four blocks: users of at least eight blocks, or whose last group holds two or more.
GROUP_SIZES = [(1400, 3 * BLOCK + 5), (1100, 4 * BLOCK), (700, 6 * BLOCK), (500, 8 * BLOCK + 62), (460, 9 * BLOCK - 1), (420, 9 * BLOCK + 1025)]


def draw_blocks(n, K, seed):
    """Blocks of short codewords; of 10 to 31 bits a symbol (a window of their own); of more; of both kinds in turn."""
    s = draw(n, K, seed, False)
    rng = np.random.default_rng(seed)
    for b in range((n + BLOCK - 1) // BLOCK):
        part = s[b * BLOCK:(b + 1) * BLOCK]
        kind = int(rng.integers(0, 4))
        if kind and K > 30:
            lo, hi = ((18, 26), (K - 8, K), (8, 16))[kind - 1]
            part[:] = rng.integers(lo, hi, part.size)
    return s


@pytest.mark.parametrize("E,M", [(3, 1), (4, 3)])
@pytest.mark.parametrize("U,n", GROUP_SIZES)
def test_groups_of_blocks(co3, E, M, U, n):
    fmt, C = co3.Fmt(E, M), 128
    w = geometric_weights(fmt.K)
    lengths = np.asarray(oracle.huffman_lengths(w))
    codes = oracle.canonical_codes(lengths)
    rows = [draw_blocks(n, fmt.K, s) for s in (1, 2, 3, 4)]
    if E == 4:
        bits = np.concatenate([lengths[r[:n // BLOCK * BLOCK]].reshape(-1, BLOCK).sum(axis=1) for r in rows]) / BLOCK
        assert (bits < 9).any() and (bits > 31.5).any() and ((bits > 10) & (bits < 31)).any()
    want = [oracle.encode(s, lengths, codes, C) for s in rows]
    cap = max((t + 63) // 64 for _, _, t in want) + 2
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=C, cap_words=cap)
    fill(pipe, rows, n)
    pipe.build(torch.from_numpy(np.tile(w.view(np.int32), (U, 1))).cuda())
    pipe.encode()
    check(pipe, rows, want, n)
    assert pipe.poll() == 0


@pytest.mark.parametrize("U,n", [(170, 24 * BLOCK + 77), (17, 262 * BLOCK + 1023)])
def test_groups_of_blocks_under_shared_codes(co3, U, n):
    fmt, C = co3.Fmt(4, 3), 256
    # a boundary on a block, one within the look-ahead of a block and one just beyond, one inside a tile, an empty group
    seg = [0, 5 * BLOCK, 10 * BLOCK + 62, 10 * BLOCK + 62, 15 * BLOCK + 63, n]
    w = np.stack([np.roll(geometric_weights(fmt.K), 3 * k) for k in range(len(seg) - 1)])
    lengths = np.stack([np.asarray(oracle.huffman_lengths(x)) for x in w])
    codes = np.stack([oracle.canonical_codes(x) for x in lengths])
    rows = [draw_blocks(n, fmt.K, s) for s in (5, 6, 7)]
    want = [oracle.encode_layers(s, lengths, codes, seg, C) for s in rows]
    cap = max((t + 63) // 64 for _, _, t in want) + 2
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=C, cap_words=cap, codes="layer", code_seg_off=seg)
    fill(pipe, rows, n)
    pipe.build(torch.from_numpy(w.view(np.int32)).cuda())
    pipe.encode()
    check(pipe, rows, want, n)
    assert pipe.poll() == 0


@pytest.mark.parametrize("U,n", [(460, 9 * BLOCK + 62), (700, 6 * BLOCK - 63)])
def test_groups_of_blocks_two_symbols_per_byte(co3, U, n):
    test_two_symbols_per_byte(co3, U, n)


@pytest.mark.parametrize("short", [1, 65, 2500, 5000])
def test_groups_of_blocks_beyond_the_capacity(co3, short):
    """As test_beyond_the_capacity; the end of the capacity lies in a block that could be packed together."""
    fmt, U, n, C = co3.Fmt(4, 3), 460, 9 * BLOCK + 62, 64
    w = geometric_weights(fmt.K)
    lengths = np.asarray(oracle.huffman_lengths(w))
    codes = oracle.canonical_codes(lengths)
    row = draw_blocks(n, fmt.K, 8)
    words, off, total = oracle.encode(row, lengths, codes, C)
    cap = ((total + 63) // 64 - short) // 2 * 2
    pipe = co3.Co3Pipeline(U, n, fmt, chunk_syms=C, cap_words=cap)
    pipe.sym[:, :n] = 0
    pipe.sym[1, :n] = torch.from_numpy(row).cuda()
    pipe.words.fill_(-1)
    pipe.build(torch.from_numpy(np.tile(w.view(np.int32), (U, 1))).cuda())
    pipe.encode()
    assert pipe.poll() == -2                                # CO3_ECAP
    ends = off[16::16].astype(np.int64)                     # of the whole tiles of 1,024
    last = int((((ends + 63) // 64) <= cap).sum())
    nw = (int(ends[last - 1]) + 63) // 64
    got = pipe.words[1].cpu().numpy().view(np.uint64)
    assert np.array_equal(got[:nw], words[:nw]) and bool((got[nw:] == np.uint64(2**64 - 1)).all())
