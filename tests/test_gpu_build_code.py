"""The code build merges a node a step (up to 16 leaves) or in rounds: the sizes at which one follows the other and
at which a round changes its form (more than 63 leaves or nodes), the weights at which the arithmetic does (2^30 in
all), ties, and very deep and very flat trees, each against the oracle; the code is then used to encode and decode, so
that codewords and decoder tables are the canonical ones.  (Symbols are drawn uniformly there; codewords beyond the
decoder's table in every order are the decoder's own test.)"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def co3():
    import paper_2203_09044_amd as pkg
    return pkg


def fibonacci(k):
    w = [1, 1]
    while len(w) < k:
        w.append(w[-1] + w[-2])
    return w[:k]


def cases():
    r = np.random.default_rng(5)
    out = []
    for k in (1, 2, 3, 4, 5, 15, 16, 17, 62, 63, 64, 65, 66, 126, 127, 128, 129, 255, 256):
        out.append((f"equal-{k}", np.full(k, 7)))
        out.append((f"two-levels-{k}", np.where(np.arange(k) % 3 == 0, 5, 10)))
    for k in (8, 40, 44):
        out.append((f"fibonacci-{k}", r.permutation(np.array(fibonacci(k)))))
    for total in ((1 << 30) - 1, 1 << 30, (1 << 30) + 1):       # 32-bit weights below, doubles from there on
        w = r.integers(1, 1000, 200).astype(np.int64)
        w[17] += total - int(w.sum())
        out.append((f"total-{total}", w))
    out.append(("all-largest", np.full(256, 2**32 - 1)))
    out.append(("powers", 2 ** (np.arange(256, dtype=np.int64) % 32)))
    out.append(("gaps", np.where(r.random(256) < 0.6, 0, r.integers(1, 9, 256))))
    out.append(("skewed", np.maximum(1, (r.random(256) ** 9 * 4e6)).astype(np.int64)))
    return out


@pytest.mark.parametrize("name,weights", cases(), ids=[c[0] for c in cases()])
def test_code_of_edge_weights(co3, name, weights):
    B = co3.binding
    fmt = co3.Fmt(4, 3)
    w = np.zeros(256, np.uint32)
    w[256 - len(weights):] = np.asarray(weights, dtype=np.uint32)
    codes = torch.zeros((1, B.CODE_BYTES), dtype=torch.uint8, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.build_code(torch.from_numpy(w.view(np.int32).reshape(1, -1)).cuda(), 1, fmt, codes, status)
    want = oracle.huffman_lengths(w)
    assert np.array_equal(codes[0, :256].cpu().numpy(), np.asarray(want, dtype=np.uint8))
    active = np.flatnonzero(w)
    n = 4096 + 3
    sym = np.concatenate([active, np.random.default_rng(1).choice(active, n - len(active))]).astype(np.uint8)
    words, off, total = oracle.encode(sym, want, oracle.canonical_codes(want), 256)
    d_sym = torch.zeros(n + 13, dtype=torch.uint8, device="cuda")
    d_sym[:n] = torch.from_numpy(sym).cuda()
    cap = (len(words) + 3) & ~1
    d_words = torch.zeros(cap, dtype=torch.int64, device="cuda")
    d_off = torch.zeros(len(off), dtype=torch.int64, device="cuda")
    d_tot = torch.zeros(1, dtype=torch.int64, device="cuda")
    ws = torch.zeros(B.encode_workspace_bytes(n, 1) // 8 + 1, dtype=torch.int64, device="cuda")
    B.encode(d_sym, n, fmt, codes, d_words, 256, d_off, d_tot, ws, status)
    back = torch.zeros_like(d_sym)
    B.decode(d_words, d_off, 256, codes, fmt, n, back, status)
    assert B.poll_status(status) == 0
    assert int(d_tot.item()) == total
    nw = (total + 63) // 64
    assert np.array_equal(d_words.cpu().numpy().view(np.uint64)[:nw], words[:nw])
    assert np.array_equal(back[:n].cpu().numpy(), sym)


@pytest.mark.parametrize("E,M", [(1, 0), (2, 0), (3, 0), (3, 1), (4, 3)])
def test_many_codes_in_one_call(co3, E, M):
    """More codes than two large workgroups per compute unit take smaller ones: the same blobs byte for byte as in
    calls of a few codes, and the oracle's lengths.  Up to 16 leaves and more, weights below and above 2^30 in all."""
    B = co3.binding
    fmt, r = co3.Fmt(E, M), np.random.default_rng(E * 8 + M)
    U = 2 * torch.cuda.get_device_properties(0).multi_processor_count + 1
    w = (r.random((U, fmt.K)) ** r.integers(1, 12, (U, 1)) * 10.0 ** r.integers(1, 10, (U, 1))).astype(np.int64)
    w = np.where(r.random((U, fmt.K)) < r.random((U, 1)), np.minimum(w, 2**32 - 1), r.integers(0, 3, (U, fmt.K)))
    w[:20] *= np.arange(fmt.K) < np.arange(20)[:, None]                   # 0 to 19 leaves
    w = w.astype(np.uint32)
    d = torch.from_numpy(w.view(np.int32)).cuda()
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    many, few = (torch.zeros((U, B.CODE_BYTES), dtype=torch.uint8, device="cuda") for _ in range(2))
    B.build_code(d, U, fmt, many, status)
    for u in range(0, U, 100):
        B.build_code(d[u:u + 100], min(100, U - u), fmt, few[u:u + 100], status)
    assert B.poll_status(status) == 0
    assert torch.equal(many, few)
    got = many[:, :256].cpu().numpy()
    for u in range(U):
        assert np.array_equal(got[u, :fmt.K], np.asarray(oracle.huffman_lengths(w[u]), dtype=np.uint8)), u
