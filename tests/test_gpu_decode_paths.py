"""The decoder's registers-held window and its workgroup sizes: stretches of codewords beyond the table in runs
that otherwise hit it, at one to eight wavefronts a workgroup.  Everything is defined bit for bit."""
import numpy as np
import pytest

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

