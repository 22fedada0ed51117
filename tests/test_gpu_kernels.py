"""GPU kernels at the sizes where their dispatch and their edges can go wrong: table build, packer, projection and
decoder variants, each against the CPU oracle (code tables, streams and symbols: equal; see test_gpu_parity for the
bars of computed values)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fmtc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_10830_amd import binding

    binding.load_library()
    return binding


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def symbols_with_counts(counts, seed, multiple):
    """A shuffled symbol array with these counts (the first symbol's padded so that the size is a multiple)."""
    counts = np.array(counts, np.int64)
    counts[0] += -int(counts.sum()) % multiple
    sym = np.repeat(np.arange(len(counts)), counts).astype(np.uint8)
    np.random.default_rng(seed).shuffle(sym)
    return sym


def counts_of(kind, K):
    i = np.arange(K)
    if kind == "equal":  # every window of the merge is full, every comparison a tie
        return np.full(K, 40)
    if kind == "ones":  # half the symbols once, the others powers of two: ties between leaves and internal nodes
        return np.where(i < K // 2, 1, 1 << (i % 5))
    if kind == "steep":  # long codes and many rounds
        return np.maximum(1, (200000 * 0.8 ** np.abs(i - K // 2)).astype(np.int64))
    if kind == "gaps":  # unused symbols in every block of 64
        return np.where(i % 3 == 1, 0, 1 + (i * 37) % 101)
    return np.where(i < 66, 1 + i, 0)  # a few more used symbols than the small merge takes


@pytest.mark.parametrize("kind", ["equal", "ones", "steep", "gaps", "just65"])
@pytest.mark.parametrize("bits", [6, 7, 8])
def test_code_table_of_crafted_counts(fmtc, oracle, bits, kind):
    C = 16
    sym = symbols_with_counts(counts_of(kind, 1 << bits), bits, C)
    hist = oracle.histogram(sym, bits)
    ln = oracle.huffman_lengths(hist)
    ref = oracle.pack(sym, C, bits, 0.5, ln, oracle.canonical_codes(ln))
    stream, nbytes = fmtc.code_symbols(dev(sym), C, bits, 0.5)
    torch.cuda.synchronize()
    got = stream[:int(nbytes.item())].cpu().numpy()
    assert np.array_equal(got[64:320], ln), "code lengths"
    assert np.array_equal(got, ref)
