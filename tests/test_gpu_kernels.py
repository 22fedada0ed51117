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


# Packer of large tensors: more than 4096 chunks.  Chunk sizes that are multiples of 8, of 4 only, of neither; a range of 17
# chunks and more per workgroup (all its images, and several ranges: RANGE_CASES); 64 images per workgroup (fewer:
# test_packer_with_two_to_four_images); code words of more than 27 bits, chunks larger than an image.
STREAM_CASES = [  # P, C, bits, chunk_syms, kind
    (4097 * 4, 16, 6, 64, "steep"),
    (15 * 300, 64, 6, 64, "steep"),
    (40001, 12, 5, 64, "equal"),
    (9999, 33, 4, 66, "steep"),
    (70001, 9, 7, 99, "gaps"),
    (4113 * 8, 128, 6, 1024, "steep"),
    (4200 * 20, 100, 8, 2048, "steep"),
    (4100 * 4, 1000, 3, 4096, "equal"),
    (16400, 1024, 6, 4096, "fibonacci"),
    (4100, 1024, 8, 1024, "fibonacci"),
]


@pytest.mark.parametrize("P,C,bits,chunk,kind", STREAM_CASES, ids=[f"P{c[0]}C{c[1]}b{c[2]}k{c[3]}{c[4]}" for c in STREAM_CASES])
def test_packer_of_large_tensors(fmtc, oracle, P, C, bits, chunk, kind):
    K, V = 1 << bits, P * C
    if kind == "fibonacci":  # the longest codes that fit: counts 1, 1, 2, 3, 5, ...
        f = [1, 1]
        while sum(f) + f[-1] + f[-2] < V and len(f) < K:
            f.append(f[-1] + f[-2])
        counts = np.array(f + [0] * (K - len(f)), np.int64)
    else:
        counts = counts_of(kind, K).astype(np.float64)
        counts = np.where(counts > 0, np.maximum(1, counts * (V / counts.sum()) * 0.9), 0).astype(np.int64)
    counts[counts.argmax()] += V - counts.sum()
    sym = np.repeat(np.arange(K), counts).astype(np.uint8)
    np.random.default_rng(bits + C).shuffle(sym)
    if kind == "fibonacci":  # the rare symbols together in one chunk: more code bits than an image holds
        sym = np.sort(sym)
        sym = np.concatenate([sym[chunk:], sym[:chunk]])
    ln = oracle.huffman_lengths(oracle.histogram(sym, bits))
    ref = oracle.pack(sym, C, bits, 0.5, ln, oracle.canonical_codes(ln), chunk)
    stream, nbytes = fmtc.code_symbols(dev(sym), C, bits, 0.5, chunk)
    torch.cuda.synchronize()
    n = int(nbytes.item())
    got = stream[:n].cpu().numpy()
    assert n == len(ref) and np.array_equal(got, ref), f"first differing byte {int(np.argmax(got[:len(ref)] != ref[:n]))}"
    back, err = fmtc.decode_symbols(stream, P, C, bits, nbytes=n)
    torch.cuda.synchronize()
    assert int(err.item()) == 0 and np.array_equal(back.cpu().numpy().reshape(-1), sym)


# ... and more: (chunks, symbols a chunk, ...) in ranges of 61 chunks, nearly all of a workgroup's 64 images, and in two ranges of
# 45 and of 38 per workgroup, the last ones short.
TURN_CASES = [(15 * 256 * 4 + 1, 66, 33, 6, "steep"), (15 * 256 * 6 - 1, 64, 16, 4, "gaps"), (15 * 256 * 5 + 1, 99, 9, 7, "gaps"),
              (15 * 256 * 4 + 16, 33, 33, 8, "steep")]


@pytest.mark.parametrize("n_chunks,chunk,C,bits,kind", TURN_CASES, ids=[f"n{c[0]}k{c[1]}b{c[3]}" for c in TURN_CASES])
def test_packer_of_many_turns(fmtc, oracle, n_chunks, chunk, C, bits, kind):
    V = n_chunks * chunk
    counts = counts_of(kind, 1 << bits).astype(np.float64)
    counts = np.where(counts > 0, np.maximum(1, counts * (V / counts.sum()) * 0.9), 0).astype(np.int64)
    counts[counts.argmax()] += V - counts.sum()
    sym = np.repeat(np.arange(1 << bits), counts).astype(np.uint8)
    np.random.default_rng(n_chunks).shuffle(sym)
    ln = oracle.huffman_lengths(oracle.histogram(sym, bits))
    ref = oracle.pack(sym, C, bits, 0.5, ln, oracle.canonical_codes(ln), max(chunk, 64))
    stream, nbytes = fmtc.code_symbols(dev(sym), C, bits, 0.5, max(chunk, 64))
    torch.cuda.synchronize()
    assert int(nbytes.item()) == len(ref) and np.array_equal(stream[:len(ref)].cpu().numpy(), ref)


# Ranges of chunks: (chunks, symbols a chunk, C, bits, counts) with as many chunks as 256 workgroups have images and one more, a
# range per workgroup and three, the fewest chunks of that kernel; images of 1024 and of 684 words (code words of nearly 8 and
# nearly 5 bits), the last of them one round and a chunk.
RANGE_CASES = [(4097, 64, 16, 6, "gaps"), (256 * 64, 66, 33, 6, "steep"), (256 * 64 + 1, 64, 16, 6, "steep"),
               (256 * 128 + 3, 99, 9, 4, "gaps"), (256 * 32 + 1, 3200, 32, 8, "flat"), (256 * 48 + 1, 4092, 33, 5, "flat")]


@pytest.mark.parametrize("n_chunks,chunk,C,bits,kind", RANGE_CASES, ids=[f"n{c[0]}k{c[1]}b{c[3]}" for c in RANGE_CASES])
def test_packer_of_chunk_ranges(fmtc, oracle, n_chunks, chunk, C, bits, kind):
    V = n_chunks * chunk
    rng = np.random.default_rng(n_chunks)
    if kind == "flat":
        sym = rng.integers(0, 1 << bits, V, dtype=np.uint8)
    else:
        counts = counts_of(kind, 1 << bits).astype(np.float64)
        counts = np.where(counts > 0, np.maximum(1, counts * (V / counts.sum()) * 0.9), 0).astype(np.int64)
        counts[counts.argmax()] += V - counts.sum()
        sym = np.repeat(np.arange(1 << bits), counts).astype(np.uint8)
        rng.shuffle(sym)
    ln = oracle.huffman_lengths(oracle.histogram(sym, bits))
    ref = oracle.pack(sym, C, bits, 0.5, ln, oracle.canonical_codes(ln), max(chunk, 64))
    for _ in range(2):
        stream, nbytes = fmtc.code_symbols(dev(sym), C, bits, 0.5, max(chunk, 64))
        torch.cuda.synchronize()
        assert int(nbytes.item()) == len(ref) and np.array_equal(stream[:len(ref)].cpu().numpy(), ref)


def test_packer_of_large_tensors_gives_up_its_waits(fmtc, oracle):
    """With the limit of its waits at once reached the kernel ends, leaves an invalid stream and harms no later call."""
    C, bits, chunk, n_chunks = 16, 6, 64, 15 * 256 * 2
    sym = symbols_with_counts(np.full(64, n_chunks * chunk // 64), 5, C)
    ln = oracle.huffman_lengths(oracle.histogram(sym, bits))
    ref = oracle.pack(sym, C, bits, 0.5, ln, oracle.canonical_codes(ln), chunk)
    for short in (1, 0):
        fmtc.test_option(fmtc.TEST_SHORT_WAITS, short)
        try:
            stream, nbytes = fmtc.code_symbols(dev(sym), C, bits, 0.5, chunk)
            torch.cuda.synchronize()
        finally:
            fmtc.test_option(fmtc.TEST_SHORT_WAITS, 0)
        if short:
            assert int(stream[:4].view(torch.int32).item()) == 0
            _, err = fmtc.decode_symbols(stream, len(sym) // C, C, bits)
            torch.cuda.synchronize()
            assert int(err.item()) & 1  # the header
    assert int(nbytes.item()) == len(ref) and np.array_equal(stream[:len(ref)].cpu().numpy(), ref)


def coder_us(fmtc, sym, C, bits, chunk):
    """Shortest of 40 coder runs in us (kernels after the histogram)."""
    P = len(sym) // C
    d = dev(sym)
    stream = torch.empty(fmtc.encode_bound(P, C, bits, chunk), dtype=torch.uint8, device="cuda")
    nbytes = torch.zeros(1, dtype=torch.int64, device="cuda")
    work = torch.empty(fmtc.workspace_size(P, C, bits, chunk), dtype=torch.uint8, device="cuda")
    fmtc.profile_enable(40)
    try:
        for _ in range(40):
            fmtc.code_symbols(d, C, bits, 0.5, chunk, stream, nbytes, work)
        torch.cuda.synchronize()
        return 1e3 * sum(v[1] for k, v in fmtc.profile_read().items() if "histogram" not in k)
    finally:
        fmtc.profile_enable(0)


def normal_symbols(n_chunks, chunk, bits, spread, seed):
    rng = np.random.default_rng(seed)
    half = 1 << (bits - 1)
    x = rng.standard_normal((n_chunks, chunk), dtype=np.float32) * np.float32(spread)
    return np.clip(np.rint(x), -half, half - 1).astype(np.int16) + half


def test_packer_takes_any_chunk_size_at_the_same_rate(fmtc):
    """Chunks that are no multiple of eight symbols (4092, measured: the same time as 4096; fetched byte by byte, 2.1 times)."""
    n = 6000
    even = coder_us(fmtc, normal_symbols(n, 4096, 6, 0.5, 3).astype(np.uint8).reshape(-1), 64, 6, 4096)
    odd = coder_us(fmtc, normal_symbols(n, 4092, 6, 0.5, 3).astype(np.uint8).reshape(-1), 33, 6, 4096)
    assert odd < 1.5 * even, f"{odd:.1f} us, {even:.1f} us for whole pieces"


def uneven_symbols(n_chunks, chunk, bits, seed=4, together=False):
    """Every tenth chunk of a flat tensor nearly uniform over the alphabet: several times the average chunk's bits."""
    sym = normal_symbols(n_chunks, chunk, bits, (1 << bits) / 128.0, seed)
    loud = np.random.default_rng(seed).random(n_chunks) < 0.1
    loud[-1] = True
    if together:
        loud = np.sort(loud)
    sym[loud] = normal_symbols(int(loud.sum()), chunk, bits, (1 << bits) / 8.0, seed + 1)
    return sym.astype(np.uint8).reshape(-1), loud


@pytest.mark.parametrize("bits,chunk,C,together", [(6, 4096, 64, False), (8, 4096, 64, False), (6, 4092, 33, False), (7, 4090, 10, False),
                                                   (5, 4032, 144, False), (6, 4096, 64, True), (8, 4096, 64, True), (7, 4090, 10, True)])
def test_packer_of_uneven_chunks(fmtc, oracle, bits, chunk, C, together):
    n = 4200
    sym, loud = uneven_symbols(n, chunk, bits, together=together)
    ln = oracle.huffman_lengths(oracle.histogram(sym, bits))
    ref = oracle.pack(sym, C, bits, 0.5, ln, oracle.canonical_codes(ln))
    words = ln[sym.reshape(n, chunk)].sum(axis=1, dtype=np.int64) // 32
    # (the images hold a third more than the average)
    assert (words[loud] > max(512, 1.4 * words.mean())).mean() > 0.9, "large chunks do not exceed their images"
    stream, nbytes = fmtc.code_symbols(dev(sym), C, bits, 0.5)
    torch.cuda.synchronize()
    assert int(nbytes.item()) == len(ref) and np.array_equal(stream[:len(ref)].cpu().numpy(), ref)


def test_packer_is_not_held_up_by_uneven_chunks(fmtc):
    """Every tenth chunk several times the others' size (measured: 1.6 times the flat tensor's time, for 1.3 times its bits;
    with later windows built symbol by symbol, 3.1 times)."""
    n = 12544
    flat = coder_us(fmtc, normal_symbols(n, 4096, 6, 0.5, 3).astype(np.uint8).reshape(-1), 64, 6, 4096)
    uneven = coder_us(fmtc, uneven_symbols(n, 4096, 6)[0], 64, 6, 4096)
    assert uneven < 2.2 * flat, f"{uneven:.1f} us, {flat:.1f} us for the flat tensor"


def test_packer_is_not_held_up_by_large_chunks_side_by_side(fmtc):
    """A tenth of the chunks large, all in a few ranges, so that some workgroups have no others (measured: 1.5 times the time
    of every tenth one, 3 times where what lies past an image went to one word)."""
    n, us = 12544, []
    loud = np.random.default_rng(5).integers(0, 64, (n // 10, 4096), dtype=np.uint8)
    for at in (slice(0, 10 * (n // 10), 10), slice(0, n // 10)):
        sym = normal_symbols(n, 4096, 6, 0.4, 3).astype(np.uint8)
        sym[at] = loud
        us.append(coder_us(fmtc, sym.reshape(-1), 64, 6, 4096))
    assert us[1] < 2.1 * us[0], f"{us[1]:.1f} us, {us[0]:.1f} us for every tenth chunk"


# The packer's last step of a chunk: one octet per lane or two, whole and broken ones, after none, one and two whole steps.
@pytest.mark.parametrize("bits", [6, 8])
@pytest.mark.parametrize("chunk", [64, 505, 512, 513, 520, 1023, 1025, 1536, 1537, 1544, 2049, 2561, 3071])
def test_packer_ends_of_chunks(fmtc, oracle, chunk, bits):
    n = 4111
    sym = normal_symbols(n, chunk, bits, (1 << bits) / 12.0, chunk).astype(np.uint8).reshape(-1)[:n * chunk - chunk // 2]
    ln = oracle.huffman_lengths(oracle.histogram(sym, bits))
    ref = oracle.pack(sym, 1, bits, 0.5, ln, oracle.canonical_codes(ln), chunk)
    stream, nbytes = fmtc.code_symbols(dev(sym), 1, bits, 0.5, chunk)
    torch.cuda.synchronize()
    assert int(nbytes.item()) == len(ref) and np.array_equal(stream[:len(ref)].cpu().numpy(), ref)


# Octets of eight symbols with long codes, all together: 65 to 96, 97 to 126 and more bits, code words beyond a table entry's
# 26 bits (alone or as a pair), each next to short ones; across the ends of images and chunks.
@pytest.mark.parametrize("bits,share,chunk", [(8, 0.2, 4096), (8, 0.03, 4096), (8, 0.03, 256), (8, 0.003, 512), (8, 0.0003, 1001),
                                              (7, 0.01, 777), (6, 0.05, 256), (6, 0.01, 4096), (6, 0.0005, 4096)])
def test_packer_of_long_octets(fmtc, oracle, bits, share, chunk):
    n, K = 4113, 1 << bits
    rng = np.random.default_rng(int(1e5 * share) + bits)
    octets = -(-n * chunk // 8)
    rare = rng.random(octets) < share
    sym = np.where(np.repeat(rare, 8), rng.integers(8, K, 8 * octets), rng.integers(0, 8, 8 * octets))[:n * chunk].astype(np.uint8)
    ln = oracle.huffman_lengths(oracle.histogram(sym, bits))
    ref = oracle.pack(sym, 1, bits, 0.5, ln, oracle.canonical_codes(ln), chunk)
    stream, nbytes = fmtc.code_symbols(dev(sym), 1, bits, 0.5, chunk)
    torch.cuda.synchronize()
    assert int(nbytes.item()) == len(ref) and np.array_equal(stream[:len(ref)].cpu().numpy(), ref)


# Images that a workgroup's room is divided into, for each of its 16 wavefronts: four up to 3 bits a symbol of a whole chunk,
# three up to 4, two beyond; pairs of symbols in the table up to 6 bits, single ones above.  Every tenth chunk is several
# times larger.
@pytest.mark.parametrize("images,bits,spread,n_chunks", [(4, 6, 0.8, 4111), (3, 6, 1.6, 4111), (3, 8, 1.2, 4124), (2, 6, 5.0, 4111),
                                                         (2, 7, 6.0, 4124), (2, 8, 14.0, 4111), (2, 8, 40.0, 4096)])
@pytest.mark.parametrize("chunk,C", [(4096, 64), (4092, 33)])
def test_packer_with_two_to_four_images(fmtc, oracle, images, bits, spread, n_chunks, chunk, C):
    if n_chunks <= 4096:
        n_chunks += 1  # (up to 4096 chunks another kernel packs)
    sym = normal_symbols(n_chunks, chunk, bits, spread, n_chunks + bits)
    loud = np.random.default_rng(bits).random(n_chunks) < 0.1
    sym[loud] = np.random.default_rng(bits + 1).integers(0, 1 << bits, (int(loud.sum()), chunk))
    sym = sym.astype(np.uint8)
    ln = oracle.huffman_lengths(oracle.histogram(sym.reshape(-1), bits))
    per_chunk = ln[sym].sum(axis=1, dtype=np.int64)
    need = int(per_chunk.sum()) // 24  # (the rule of images_for)
    assert images == (4 if need <= 512 * n_chunks else 3 if need <= 684 * n_chunks else 2), per_chunk.mean() / chunk
    sym = sym.reshape(-1)
    ref = oracle.pack(sym, C, bits, 0.5, ln, oracle.canonical_codes(ln))
    stream, nbytes = fmtc.code_symbols(dev(sym), C, bits, 0.5)
    torch.cuda.synchronize()
    assert int(nbytes.item()) == len(ref) and np.array_equal(stream[:len(ref)].cpu().numpy(), ref)


def identity_activations(fmtc, sym, C, bits):
    """A basis and activations [1, 1, P, C] whose symbols are these."""
    top = (1 << (bits - 1)) - 1
    basis = fmtc.basis_import(np.eye(C, dtype=np.float32), np.zeros(C, np.float32), np.float32(0.5 * top))
    x = ((sym.astype(np.float32) - (top + 1)) * 0.5).reshape(1, 1, -1, C)
    return basis, dev(x)


# Fixed tables, more chunks than the small packer takes: pairs and single symbols in the table, whole and odd chunk sizes,
# a code with words of more than 26 bits, chunks beyond the image's 1024 words.
@pytest.mark.parametrize("bits,chunk,C,table", [(5, 256, 16, "fit"), (6, 250, 10, "long"), (7, 256, 16, "fit"), (7, 99, 9, "long"),
                                                (8, 256, 32, "fit"), (8, 250, 10, "long"), (8, 4096, 64, "long"), (6, 4092, 33, "long")])
def test_packer_of_large_tensors_with_a_fixed_table(fmtc, oracle, bits, chunk, C, table):
    n_chunks, K = 4111, 1 << bits
    sym = normal_symbols(n_chunks, chunk, bits, K / 16.0, bits).astype(np.uint8)
    sym[::10] = np.random.default_rng(bits).integers(0, K, sym[::10].shape)
    sym = sym.reshape(-1)
    ln = oracle.huffman_lengths(oracle.histogram(sym, bits)[:K] + 1)
    if table == "long":  # 1, 2, 3, ... 40 and the rest at one length (Kraft sum 1), the short words for the frequent symbols
        short = 16 if K == 64 else 24
        deep = short + int(np.ceil(np.log2(K - short)))
        n_deep = 2 * (K - short) - (1 << (deep - short))  # the others one bit shorter
        lengths = list(range(1, short + 1)) + [deep - 1] * (K - short - n_deep) + [deep] * n_deep
        order = np.argsort(np.abs(np.arange(K) - K // 2), kind="stable")
        ln = np.zeros_like(ln)
        ln[order] = sorted(lengths)
    assert sum(2.0 ** -int(v) for v in ln[:K]) == 1.0
    basis, x = identity_activations(fmtc, sym, C, bits)
    t = fmtc.table_import(ln[:K].astype(np.uint8), bits)
    stream, nbytes = fmtc.encode_static(basis, t, x, chunk_syms=chunk)
    torch.cuda.synchronize()
    n = int(nbytes.item())
    ref = oracle.pack(sym, C, bits, fmtc.delta(0.5 * (K // 2 - 1), bits), ln, oracle.canonical_codes(ln), chunk, cap=n + 4096)
    got = stream[:n].cpu().numpy()
    assert n == len(ref) and np.array_equal(got, ref), f"first differing byte {int(np.argmax(got[:len(ref)] != ref[:n]))}"
    # a buffer that holds about half of the payload: nothing past it, and no valid stream
    small = n - (n - 320 - 4 * (n_chunks + 1) - 2 * (-(-chunk // 64)) * n_chunks) // 2
    guard = torch.full((small + 8192,), 0xAB, dtype=torch.uint8, device="cuda")
    fmtc.encode_static(basis, t, x, chunk_syms=chunk, stream_out=guard[:small])
    torch.cuda.synchronize()
    assert (guard[small:] == 0xAB).all(), "wrote past the capacity it was given"
    _, err = fmtc.decode_symbols(guard[:small], len(sym) // C, C, bits)
    torch.cuda.synchronize()
    assert int(err.item()) & 1  # the header


@pytest.mark.parametrize("bits,chunk,C", [(6, 1024, 64), (8, 1024, 64), (6, 4096, 64)])
def test_packer_is_no_slower_with_a_fixed_table(fmtc, oracle, bits, chunk, C):
    """The same symbols, without a table to build (measured: 0.83, 0.57 and 0.87 of the time; with two images per packer
    whatever the chunk and the code bits counted in memory every turn 1.08, 0.72 and 0.96)."""
    n, K = 12 * 1024 * 1024 // chunk + 1500, 1 << bits
    sym = normal_symbols(n, chunk, bits, K / 32.0, bits).astype(np.uint8).reshape(-1)
    ln = oracle.huffman_lengths(oracle.histogram(sym, bits)[:K] + 1)
    basis, x = identity_activations(fmtc, sym, C, bits)
    t = fmtc.table_import(ln.astype(np.uint8), bits)
    own = coder_us(fmtc, sym, C, bits, chunk)
    P = len(sym) // C
    stream = torch.empty(fmtc.encode_static_bound(t, P, C, chunk), dtype=torch.uint8, device="cuda")
    nbytes = torch.zeros(1, dtype=torch.int64, device="cuda")
    work = torch.empty(fmtc.workspace_size(P, C, bits, chunk), dtype=torch.uint8, device="cuda")
    fmtc.profile_enable(40)
    try:
        for _ in range(40):
            fmtc.encode_static(basis, t, x, chunk_syms=chunk, stream_out=stream, out_bytes=nbytes, workspace=work)
        torch.cuda.synchronize()
        fixed = 1e3 * fmtc.profile_read()["k_pack"][1]
    finally:
        fmtc.profile_enable(0)
    assert fixed < 1.05 * own, f"{fixed:.1f} us with the fixed table, {own:.1f} us with the tensor's own"


# Tiled projection of wide tensors, more 128 x 128 tiles than compute units: channel counts with and without a half step
# of 16 at the end and with a last coefficient group of one to four tiles; ragged last tiles; a pixel beyond f16.
WIDE_CASES = [(176, 16411, 4), (192, 16388, 6), (240, 16500, 8), (256, 16385, 3), (272, 11000, 5), (528, 6700, 4)]


def check_projection(fmtc, oracle, C, N, H, W, bits, layout, T_scale=None, keep=None, reach=4.0):
    from paper_1905_10830_amd import synth

    P = N * H * W
    rng = np.random.default_rng(C)
    T = np.linalg.qr(rng.standard_normal((C, C)))[0].astype(np.float32)
    if T_scale is not None:
        T = T * np.asarray(T_scale, np.float32)[:, None]
    mu = rng.standard_normal(C).astype(np.float32)
    x = (rng.standard_normal((P, C)) * np.linspace(2.0, 0.1, C) + mu).astype(np.float32)
    x[[P // 2, max(0, P - 5)]] *= 1.0e5
    A = np.float32(reach if T_scale is None else reach * np.max(T_scale))
    y = (x.astype(np.float64) - mu) @ T.T.astype(np.float64)
    basis = fmtc.basis_import(T, mu, A)
    if keep is not None:
        y[:, keep:] = 0.0
        basis = basis.truncate(keep)
    sym, margin = oracle.quantize(y, oracle.delta(A, bits), bits, want_margin=True)
    xs = x.reshape(N, H, W, C)
    xs = xs if layout == "nhwc" else np.ascontiguousarray(xs.transpose(0, 3, 1, 2))
    got, hist = fmtc.quantize(basis, dev(xs), bits, synth.NHWC if layout == "nhwc" else synth.NCHW)
    torch.cuda.synchronize()
    got, hist = got.cpu().numpy().reshape(P, C), hist.cpu().numpy()
    diff = got != sym.reshape(P, C)
    # differences only where the fp64 value is at a rounding boundary (1e-9 steps: the order of an fp64 sum)
    assert not diff.any() or margin.reshape(P, C)[diff].max() <= 1e-9, f"{int(diff.sum())} symbols differ"
    assert hist.tolist() == np.bincount(got.reshape(-1), minlength=256).tolist()


# Every form of the projection that a tensor can take (the rows' and the streaming kernel's coefficient tiles, loads with and
# without masks, ...), at a size just beyond where it begins (or where its wavefronts come to a second tile): three images of
# 7 x w pixels, ragged last tiles, a pixel beyond f16 in the middle and one in the last tile.
FORM_CASES = [  # form, channels, w, bits, kept components (all of them if not given)
    ("rows 1 nhwc", 5, 77, 4), ("rows 1 nchw", 30, 77, 8), ("rows 1 vec nhwc", 28, 1600, 8), ("rows 1 vec nchw", 32, 77, 3),
    ("rows 2 nhwc", 33, 790, 6), ("rows 2 nchw", 63, 790, 5), ("rows 2 vec nhwc", 64, 790, 6), ("rows 2 vec nchw", 48, 790, 8),
    ("rows 3 nhwc", 65, 530, 6), ("rows 3 nchw", 95, 530, 8), ("rows 3 vec nhwc", 96, 530, 5), ("rows 3 vec nchw", 80, 530, 6),
    ("rows 4 nhwc", 97, 6250, 8), ("rows 4 nchw", 99, 6250, 4), ("rows 4 vec nhwc", 100, 6250, 8), ("rows 4x8 nhwc", 98, 6250, 5),
    ("rows 4x8 vec nhwc", 100, 6250, 6), ("rows 5 nhwc", 129, 320, 6), ("rows 5 vec nhwc", 140, 320, 7),
    ("stream 4 nhwc", 128, 400, 6), ("stream 4 nchw", 128, 400, 7), ("stream 4 half nhwc", 112, 400, 5), ("stream 4 half nchw", 112, 400, 6),
    ("stream 5 nhwc", 160, 320, 6), ("stream 5 nchw", 160, 320, 5), ("stream 5 half nhwc", 144, 320, 5), ("stream 5 half nchw", 144, 320, 7),
    # (2068 tiles: a whole round of the grid's wavefronts, and 20 more)
    ("stream 4x8 nhwc", 128, 3150, 8), ("stream 4x8 nchw", 128, 3150, 6), ("stream 4x8 half nhwc", 112, 3150, 6), ("stream 4x8 half nchw", 112, 3150, 5),
    ("stream 5x8 nhwc", 160, 3150, 7), ("stream 5x8 nchw", 160, 3150, 6), ("stream 5x8 half nhwc", 144, 3150, 4), ("stream 5x8 half nchw", 144, 3150, 5),
    ("split 1x1 nhwc", 64, 38, 6), ("split 1x1 nchw", 101, 38, 8), ("split 1x2 nhwc", 300, 70, 8), ("split 1x2 nchw", 64, 500, 6),
    ("split 1x4 nhwc", 250, 390, 6), ("split 1x4 nchw", 256, 570, 5), ("split 2x2 nhwc", 161, 600, 7), ("split 2x2 nchw", 133, 1590, 6),
    ("gemm8 nhwc", 256, 320, 6), ("gemm8 nchw", 176, 720, 4), ("gemm4 nhwc", 176, 785, 8), ("gemm4 nchw", 240, 785, 5),
    ("gemm8 fill nhwc", 256, 320, 6, 40), ("gemm8 fill nchw", 256, 790, 5, 128), ("gemm4 fill nhwc", 256, 1570, 5, 100),
    ("gemm4 fill nchw", 272, 1570, 4, 1), ("wide nhwc", 452, 600, 6), ("wide nchw", 161, 600, 4),
]


def form_of(fmtc, C, w, bits, layout, keep=None):
    from paper_1905_10830_amd import synth

    shape, tag = ((3, 7, w, C), synth.NHWC) if layout == "nhwc" else ((3, C, 7, w), synth.NCHW)
    head, rest = fmtc.test_projection(shape, tag, bits, keep).split(layout)
    return head + layout  # (without the rows of counts)


@pytest.mark.parametrize("case", FORM_CASES, ids=[c[0].replace(" ", "-") for c in FORM_CASES])
def test_every_form_of_the_projection(fmtc, oracle, case):
    form, C, w, bits, *keep = case
    layout, keep = form.rsplit(" ", 1)[1], keep[0] if keep else None
    assert form_of(fmtc, C, w, bits, layout, keep) == form
    check_projection(fmtc, oracle, C, 3, 7, w, bits, layout, keep=keep)


@pytest.mark.parametrize("case", [c for c in FORM_CASES if len(c) == 4], ids=[c[0].replace(" ", "-") for c in FORM_CASES if len(c) == 4])
def test_every_form_with_basis_entries_beyond_f16(fmtc, oracle, case):
    form, C, w, bits = case
    scale = np.ones(C)
    scale[[0, C // 2, C - 1]] = 3.0e6
    check_projection(fmtc, oracle, C, 3, 7, w, bits, form.rsplit(" ", 1)[1], scale)


# ... with a truncated basis, whose zero rows the forms leave out in units of their own (see also test_gpu_truncation)
@pytest.mark.parametrize("case", [c for c in FORM_CASES if len(c) == 4], ids=[c[0].replace(" ", "-") for c in FORM_CASES if len(c) == 4])
def test_every_form_with_a_truncated_basis(fmtc, oracle, case):
    form, C, w, bits = case
    check_projection(fmtc, oracle, C, 3, 7, w, bits, form.rsplit(" ", 1)[1], keep=max(1, C // 3))


# Rows of a basis with entries that f16 does not hold (not orthonormal, but accepted), of one image: their coefficients are
# decided exactly.  (Every form: above.)
@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("C,P", [(32, 500), (64, 3000), (100, 700), (128, 40000), (144, 5000), (176, 16411), (256, 2000), (250, 900)])
def test_projection_with_basis_entries_beyond_f16(fmtc, oracle, C, P, layout):
    scale = np.ones(C)
    scale[[0, C // 2, C - 1]] = 3.0e6
    check_projection(fmtc, oracle, C, 1, 1, P, 5, layout, scale)


# Rows of any norm, pixels that fill the quantizer's range and a tenth of it: the streaming form, whose operands are scaled by
# the two, with fewer and with more pixel tiles than SIMDs.  (Every norm, against a model of the sums: test_projection_band.)
LONG_ROWS = [(c, layout, reach) for c in ((128, 400, 8), (160, 320, 7), (128, 1800, 8)) for layout in ("nhwc", "nchw") for reach in (4.0, 40.0)]


@pytest.mark.parametrize("case,layout,reach", LONG_ROWS, ids=[f"C{c[0]}w{c[1]}{l}{int(r)}" for c, l, r in LONG_ROWS])
def test_streaming_projection_with_long_rows(fmtc, oracle, case, layout, reach):
    C, w, bits = case
    assert form_of(fmtc, C, w, bits, layout).startswith("stream")
    check_projection(fmtc, oracle, C, 3, 7, w, bits, layout, np.full(C, 32768.0), reach=reach)


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("C,w", [(128, 400), (144, 1800)])
def test_streaming_projection_with_short_rows(fmtc, oracle, C, w, layout):
    """... and no more values decided exactly because of the rows' norm, which is most of the kernel's time then (some 30 times
    as long where all of them were).  The limit leaves room for what timings differ by."""
    from paper_1905_10830_amd import synth

    bits, P, norm = 6, 21 * w, 2.0 ** -9
    check_projection(fmtc, oracle, C, 3, 7, w, bits, layout, np.full(C, norm))
    rng = np.random.default_rng(C)
    T = np.linalg.qr(rng.standard_normal((C, C)))[0].astype(np.float32)
    x = rng.standard_normal((P, C)).astype(np.float32)
    xs, tag = (dev(x.reshape(3, 7, w, C)), synth.NHWC) if layout == "nhwc" else (dev(x.reshape(3, 7, w, C).transpose(0, 3, 1, 2)), synth.NCHW)
    us = []
    for scale in (1.0, norm):
        basis = fmtc.basis_import(T * np.float32(scale), np.zeros(C, np.float32), np.float32(4.0 * scale))
        fmtc.quantize(basis, xs, bits, tag)
        fmtc.profile_enable(20)
        try:
            for _ in range(20):
                fmtc.quantize(basis, xs, bits, tag)
            torch.cuda.synchronize()
            us.append(1e3 * next(v[1] for k, v in fmtc.profile_read().items() if "project" in k))
        finally:
            fmtc.profile_enable(0)
    assert us[1] < 1.5 * us[0] + 2.0, f"{us[1]:.1f} us with short rows, {us[0]:.1f} us with unit rows"


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("C,P,bits", WIDE_CASES, ids=[f"C{c[0]}P{c[1]}b{c[2]}" for c in WIDE_CASES])
def test_projection_of_wide_tensors(fmtc, oracle, C, P, bits, layout):
    H = next(h for h in (10, 7, 5, 3, 2, 1) if P % h == 0)
    check_projection(fmtc, oracle, C, 1, H, P // H, bits, layout)


# The split contraction: one, two and four coefficient tiles per workgroup and two by two of them; one step per wavefront (33
# channels), last steps of 1 to 15 channels, ragged last pixel and coefficient tiles, more pixel groups than workgroups; a
# pixel beyond f16, decided exactly in all coefficients.  (Wavefronts without a step: truncated bases, test_gpu_truncation.)
SPLIT_CASES = [(33, 1, 2), (48, 8192, 8), (80, 3333, 5), (99, 9000, 6), (128, 5000, 3), (161, 40, 4), (250, 1300, 8), (255, 2600, 5),
               (316, 20000, 6), (353, 13000, 7), (1023, 70, 4), (1024, 33, 8), (1024, 1400, 5), (701, 6100, 2)]


@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("C,P,bits", SPLIT_CASES, ids=[f"C{c[0]}P{c[1]}b{c[2]}" for c in SPLIT_CASES])
def test_split_projection(fmtc, oracle, C, P, bits, layout):
    H = next(h for h in (10, 7, 5, 3, 2, 1) if P % h == 0)
    check_projection(fmtc, oracle, C, 1, H, P // H, bits, layout)


# Channel counts that are no multiple of 16, a workgroup's pixels with all channels in LDS: one and many coefficient groups,
# a group of fewer tiles than wavefronts, ragged last pixel and coefficient tiles, more pixel tiles than workgroups.
WIDE_FORM_CASES = [(1000, 1021, 8, "nhwc"), (452, 12001, 6, "nhwc"), (516, 16500, 8, "nhwc"), (1020, 4090, 3, "nhwc"), (129, 12001, 5, "nchw"),
                   (1001, 1021, 8, "nchw"), (250, 16320, 2, "nchw"), (502, 8161, 6, "nchw"), (510, 32800, 8, "nchw")]


@pytest.mark.parametrize("C,P,bits,layout", WIDE_FORM_CASES, ids=[f"C{c[0]}P{c[1]}b{c[2]}{c[3]}" for c in WIDE_FORM_CASES])
def test_projection_with_all_channels_in_lds(fmtc, oracle, C, P, bits, layout):
    from paper_1905_10830_amd import synth

    tag = synth.NHWC if layout == "nhwc" else synth.NCHW
    H = next(h for h in (10, 7, 5, 3, 2, 1) if P % h == 0)
    shape = (1, H, P // H, C) if layout == "nhwc" else (1, C, H, P // H)
    assert fmtc.test_projection(shape, tag, bits) == "wide " + layout
    check_projection(fmtc, oracle, C, 1, H, P // H, bits, layout)


# Planar projection of up to 160 channels: even and odd numbers of 32-channel pairs with and without a half step, tiles
# across one and many images, ragged last tiles, fewer and more tiles than wavefronts; 8 bits (five coefficient tiles: the
# tiled kernel, for LDS); a channel count that is no multiple of 16.
PLANAR_PROJECTION_CASES = [(16, 300, 11, 13, 8), (32, 2, 3, 3, 4), (32, 5000, 1, 1, 6), (48, 90, 27, 27, 5), (64, 16, 57, 61, 6),
                           (64, 5000, 3, 5, 4), (80, 300, 14, 14, 8), (96, 33, 31, 29, 5), (100, 40, 9, 9, 5), (112, 40, 29, 31, 5), (128, 3, 1, 1, 6), (128, 700, 7, 7, 8), (128, 4100, 3, 3, 4), (144, 170, 14, 15, 7),
                           (144, 1, 5, 5, 3), (144, 50, 9, 9, 8), (160, 36, 31, 31, 4), (160, 2000, 1, 1, 7)]


@pytest.mark.parametrize("C,N,H,W,bits", PLANAR_PROJECTION_CASES, ids=["_".join(map(str, c)) for c in PLANAR_PROJECTION_CASES])
def test_planar_projection(fmtc, oracle, C, N, H, W, bits):
    check_projection(fmtc, oracle, C, N, H, W, bits, "nchw")


# 129 to 160 channels at 8 bits (and at 7, where the basis and the histograms still share LDS), both layouts
@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("C,P,bits", [(129, 700, 8), (132, 2100, 8), (144, 4500, 8), (150, 33, 8), (160, 40000, 8), (160, 40000, 7), (144, 33, 7)])
def test_129_to_160_channels_at_8_bits(fmtc, oracle, C, P, bits, layout):
    from paper_1905_10830_amd import synth

    check_projection(fmtc, oracle, C, 1, 1, P, bits, layout)
    rng = np.random.default_rng(P)
    T = np.linalg.qr(rng.standard_normal((C, C)))[0].astype(np.float32)
    x = (rng.standard_normal((P, C)) * np.linspace(2.0, 0.1, C)).astype(np.float32)
    mu, A = np.zeros(C, np.float32), np.float32(8.0)
    basis, tag = fmtc.basis_import(T, mu, A), synth.NHWC if layout == "nhwc" else synth.NCHW
    xs = x.reshape(1, 1, P, C) if layout == "nhwc" else np.ascontiguousarray(x.T).reshape(1, C, 1, P)
    stream, nbytes = fmtc.encode(basis, dev(xs), bits, tag)
    out, err = fmtc.decode(basis, stream, xs.shape, bits, tag, nbytes=int(nbytes.item()))
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    out = out.cpu().numpy()
    out = out.reshape(P, C) if layout == "nhwc" else out.reshape(C, P).T
    d = float(oracle.delta(A, bits))
    sym = oracle.quantize(x.astype(np.float64) @ T.T.astype(np.float64), np.float32(d), bits).reshape(P, C)
    level = sym.astype(np.float64) - (1 << (bits - 1))
    ref = (level * d) @ T.astype(np.float64)
    # as in test_planar_decoder, and one step for a value at a rounding boundary
    tol = (2.0 ** -22 + C * 2.0 ** -24) * ((np.abs(level) * d) @ np.abs(T.astype(np.float64))) + 1e-7
    wrong = (np.abs(out - ref) > tol).any(axis=1)
    assert wrong.sum() <= 1 and np.abs(out - ref).max() <= d


# Planar decoder variants built for one channel count (32, 64: more than 3072 chunks; 128, 144: more than 2048), the
# shared one below that; images larger and smaller than a chunk, chunks across images, ragged last chunks, both sizes of
# payload buffers (4 and 8 bits), another chunk size than the nominal one.
PLANAR_CASES = [  # C, H, W, N, bits, chunk
    (32, 13, 11, 2751, 4, 4096), (64, 57, 61, 58, 6, 4096), (64, 3, 5, 13200, 8, 4096), (64, 40, 40, 8, 5, 4096),
    (128, 7, 7, 1350, 4, 4096), (128, 1, 1, 66001, 8, 4096), (128, 31, 33, 66, 6, 3968), (128, 9, 9, 30, 5, 4096),
    (144, 19, 17, 180, 5, 4096), (144, 7, 7, 1181, 8, 4096), (144, 14, 14, 20, 6, 4096),
]


@pytest.mark.parametrize("C,H,W,N,bits,chunk", PLANAR_CASES, ids=["_".join(map(str, c)) for c in PLANAR_CASES])
def test_planar_decoder(fmtc, oracle, C, H, W, N, bits, chunk):
    from paper_1905_10830_amd import synth

    rng = np.random.default_rng(C + H)
    T = np.linalg.qr(rng.standard_normal((C, C)))[0].astype(np.float32)
    mu = rng.standard_normal(C).astype(np.float32)
    P, A = N * H * W, np.float32(4.0)
    d = oracle.delta(A, bits)
    level = np.clip(np.rint(rng.laplace(0.0, 0.08 * (1 << bits), (P, C))), -(1 << (bits - 1)), (1 << (bits - 1)) - 1)
    sym = (level + (1 << (bits - 1))).astype(np.uint8)
    stream, nbytes = fmtc.code_symbols(dev(sym), C, bits, float(d), chunk)
    basis = fmtc.basis_import(T, mu, A)
    torch.cuda.synchronize()
    n = int(nbytes.item())
    ref = (level * float(d)) @ T.astype(np.float64) + mu
    # 22-bit basis entries and C fp32 additions, each relative to the sum of the products' magnitudes
    tol = (2.0 ** -22 + C * 2.0 ** -24) * ((np.abs(level) * float(d)) @ np.abs(T.astype(np.float64)) + np.abs(mu)) + 1e-7
    for tag in (synth.NCHW, synth.NHWC):
        shape = (N, C, H, W) if tag == synth.NCHW else (N, H, W, C)
        out, err = fmtc.decode(basis, stream, shape, bits, tag, nbytes=n)
        torch.cuda.synchronize()
        assert int(err.item()) == 0
        out = out.cpu().numpy()
        out = (out.transpose(0, 2, 3, 1) if tag == synth.NCHW else out).reshape(P, C)
        assert (np.abs(out - ref) <= tol).all(), f"largest error {np.abs(out - ref).max():.3e}"


# Chunks decoded several at a time (a unit: as many as 64 lanes hold runs of): one to 64 chunks per unit, chunks of whole
# and of broken runs, 33 runs (one chunk per unit again), a last unit of one chunk and a chunk of one pixel; narrow and
# wide kernels, with and without 4-byte rows; the first chunks so busy that their unit does not fit the LDS copy.
UNIT_CASES = [  # C, chunk, P
    (64, 64, 1000), (3, 65, 4000), (100, 2048, 2101), (24, 330, 3003), (32, 1056, 4000), (128, 2176, 1200), (144, 288, 1001),
    (160, 1000, 700), (50, 800, 1601), (200, 64, 777), (313, 1024, 430), (576, 1024, 641), (1000, 64, 150), (257, 600, 509),
    (960, 2048, 131),
    # a chunk per unit, by the wide decoder's tiles: 32 pixels and four, two or one wavefronts per channel tile, 64 and 128
    # pixels, workgroups that walk several tiles; the last pixel tile and the last channel group ragged
    (512, 4096, 121), (1023, 4096, 203), (500, 4096, 1728), (1000, 4096, 3001), (250, 4096, 9500), (170, 4096, 13001),
    (300, 4096, 12001), (640, 4096, 9001), (256, 4096, 33000),
]


@pytest.mark.parametrize("C,chunk,P", UNIT_CASES, ids=[f"C{c[0]}k{c[1]}P{c[2]}" for c in UNIT_CASES])
def test_decoder_of_small_chunks(fmtc, oracle, C, chunk, P):
    from paper_1905_10830_amd import synth

    bits, A = 8, np.float32(4.0)
    rng = np.random.default_rng(C + chunk)
    T = np.linalg.qr(rng.standard_normal((C, C)))[0].astype(np.float32)
    mu = rng.standard_normal(C).astype(np.float32)
    d = oracle.delta(A, bits)
    level = np.clip(np.rint(rng.laplace(0.0, 1.0, (P, C))), -128, 127)
    busy = min(P // 8, max(1, 4096 // C))
    level[:busy] = rng.integers(-128, 128, (busy, C))
    sym = (level + 128).astype(np.uint8)
    stream, nbytes = fmtc.code_symbols(dev(sym), C, bits, float(d), chunk)
    basis = fmtc.basis_import(T, mu, A)
    torch.cuda.synchronize()
    n = int(nbytes.item())
    back, err = fmtc.decode_symbols(stream, P, C, bits, nbytes=n)
    torch.cuda.synchronize()
    assert int(err.item()) == 0 and np.array_equal(back.cpu().numpy().reshape(P, C), sym)
    ref = (level * float(d)) @ T.astype(np.float64) + mu
    # as in test_planar_decoder
    tol = (2.0 ** -22 + C * 2.0 ** -24) * ((np.abs(level) * float(d)) @ np.abs(T.astype(np.float64)) + np.abs(mu)) + 1e-7
    for tag in (synth.NHWC, synth.NCHW):
        shape = (1, 1, P, C) if tag == synth.NHWC else (1, C, 1, P)
        out, err = fmtc.decode(basis, stream, shape, bits, tag, nbytes=n)
        torch.cuda.synchronize()
        assert int(err.item()) == 0
        out = out.cpu().numpy().reshape((P, C) if tag == synth.NHWC else (C, P))
        assert (np.abs((out if tag == synth.NHWC else out.T) - ref) <= tol).all()
    # 8-bit activations: the same values whatever the chunk size
    basis8 = fmtc.Basis8(basis, 0.05)
    plain, plain_bytes = fmtc.code_symbols(dev(sym), C, bits, float(d))
    outs = []
    for s, b in ((stream, nbytes), (plain, plain_bytes)):
        out, err = fmtc.decode_u8(basis8, s, (1, 1, P, C), bits, synth.NHWC, nbytes=int(b.item()))
        torch.cuda.synchronize()
        assert int(err.item()) == 0
        outs.append(out)
    assert torch.equal(outs[0], outs[1])
    # two neighbouring chunk offsets exchanged
    bad = stream[:n].clone()
    co = bad[320:320 + 16].view(torch.int32)
    co[[1, 2]] = co[[2, 1]]
    for decode in (lambda: fmtc.decode(basis, bad, (1, 1, P, C), bits, synth.NHWC), lambda: fmtc.decode_symbols(bad, P, C, bits)):
        _, err = decode()
        torch.cuda.synchronize()
        assert int(err.item()) & fmtc.ERR_OFFSETS
