"""GPU parity of the encoder with a code table fixed at calibration time: the table the library fits against the
oracle's (same counts), the stream against the oracle's packing of the same symbols with the same table, bit for
bit, and the unchanged decoder on those streams."""
import numpy as np
import pytest

from paper_1905_10830_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import RECON_TOL, check_symbols, dev, make_case  # noqa: E402


@pytest.fixture(scope="module")
def fmtc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_10830_amd import binding

    binding.load_library()
    return binding


# (C, H, W, calib images, data images, rank, act, bits, chunk_syms)
CASES = [
    (128, 28, 28, 2, 3, 32, "relu", 6, 4096),   # stage-2 shape: one chunk per 32-pixel tile
    (128, 28, 28, 2, 2, 32, "relu", 4, 4096),
    (64, 56, 56, 1, 1, 16, "relu", 8, 4096),    # two tiles per chunk
    (32, 9, 7, 1, 5, 8, "relu", 3, 4096),       # four tiles per chunk, ragged end
    (128, 5, 5, 1, 3, 32, "relu", 5, 4096),     # 75 pixels: last chunk and last tile partial
    (64, 28, 28, 1, 2, 16, "relu", 6, 1000),    # chunk size that is no multiple of a pixel
    (144, 13, 11, 2, 3, 18, "relu6", 5, 4096),
    (256, 14, 14, 2, 3, 64, "relu", 4, 4096),   # wide
    (50, 10, 10, 1, 2, 10, "relu", 5, 4096),
    (3, 17, 5, 1, 1, 2, "none", 2, 64),
]
IDS = [f"C{c[0]}_{c[1]}x{c[2]}_n{c[4]}_b{c[7]}_cs{c[8]}" for c in CASES]


def split_case(oracle, case, seed, layout):
    """Calibration tensor and a different data tensor of the same stream, basis fitted on the calibration part."""
    C, H, W, ncal, ndat, rank, act, bits, cs = case
    s = synth.FeatureMapStream(C, H, W, rank, act, seed)
    cal = synth.to_layout(s.images(ncal), layout)
    dat = synth.to_layout(s.images(ndat), layout)
    if C <= 160:
        T, mu, eig, A = oracle.fit(cal, layout)
    else:
        mean, cov = oracle.covariance(cal, layout)
        w, v = np.linalg.eigh(cov)
        T = np.ascontiguousarray(v[:, ::-1].T).astype(np.float32)
        mu = mean.astype(np.float32)
        A = np.float32(np.abs(oracle.project(cal, T, mu, layout)[:, 0]).max())
    return cal, dat, T, mu, A


@pytest.mark.parametrize("layout", [synth.NHWC, synth.NCHW], ids=["nhwc", "nchw"])
@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_static_table_encode_matches_oracle(fmtc, oracle, case, layout):
    C, H, W, ncal, ndat, rank, act, bits, cs = case
    cal, dat, T, mu, A = split_case(oracle, case, 700 + C, layout)
    d = oracle.delta(A, bits)
    K = 1 << bits
    basis = fmtc.basis_import(T, mu, A)

    # ---- the table: Huffman lengths of the calibration symbols' counts plus one ----
    table = fmtc.fit_table(basis, dev(cal), bits, layout)
    ln, tb = table.export()
    assert tb == bits and ln.size == K
    cal_sym, cal_hist = fmtc.quantize(basis, dev(cal), bits, layout)  # the symbols the fit counted
    torch.cuda.synchronize()
    cal_hist = cal_hist.cpu().numpy()[:K].astype(np.uint64)
    ref_sym, margin = oracle.quantize(oracle.project(cal, T, mu, layout), d, bits, want_margin=True)
    check_symbols(cal_sym.cpu().numpy(), ref_sym, margin)
    assert ln.tolist() == oracle.static_lengths(cal_hist).tolist()

    # ---- the stream of a tensor the table has not seen ----
    P = dat.size // C
    stream, nbytes = fmtc.encode_static(basis, table, dev(dat), layout, chunk_syms=cs)
    torch.cuda.synchronize()
    n = int(nbytes.item())
    got = stream[:n].cpu().numpy()
    sym_gpu, d2, pbits = oracle.unpack(got, P, C, bits)
    assert d2 == d
    ref = oracle.encode_static(dat, T, mu, d, bits, ln, layout, chunk_syms=cs)
    ref_margin = oracle.quantize(oracle.project(dat, T, mu, layout), d, bits, want_margin=True)[1]
    n_bad = check_symbols(sym_gpu, ref["sym"], ref_margin)
    again = ref["stream"] if n_bad == 0 else oracle.pack(sym_gpu, C, bits, d, ln, oracle.canonical_codes(ln),
                                                         chunk_syms=cs, cap=n + 4096)
    assert len(again) == n and (got == again).all(), "stream differs from the oracle's packing of the same symbols"
    assert got[64:64 + K].tolist() == ln.tolist() and not got[64 + K:320].any()
    assert pbits == int(ln[sym_gpu].astype(np.uint64).sum())
    info = fmtc.stream_info(got[:64])
    assert info["payload_bits"] == pbits and info["stream_bytes"] == n

    # ---- the decoder needs no change: the container carries the table ----
    xhat, err = fmtc.decode(basis, stream, dat.shape, bits, layout)
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    ref_xhat = oracle.reconstruct(sym_gpu, dat.shape, T, mu, d, bits, layout)
    assert np.abs(xhat.cpu().numpy().astype(np.float64) - ref_xhat).max() <= RECON_TOL
    # ... and the decoder that takes its tables ready-made from the handle gives the same tensor, bit for bit
    xhat_s, err_s = fmtc.decode_static(basis, table, stream, dat.shape, layout)
    torch.cuda.synchronize()
    assert int(err_s.item()) == 0 and torch.equal(xhat_s, xhat)
    # deterministic
    stream2, nbytes2 = fmtc.encode_static(basis, table, dev(dat), layout, chunk_syms=cs)
    torch.cuda.synchronize()
    assert int(nbytes2.item()) == n and (stream2[:n].cpu().numpy() == got).all()


@pytest.mark.parametrize("case", [CASES[0], CASES[2], CASES[3], CASES[4]], ids=[IDS[0], IDS[2], IDS[3], IDS[4]])
def test_single_kernel_and_two_kernel_paths_agree(fmtc, oracle, case, monkeypatch):
    """Small shapes, which take two kernels with and without that forced: the same call gives the same bytes."""
    C, H, W, ncal, ndat, rank, act, bits, cs = case
    cal, dat, T, mu, A = split_case(oracle, case, 750 + C, synth.NHWC)
    basis = fmtc.basis_import(T, mu, A)
    table = fmtc.fit_table(basis, dev(cal), bits)
    a, na = fmtc.encode_static(basis, table, dev(dat))
    torch.cuda.synchronize()
    fmtc.test_option(fmtc.TEST_STATIC_TWO_KERNELS, 1)
    try:
        b, nb = fmtc.encode_static(basis, table, dev(dat))
        torch.cuda.synchronize()
    finally:
        fmtc.test_option(fmtc.TEST_STATIC_TWO_KERNELS, 0)
    n = int(na.item())
    assert int(nb.item()) == n and (a[:n] == b[:n]).all()


def one_kernel(fmtc, call):
    """Whether `call` launched the one-kernel encoder (projection without a packing kernel after it)."""
    fmtc.profile_enable(4)
    try:
        call()
        torch.cuda.synchronize()
        launches = {k: v[2] for k, v in fmtc.profile_read().items()}
    finally:
        fmtc.profile_enable(0)
    assert launches["k_project_quantize"] == 1
    return not launches.get("k_pack", 0)


# The sizes of the one-kernel encoder (145 chunk groups of four chunks to one per compute unit) against the oracle: pixels
# beyond f16, a truncated basis, a last group of one to four chunks and a last chunk that is not full, a buffer too small.
@pytest.mark.parametrize("keep", [None, 9])
@pytest.mark.parametrize("C,bits,layout,groups", [(64, 4, synth.NHWC, 144.3), (64, 6, synth.NHWC, 200.8), (64, 8, synth.NHWC, 256.0),
                                                  (64, 8, synth.NCHW, 150.5), (32, 8, synth.NHWC, 145.7)])
def test_one_kernel_encoder_matches_oracle(fmtc, oracle, C, bits, layout, groups, keep):
    P, K = int(groups * 4 * 4096) // C // 2 * 2, 1 << bits
    rng = np.random.default_rng(C + bits)
    T = np.linalg.qr(rng.standard_normal((C, C)))[0].astype(np.float32)
    mu = rng.standard_normal(C).astype(np.float32)
    x = (rng.standard_normal((P, C)) * np.linspace(2.0, 0.1, C) + mu).astype(np.float32)
    x[5, 3], x[40, C - 1], x[100, 0], x[P - 1, 1] = 3.0e5, -7.0e6, 1.0e25, 7.0e4
    x[41] *= 1.0e4
    A = np.float32(6.0)
    d = oracle.delta(A, bits)
    y = (x.astype(np.float64) - mu) @ T.T.astype(np.float64)
    basis = fmtc.basis_import(T, mu, A)
    if keep:
        y[:, keep:] = 0.0
        basis = basis.truncate(keep)
    sym, margin = oracle.quantize(y, d, bits, want_margin=True)
    ln = oracle.static_lengths(oracle.histogram(sym, bits)[:K])
    table = fmtc.table_import(ln, bits)
    xs = dev(x.reshape(1, 2, P // 2, C) if layout == synth.NHWC else np.ascontiguousarray(x.T).reshape(1, C, 2, P // 2))
    stream, nbytes = fmtc.encode_static(basis, table, xs, layout)
    assert one_kernel(fmtc, lambda: fmtc.encode_static(basis, table, xs, layout, stream_out=stream, out_bytes=nbytes))
    n = int(nbytes.item())
    got = stream[:n].cpu().numpy()
    sym_gpu, _, pbits = oracle.unpack(got, P, C, bits)
    diff = sym_gpu.reshape(P, C) != sym.reshape(P, C)
    assert not diff.any() or margin.reshape(P, C)[diff].max() <= 1e-9  # (the order of an fp64 sum)
    ref = oracle.pack(sym_gpu, C, bits, d, ln, oracle.canonical_codes(ln), cap=n + 4096)
    assert n == len(ref) and np.array_equal(got, ref)
    # a buffer that holds about half of the payload: nothing past it, and no valid stream
    small = n - int(pbits) // 16
    guard = torch.full((small + 8192,), 0xAB, dtype=torch.uint8, device="cuda")
    fmtc.encode_static(basis, table, xs, layout, stream_out=guard[:small])
    torch.cuda.synchronize()
    assert (guard[small:] == 0xAB).all(), "wrote past the capacity it was given"
    _, err = fmtc.decode_symbols(guard[:small], P, C, bits)
    torch.cuda.synchronize()
    assert int(err.item()) & fmtc.ERR_HEADER


# Around the number of chunk groups from which one kernel is used (four chunks a group: two kernels at 144 of them, one at
# 145), a last group of one chunk, and the largest number (one group per compute unit)
@pytest.mark.parametrize("C,bits,layout", [(64, 5, synth.NHWC), (64, 8, synth.NHWC), (64, 8, synth.NCHW), (32, 8, synth.NHWC)])
@pytest.mark.parametrize("groups", [144.0, 144.25, 160.5, 256.0])
def test_one_kernel_and_two_agree_on_larger_tensors(fmtc, C, bits, layout, groups):
    P = int(groups * 4 * 4096) // C
    rng = np.random.default_rng(C + bits)
    T = np.linalg.qr(rng.standard_normal((C, C)))[0].astype(np.float32)
    x = (rng.standard_normal((P, C)) * np.linspace(2.0, 0.1, C)).astype(np.float32)
    basis = fmtc.basis_import(T, np.zeros(C, np.float32), np.float32(8.0))
    xs = dev(x.reshape(1, P // 32, 32, C) if layout == synth.NHWC else x.T.reshape(1, C, P // 32, 32))
    table = fmtc.fit_table(basis, xs, bits, layout)
    a, na = fmtc.encode_static(basis, table, xs, layout)
    assert one_kernel(fmtc, lambda: fmtc.encode_static(basis, table, xs, layout, stream_out=a, out_bytes=na)) == (
        groups > 144 and (C == 64 and layout == synth.NHWC or bits == 8))
    fmtc.test_option(fmtc.TEST_STATIC_TWO_KERNELS, 1)
    try:
        b, nb = fmtc.encode_static(basis, table, xs, layout)
        torch.cuda.synchronize()
    finally:
        fmtc.test_option(fmtc.TEST_STATIC_TWO_KERNELS, 0)
    n = int(na.item())
    assert int(nb.item()) == n and (a[:n] == b[:n]).all()


def test_table_import_export_and_bad_tables(fmtc, oracle):
    case = CASES[1]
    C, H, W, ncal, ndat, rank, act, bits, cs = case
    cal, dat, T, mu, A = split_case(oracle, case, 811, synth.NHWC)
    basis = fmtc.basis_import(T, mu, A)
    fitted = fmtc.fit_table(basis, dev(cal), bits)
    ln, _ = fitted.export()
    imported = fmtc.table_import(ln, bits)
    assert imported.export()[0].tolist() == ln.tolist()
    a, na = fmtc.encode_static(basis, fitted, dev(dat))
    b, nb = fmtc.encode_static(basis, imported, dev(dat))
    torch.cuda.synchronize()
    n = int(na.item())
    assert int(nb.item()) == n and (a[:n] == b[:n]).all()
    # a long-code table (lengths 1, 2, ..., 15, 15) through the same path
    skew = np.array(list(range(1, 16)) + [15], np.uint8)
    long_table = fmtc.table_import(skew, 4)
    stream, nbytes = fmtc.encode_static(basis, long_table, dev(dat))
    torch.cuda.synchronize()
    n = int(nbytes.item())
    got = stream[:n].cpu().numpy()
    sym_gpu, d2, pbits = oracle.unpack(got, dat.size // C, C, bits)
    d = oracle.delta(A, bits)
    again = oracle.pack(sym_gpu, C, bits, d, skew, oracle.canonical_codes(skew), cap=n + 4096)
    assert len(again) == n and (got == again).all()
    # not a complete prefix code: rejected on the host
    for bad in (np.full(16, 3, np.uint8), np.array([1] + [0] * 15, np.uint8), np.full(16, 5, np.uint8)):
        with pytest.raises(fmtc.FmtcError) as e:
            fmtc.table_import(bad, 4)
        assert e.value.status == fmtc.EINVAL
    # a table of another bit depth than the basis' step is fine (the step follows the table's bits), but the channel
    # count must match the basis
    with pytest.raises(fmtc.FmtcError) as e:
        fmtc.encode_static(basis, fitted, torch.zeros((1, 4, 4, 16), device="cuda"))
    assert e.value.status == fmtc.EINVAL


@pytest.mark.parametrize("case", [CASES[1], CASES[7]], ids=[IDS[1], IDS[7]])
def test_static_decoder_refuses_a_stream_of_another_table(fmtc, oracle, case):
    C, H, W, ncal, ndat, rank, act, bits, cs = case
    cal, dat, T, mu, A = split_case(oracle, case, 813, synth.NHWC)
    basis = fmtc.basis_import(T, mu, A)
    table = fmtc.fit_table(basis, dev(cal), bits)
    ln, _ = table.export()
    # the tensor's own table differs from the calibration table (at least one length)
    own, nown = fmtc.encode(basis, dev(dat), bits)
    torch.cuda.synchronize()
    own_len = own[64:64 + (1 << bits)].cpu().numpy()
    assert own_len.tolist() != ln.tolist()
    xhat, err = fmtc.decode_static(basis, table, own, dat.shape)
    torch.cuda.synchronize()
    assert int(err.item()) & fmtc.ERR_TABLE
    # the general decoder reads it, and a damaged stream of the right table still raises its flag
    xhat, err = fmtc.decode(basis, own, dat.shape, bits)
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    good, ngood = fmtc.encode_static(basis, table, dev(dat))
    torch.cuda.synchronize()
    bad = good.clone()
    bad[320 + 7] = 0xFF  # a chunk offset far past the payload
    xhat, err = fmtc.decode_static(basis, table, bad, dat.shape)
    torch.cuda.synchronize()
    assert int(err.item()) & fmtc.ERR_OFFSETS


def test_static_stream_that_outgrows_its_buffer_is_marked_invalid(fmtc, oracle):
    case = CASES[1]
    C, H, W, ncal, ndat, rank, act, bits, cs = case
    cal, dat, T, mu, A = split_case(oracle, case, 812, synth.NHWC)
    basis = fmtc.basis_import(T, mu, A)
    table = fmtc.fit_table(basis, dev(cal), bits)
    P = dat.size // C
    full = fmtc.encode_static_bound(table, P, C)
    good, ngood = fmtc.encode_static(basis, table, dev(dat))
    torch.cuda.synchronize()
    need = int(ngood.item())
    small = need - 4096  # room for the side information and most, not all, of the payload
    assert small < need <= full
    guard = torch.full((small + 4096,), 0xAB, dtype=torch.uint8, device="cuda")
    fmtc.encode_static(basis, table, dev(dat), stream_out=guard[:small])
    torch.cuda.synchronize()
    assert (guard[small:] == 0xAB).all(), "wrote past the capacity it was given"
    xhat, err = fmtc.decode(basis, guard[:small], dat.shape, bits)
    torch.cuda.synchronize()
    assert int(err.item()) & fmtc.ERR_HEADER
