"""GPU parity: every C-ABI entry point against the CPU oracle on the same seeded inputs.

Bars: packed words and integer results bit-exact; fp32 results within 1e-6 relative of the
oracle (they are in practice bit-identical: one fp32 multiply or one IEEE division of an
exactly representable integer).  All calls go through paper_1705_09864_amd.binding, i.e.
through the C ABI of libbmx.so.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1705_09864_amd import binding as B
from paper_1705_09864_amd import synth

pytestmark = pytest.mark.gpu
RTOL = 1e-6
POISON = np.uint64(0xCDCDCDCDCDCDCDCD)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host_u64(t):
    return t.cpu().numpy().view(np.uint64)


def assert_f32_close(got, ref, atol=0.0):
    """|got - ref| <= 1e-6 * |ref| (+ atol).  atol is non-zero only against the oracle's
    double-precision sum of quantised values, whose own rounding noise (about K * 2^-53 * K,
    below 1e-9 for every K used here) is all that separates it from the exact rational."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    err = np.abs(got - ref)
    assert (err <= RTOL * np.abs(ref) + atol).all(), "max rel err %g" % (err / np.maximum(np.abs(ref), 1e-30)).max()


# ------------------------------------------------------------------ binarize + pack
@pytest.mark.parametrize("rows,K", [(1, 1), (3, 63), (2, 64), (5, 65), (7, 500), (4, 576), (3, 1000),
                                    (9, 4095), (33, 512), (2, 8192), (130, 27)])
def test_pack_rows(rows, K):
    rng = np.random.default_rng(rows * 100003 + K)
    x = rng.standard_normal((rows, K)).astype(np.float32)
    x.flat[:: 7] = 0.0
    x.flat[3:: 11] = -0.0
    got = host_u64(B.binarize_pack(dev(x), 1))
    np.testing.assert_array_equal(got, oracle.binarize_pack(x, 1))


def test_pack_rows_special_values():
    v = np.array([0.0, -0.0, 1e-45, -1e-45, 1.1754942e-38, -1.1754942e-38, np.inf, -np.inf,
                  1.0, -1.0, 3e38, -3e38, np.nan, -np.nan, 2.5, -2.5], dtype=np.float32)
    x = np.tile(v, 16)[None, :].copy()
    got = host_u64(B.binarize_pack(dev(x), 1))
    np.testing.assert_array_equal(got, oracle.binarize_pack(x, 1))  # negative denormals stay -1
    # the pattern itself, from the reading of the sign function: (x >= 0) as an IEEE compare,
    # so +-0, positive denormals and +inf give 1, NaN of either sign gives 0
    assert got[0, 0] & np.uint64(0xFFFF) == np.uint64(0b0100_0101_0101_0111)
    # the same values down a strided column and through the channel pack of a convolution
    col = np.tile(v, 8)[:, None] * np.ones((1, 3), dtype=np.float32)
    np.testing.assert_array_equal(host_u64(B.binarize_pack(dev(col), 0)), oracle.binarize_pack(col, 0))


def test_conv_special_values_in_the_image():
    """NaN, +-0, denormals and infinities in a convolution input: the channel pack takes the same
    IEEE compare as the row pack, and the layer equals the oracle's (which binarises the
    zero-padded float image element by element)."""
    v = np.array([0.0, -0.0, 1e-45, -1e-45, np.inf, -np.inf, np.nan, -np.nan, 1.0, -1.0], dtype=np.float32)
    rng = np.random.default_rng(41)
    x = rng.choice(v, size=(2, 70, 9, 7)).astype(np.float32)
    w = rng.standard_normal((5, 70, 3, 3)).astype(np.float32)
    ri, _ = oracle.binary_conv2d(x, w, 1, 1)
    np.testing.assert_array_equal(run_conv(x, w, 1, 1, integer_out=True), ri)
    xp = host_u64(B.pack_nchw(dev(x), 0))
    rows = np.transpose(x, (0, 2, 3, 1)).reshape(-1, 70)
    np.testing.assert_array_equal(xp.reshape(-1, 2), oracle.binarize_pack(rows, 1))


@pytest.mark.parametrize("N,H,W", [(65535, 129, 129), (1, 32768, 32768)])
def test_channel_pack_of_2_to_30_pixels(N, H, W):
    """More pixels than a launch has threads for, over many images and in one: every word, halo included."""
    x = torch.empty((N, 1, H, W), device="cuda").uniform_(-1.0, 1.0)
    xp = B.pack_nchw(x, 1).view(N, H + 2, W + 2)
    assert torch.equal(xp[:, 1:-1, 1:-1], (x >= 0).view(N, H, W).to(torch.int64))
    xp[:, 1:-1, 1:-1] = 1
    assert bool((xp == 1).all())
    del x, xp
    torch.cuda.empty_cache()


def test_pack_rows_strided_and_poisoned():
    rng = np.random.default_rng(11)
    rows, K, ldx, ld = 6, 200, 260, 6
    buf = rng.standard_normal((rows, ldx)).astype(np.float32)
    xd = dev(buf)[:, :K]
    out = torch.from_numpy(np.full((rows, ld), POISON, dtype=np.uint64).view(np.int64)).cuda()
    B.binarize_pack(xd, 1, out=out)
    got = host_u64(out)
    ref = oracle.binarize_pack(buf[:, :K].copy(), 1, out_ld_words=ld, fill=POISON)
    np.testing.assert_array_equal(got, ref)       # tail bits 0, words past Kw untouched


@pytest.mark.parametrize("K,N", [(1, 1), (64, 64), (65, 3), (130, 7), (512, 256), (500, 300), (27, 1000)])
def test_pack_dim0(K, N):
    rng = np.random.default_rng(K * 7919 + N)
    x = rng.standard_normal((K, N)).astype(np.float32)
    got = host_u64(B.binarize_pack(dev(x), 0))
    np.testing.assert_array_equal(got, oracle.binarize_pack(x, 0))


# ------------------------------------------------------------------ xnor GEMM
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (4, 4, 64), (3, 5, 65), (17, 29, 333), (64, 256, 512),
                                   (70, 130, 1000), (33, 300, 2304), (129, 65, 4095), (8, 600, 576)])
def test_xnor_gemm(M, N, K):
    rng = np.random.default_rng(M * 31 + N * 17 + K)
    A = oracle.binarize_pack(rng.standard_normal((M, K)).astype(np.float32), 1)
    Bm = oracle.binarize_pack(rng.standard_normal((N, K)).astype(np.float32), 1)
    got = B.xnor_gemm(dev(A.view(np.int64)), dev(Bm.view(np.int64)), K).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.xnor_gemm(A, Bm, K))


@pytest.mark.parametrize("engine", [1, 2, 3])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (5, 7, 63), (33, 65, 500), (70, 130, 1100), (256, 300, 4096)])
def test_xnor_gemm_count_range(M, N, K, engine):
    """The other range of Eq. 2: the number of agreeing positions, counted from the definition on
    the unpacked +-1 values, from every GEMM engine (rows padded to an even word count so that
    the matrix-core kernels take the problem)."""
    rng = np.random.default_rng(M + N + K)
    a = rng.standard_normal((M, K)).astype(np.float32)
    b = rng.standard_normal((N, K)).astype(np.float32)
    want = (oracle.sign(a)[:, None, :] == oracle.sign(b)[None, :, :]).sum(axis=2).astype(np.int32)

    def even_rows(x):
        p = oracle.binarize_pack(x, 1)
        out = np.zeros((p.shape[0], (p.shape[1] + 1) // 2 * 2), dtype=np.uint64)
        out[:, :p.shape[1]] = p
        return dev(out.view(np.int64))

    with tuned(k7=engine):
        got = B.xnor_gemm(even_rows(a), even_rows(b), K, count=True).cpu().numpy()
    np.testing.assert_array_equal(got, want)
    np.testing.assert_array_equal(2 * got - K, oracle.xnor_gemm(oracle.binarize_pack(a, 1), oracle.binarize_pack(b, 1), K))


def test_xnor_gemm_wide_rows_and_invariants():
    """Row stride wider than ceil(K/64): extra words are ignored (they hold garbage here)."""
    rng = np.random.default_rng(5)
    M, N, K = 20, 40, 200
    a = rng.standard_normal((M, K)).astype(np.float32)
    A = oracle.binarize_pack(a, 1, out_ld_words=6, fill=POISON)
    Bm = oracle.binarize_pack(rng.standard_normal((N, K)).astype(np.float32), 1, out_ld_words=5,
                              fill=POISON)
    got = B.xnor_gemm(dev(A.view(np.int64)), dev(Bm.view(np.int64)), K).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.xnor_gemm(A, Bm, K))
    assert (np.abs(got) <= K).all() and ((got - K) % 2 == 0).all()
    same = B.xnor_gemm(dev(A.view(np.int64)), dev(A.view(np.int64)), K).cpu().numpy()
    assert (np.diag(same) == K).all()


class tuned:
    """Pin kernel choices through bmx_tune_set for a block of code (results must not depend on them)."""

    def __init__(self, **kv):
        self.kv = kv

    def __enter__(self):
        for k, v in self.kv.items():
            assert B.lib().bmx_tune_set(int(k[1:]), v) == 0
        return self

    def __exit__(self, *exc):
        for k in self.kv:
            B.lib().bmx_tune_set(int(k[1:]), 0)


# every GEMM engine: automatic (FP4 matrix cores), xor/popcount, int8 matrix cores
GEMM_ENGINES = [dict(), dict(k7=1), dict(k7=2)]


# ------------------------------------------------------------------ binary FC
def test_config1_fc_gemm_exact():
    c = synth.config1()
    a, w_kn = c["a"], c["w_kn"]                       # A [64,512], W stored [K=512, N=256]
    Wp = B.binarize_pack(dev(w_kn), 0)                # pack down the K rows -> [256, 8]
    np.testing.assert_array_equal(host_u64(Wp), oracle.binarize_pack(w_kn, 0))
    got = B.binary_fc(dev(a), Wp, integer_out=True).cpu().numpy()
    assert "fc_small_kernel" in B.last_kernel()       # the one-launch form of very small layers
    ref, _ = oracle.binary_fc(a, w_kn.T.copy())
    assert got.dtype == np.int32 and got.shape == (64, 256)
    np.testing.assert_array_equal(got, ref)
    with tuned(k15=1):                                 # the general path: pack, then the GEMM
        got = B.binary_fc(dev(a), Wp, integer_out=True).cpu().numpy()
        assert "fc_small_kernel" not in B.last_kernel()
        np.testing.assert_array_equal(got, ref)
    # the same through pack + xnor_gemm
    Ap = B.binarize_pack(dev(a), 1)
    np.testing.assert_array_equal(B.xnor_gemm(Ap, Wp, 512).cpu().numpy(), ref)


@pytest.mark.parametrize("small", [True, False])
def test_config3_fc_chain(small):
    c = synth.config3(small=small)
    x, w1, w2 = c["x"], c["w1"], c["w2"]
    a1, a2 = oracle.alpha_mean_abs(w1), oracle.alpha_mean_abs(w2)
    W1p, W2p = B.binarize_pack(dev(w1), 1), B.binarize_pack(dev(w2), 1)
    r1i, r1f = oracle.binary_fc(x, w1, a1)
    r2i, r2f = oracle.binary_fc(r1f, w2, a2)
    for engine in GEMM_ENGINES:
        with tuned(**engine):
            h1 = B.binary_fc(dev(x), W1p, alpha=dev(a1))
            h2 = B.binary_fc(h1, W2p, alpha=dev(a2))
            i1 = B.binary_fc(dev(x), W1p, integer_out=True)
            np.testing.assert_array_equal(i1.cpu().numpy(), r1i)
            assert_f32_close(h1.cpu().numpy(), r1f)
            np.testing.assert_array_equal(h1.cpu().numpy(), r1f)   # one fp32 multiply: bit-identical
            assert_f32_close(h2.cpu().numpy(), r2f)
            i2 = B.binary_fc(h1, W2p, integer_out=True)
            np.testing.assert_array_equal(i2.cpu().numpy(), r2i)


@pytest.mark.parametrize("batch,fin,fout", [(1, 1, 1), (64, 512, 256), (7, 65, 3), (100, 1000, 70), (4096, 64, 1),
                                            (3, 64 * 33 + 5, 7), (2, 65536, 16), (33, 4000, 257), (1, 130, 5000)])
def test_fc_small_layers_one_launch(batch, fin, fout):
    """bmx_binary_fc on layers small enough for its one-launch form (sign bits of a batch row in
    LDS, xor + popcount per output feature): K tails inside a word, more and fewer than four
    words per wave, more than 256 output features, rows of x and of the output further apart
    than their length with poison between them, special values in x; int32 and scaled fp32."""
    rng = np.random.default_rng(batch + 3 * fin + 7 * fout)
    x = rng.standard_normal((batch, fin)).astype(np.float32)
    x.flat[:: 7] = 0.0
    x.flat[3:: 11] = -0.0
    x.flat[5:: 13] = np.nan
    x.flat[1:: 17] = np.inf
    x.flat[2:: 19] = -np.inf
    w = rng.uniform(-1, 1, (fout, fin)).astype(np.float32)
    alpha = rng.standard_normal(fout).astype(np.float32)
    alpha[::3] = 0.0
    ri, rf = oracle.binary_fc(x, w, alpha)
    Wp = B.binarize_pack(dev(w), 1)
    xw = torch.full((batch, fin + 5), float("nan"), dtype=torch.float32, device="cuda")   # rows fin + 5 apart
    xw[:, :fin] = dev(x)
    oi = torch.full((batch, fout + 3), -7, dtype=torch.int32, device="cuda")
    of = torch.full((batch, fout + 3), 123.0, dtype=torch.float32, device="cuda")
    B.binary_fc(xw[:, :fin], Wp, integer_out=True, out=oi[:, :fout])
    assert "fc_small_kernel" in B.last_kernel()
    B.binary_fc(xw[:, :fin], Wp, alpha=dev(alpha), out=of[:, :fout])
    assert "fc_small_kernel" in B.last_kernel()
    np.testing.assert_array_equal(oi[:, :fout].cpu().numpy(), ri)
    np.testing.assert_array_equal(of[:, :fout].cpu().numpy(), rf)      # one fp32 multiply: bit-identical
    assert (oi[:, fout:] == -7).all() and (of[:, fout:] == 123.0).all()
    np.testing.assert_array_equal(B.binary_fc(dev(x), Wp).cpu().numpy(), ri.astype(np.float32))
    with tuned(k15=1):
        np.testing.assert_array_equal(B.binary_fc(dev(x), Wp, integer_out=True).cpu().numpy(), ri)
        assert "fc_small_kernel" not in B.last_kernel()


@pytest.mark.parametrize("batch,fin,fout,call,graph,static", [
    (241, 3596, 440, True, True, True), (600, 600, 1400, True, False, True), (600, 512, 1400, True, True, True), (168, 2432, 1064, True, False, True),  # one round of workgroups
    (900, 127, 1900, False, False, True), (892, 318, 1100, True, True, True), (892, 322, 1130, False, False, True),  # several
    (2, 65536, 16, True, True, True), (1000, 130, 2000, False, False, False)])
def test_fc_small_lines(batch, fin, fout, call, graph, static):
    """The lines between one launch and two, for calls, captured calls and calls on the library's scratch memory; replays between
    calls give what the calls give."""
    g = torch.Generator(device="cuda")
    g.manual_seed(fin)
    x = torch.randn((batch, fin), device="cuda", generator=g)
    w = torch.randn((fout, fin), device="cuda", generator=g)
    Wp, alpha = B.binarize_pack(w, 1), B.alpha_mean_abs(w)
    run = lambda: B.binary_fc(x, Wp, alpha=alpha)  # noqa: E731
    out_static = torch.empty((batch, fout), device="cuda")
    for f, one in ((run, call), (lambda: B.binary_fc_static(x, Wp, alpha=alpha, out=out_static), static)):
        f()
        assert ("fc_small" in B.last_kernel()) == one, B.last_kernel()
    torch.cuda.synchronize()
    captured, captured_static = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(captured):
        out = run()
        assert ("fc_small" in B.last_kernel()) == graph, B.last_kernel()
    with torch.cuda.graph(captured_static):
        B.binary_fc_static(x, Wp, alpha=alpha, out=out_static)
        assert ("fc_small" in B.last_kernel()) == static, B.last_kernel()
    for _ in range(3):
        x.normal_(generator=g)
        captured.replay()
        captured_static.replay()
        want = run()
        assert ("fc_small" in B.last_kernel()) == call, B.last_kernel()
        assert torch.equal(out, want) and torch.equal(out_static, want)
        with tuned(k15=1):
            assert torch.equal(run(), want)


@pytest.mark.parametrize("batch,fin,fout", [(1, 512, 1), (3, 513, 17), (5, 1024, 33), (6, 1025, 40), (9, 2049, 31), (4, 3073, 65),
                                            (7, 4097, 50), (2, 8193, 130), (8, 12289, 20), (3, 20481, 9), (33, 2048, 600)])
def test_fc_small_row_lengths(batch, fin, fout):
    """Every split of a row over lanes (4, 16 or 64 of them, two to four words each), at the row
    lengths where it changes, with rows and features that do not fill their workgroup."""
    rng = np.random.default_rng(fin)
    x = rng.standard_normal((batch, fin)).astype(np.float32)
    w = rng.uniform(-1, 1, (fout, fin)).astype(np.float32)
    alpha = rng.standard_normal(fout).astype(np.float32)
    ri, rf = oracle.binary_fc(x, w, alpha)
    Wp = B.binarize_pack(dev(w), 1)
    np.testing.assert_array_equal(B.binary_fc(dev(x), Wp, integer_out=True).cpu().numpy(), ri)
    assert "fc_small_kernel" in B.last_kernel()
    np.testing.assert_array_equal(B.binary_fc(dev(x), Wp, alpha=dev(alpha)).cpu().numpy(), rf)


@pytest.mark.parametrize("lanes,words,waves,batch,fin,fout", [
    (4, 2, 4, 3, 64, 714), (4, 4, 4, 2, 1024, 16), (4, 3, 12, 100, 2100, 1000), (16, 3, 12, 23, 3072, 1920), (16, 3, 12, 599, 2940, 64),
    (16, 2, 4, 1, 1280, 64), (4, 4, 16, 213, 1916, 941), (16, 3, 16, 23, 4206, 1920), (64, 2, 8, 5, 5593, 64), (64, 3, 12, 1, 9216, 4096), (64, 4, 16, 2, 15400, 33)])
def test_fc_small_lanes_and_waves(lanes, words, waves, batch, fin, fout):
    """The one-launch layer's lanes a feature, words a lane and waves a workgroup, rows in one to three steps, features and rows
    that do not fill a pass, rows further apart than their length."""
    rng = np.random.default_rng(fin + fout)
    x, w = rng.standard_normal((batch, fin + 1)).astype(np.float32), rng.standard_normal((fout, fin)).astype(np.float32)
    x[rng.random(x.shape) < 0.02] = -0.0
    x[rng.random(x.shape) < 0.02] = np.nan
    ri, _ = oracle.binary_fc(x[:, :fin].copy(), w)
    got = B.binary_fc(dev(x)[:, :fin], B.binarize_pack(dev(w)), integer_out=True)
    assert "fc_small_kernel<" in B.last_kernel() and ",%d,%d> " % (lanes, words) in B.last_kernel() and "x %d," % (64 * waves) in B.last_kernel(), B.last_kernel()
    np.testing.assert_array_equal(got.cpu().numpy(), ri)


@pytest.mark.parametrize("batch,fin,fout", [(1, 1, 1), (5, 27, 3), (3, 180, 70), (66, 1000, 130)])
def test_fc_ragged(batch, fin, fout):
    rng = np.random.default_rng(batch + fin + fout)
    x = rng.standard_normal((batch, fin)).astype(np.float32)
    w = rng.uniform(-1, 1, (fout, fin)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    Wp = B.binarize_pack(dev(w), 1)
    ri, rf = oracle.binary_fc(x, w, alpha)
    np.testing.assert_array_equal(B.binary_fc(dev(x), Wp, integer_out=True).cpu().numpy(), ri)
    assert_f32_close(B.binary_fc(dev(x), Wp, alpha=dev(alpha)).cpu().numpy(), rf)


# ------------------------------------------------------------------ binary conv2d
CONV_CASES = [
    # N, C, H, W, O, k, s, p
    (1, 1, 1, 1, 1, 1, 1, 0),
    (2, 3, 5, 5, 4, 3, 1, 1),
    (1, 20, 8, 5, 3, 3, 2, 1),
    (2, 64, 5, 8, 5, 3, 1, 1),
    (1, 65, 8, 8, 2, 5, 2, 2),
    (1, 3, 8, 8, 2, 5, 1, 0),
    (1, 2, 2, 2, 3, 3, 1, 1),
    (2, 4, 7, 7, 3, 1, 2, 0),
    (1, 5, 9, 9, 2, 7, 1, 3),
    (3, 130, 9, 11, 70, 3, 1, 1),
    (2, 64, 56, 56, 64, 3, 1, 1),
    (2, 128, 28, 28, 128, 3, 2, 1),
    (1, 256, 14, 14, 19, 3, 1, 2),
]


def run_conv(x, w, s, p, alpha=None, integer_out=False):
    O, C, KH, KW = w.shape
    Wp = B.pack_conv_weights(dev(w))
    out = B.binary_conv2d(dev(x), Wp, O, KH, KW, s, p, alpha=None if alpha is None else dev(alpha),
                          integer_out=integer_out)
    return out.cpu().numpy()


@pytest.mark.parametrize("N,C,H,W,O,k,s,p", CONV_CASES)
def test_conv_cases(N, C, H, W, O, k, s, p):
    rng = np.random.default_rng(N + 10 * C + 100 * H + 1000 * O + k + s + p)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    np.testing.assert_array_equal(run_conv(x, w, s, p, integer_out=True), ri)
    got = run_conv(x, w, s, p, alpha=alpha)
    assert_f32_close(got, rf)


def test_conv_output_offsets_beyond_two_gib():
    """A convolution whose fp32 output is 3.3 GB (130 x 512 x 112 x 112): the short-K matrix-core
    kernel addresses its output with 32-bit byte offsets from a uniform base, which here pass
    2^31.  The first, one middle and the last image against the oracle (image by image: the
    oracle would need minutes for the whole batch), every other image against the popcount
    kernel on a sample of rows."""
    N, C, H, W, O = 130, 64, 112, 112, 512
    gen = torch.Generator(device="cuda").manual_seed(130)
    x = torch.randn((N, C, H, W), device="cuda", generator=gen)
    rng = np.random.default_rng(130)
    w = rng.standard_normal((O, C, 3, 3)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    Wp = B.pack_conv_weights(dev(w))
    got = B.binary_conv2d(x, Wp, O, 3, 3, 1, 1, alpha=dev(alpha))
    assert "conv_mfma_ws_kernel" in B.last_kernel()
    assert got.shape == (N, O, H, W) and got.numel() * 4 > 2 ** 31
    for n in (0, 77, N - 1):
        _, rf = oracle.binary_conv2d(x[n:n + 1].cpu().numpy(), w, 1, 1, alpha)
        assert_f32_close(got[n:n + 1].cpu().numpy(), rf)
    with tuned(k5=1):
        ref = B.binary_conv2d(x, Wp, O, 3, 3, 1, 1, alpha=dev(alpha))
        assert "conv_stationary_kernel" in B.last_kernel()
    assert torch.equal(got[:, ::37], ref[:, ::37])
    del got, ref, x
    torch.cuda.empty_cache()


@pytest.mark.parametrize("C,k", [(64, 3), (100, 3), (64, 5), (192, 3), (200, 3), (40, 7), (128, 5)])
@pytest.mark.parametrize("integer_out", [False, True])
def test_conv_result_stores_with_and_without_the_streaming_hint(C, k, integer_out):
    """Planes that are not whole 128-byte lines: a result of more than 20 MB leaves through the caches, its parts of
    ten images bypass them, each in a kernel of its own; blocks inside the result and at both its edges."""
    N, H, O = 130, 33, 40
    rng = np.random.default_rng(C + k)
    x = rng.standard_normal((N, C, H, H)).astype(np.float32)
    w = rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    got = run_conv(x, w, 1, k // 2, alpha=None if integer_out else alpha, integer_out=integer_out)
    assert "conv_mfma_ws_kernel" in B.last_kernel() and got.nbytes > 20 << 20
    for n in range(0, N, 10):
        part = run_conv(x[n:n + 10], w, 1, k // 2, alpha=None if integer_out else alpha, integer_out=integer_out)
        np.testing.assert_array_equal(got[n:n + 10], part)
    ri, rf = oracle.binary_conv2d(x[-1:], w, 1, k // 2, alpha)
    if integer_out:
        np.testing.assert_array_equal(got[-1:], ri)
    else:
        assert_f32_close(got[-1:], rf)


@pytest.mark.parametrize("N,C,H,W,O,k", [
    (48, 64, 20, 20, 96, 3),     # 9 words, planes of whole 64-byte halves: hint
    (1100, 40, 16, 16, 42, 3),   # the same past 44 MB: none
    (60, 64, 21, 19, 70, 3),     # 9 words, parts of lines: none
    (75, 100, 33, 33, 40, 3),    # 18 words, 13 MB (none), and
    (50, 128, 33, 33, 40, 3),    # 8.7 MB: hint
    (70, 200, 31, 33, 40, 3), (25, 250, 31, 33, 39, 3),  # 36 words, 11 MB (hint) and 4 MB (none)
    (130, 33, 25, 26, 38, 5)])   # 25 words, 12 MB: hint
def test_conv_ws_blocks_in_turn_and_hint(N, C, H, W, O, k):
    """Several pixel blocks per wave, taken in turn by the waves of a workgroup, blocks that straddle images and
    the result's edge, and either kind of result store: the whole batch against its images one by one, on a kernel that
    holds a single block per wave, and a few against the oracle."""
    rng = np.random.default_rng(N + C + H)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    Wp, xp = B.pack_conv_weights(dev(w)), B.pack_nchw(dev(x), k // 2)
    with tuned(k18=1):
        got = B.binary_conv2d_packed(xp, C, Wp, O, k, k, 1, k // 2, alpha=dev(alpha))
        assert "conv_mfma_ws_kernel" in B.last_kernel()
        goti = B.binary_conv2d_packed(xp, C, Wp, O, k, k, 1, k // 2, integer_out=True)
        for n in range(0, N, 7):
            one = xp[n:n + 1].contiguous()
            assert torch.equal(goti[n:n + 1], B.binary_conv2d_packed(one, C, Wp, O, k, k, 1, k // 2, integer_out=True))
    at = np.array([0, N // 2, N - 1])
    ri, rf = oracle.binary_conv2d(x[at], w, 1, k // 2, alpha)
    np.testing.assert_array_equal(goti[at].cpu().numpy(), ri)
    assert_f32_close(got[at].cpu().numpy(), rf)
    assert torch.equal(got, dev(alpha)[None, :, None, None] * goti.float())


@pytest.mark.parametrize("N,H,W,O,nt", [(64, 14, 14, 256, True), (120, 14, 14, 256, False), (110, 7, 7, 256, True),
                                        (230, 7, 7, 256, False), (200, 5, 6, 64, False), (85, 16, 16, 256, True)])
def test_popcount_conv_streams_small_results_and_whole_lines(N, H, W, O, nt):
    """1 x 1 over 256 channels: the hint of the result stores by plane and size, and the results it leaves."""
    rng = np.random.default_rng(N + H)
    x = rng.standard_normal((N, 256, H, W)).astype(np.float32)
    w = rng.standard_normal((O, 256, 1, 1)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    with tuned(k5=1):
        got = run_conv(x, w, 1, 0, alpha=alpha)
        kernel = B.last_kernel()
        goti = run_conv(x, w, 1, 0, integer_out=True)
    assert "conv_stationary_kernel" in kernel and (",nt>" in kernel) == nt, kernel
    at = np.r_[0:3, N - 3:N]
    ri, rf = oracle.binary_conv2d(x[at], w, 1, 0, alpha)
    np.testing.assert_array_equal(goti[at], ri)
    assert_f32_close(got[at], rf)
    np.testing.assert_array_equal(got, (alpha[None, :, None, None] * goti.astype(np.float32)).astype(np.float32))


def test_conv_padding_closed_form_on_gpu():
    C, H, W, O = 5, 6, 6, 2
    K = 9 * C
    wp = np.ones((O, C, 3, 3), dtype=np.float32)
    assert (run_conv(np.ones((1, C, H, W), dtype=np.float32), wp, 1, 1, integer_out=True) == K).all()
    x = -np.ones((1, C, H, W), dtype=np.float32)
    np.testing.assert_array_equal(run_conv(x, wp, 1, 1, integer_out=True),
                                  oracle.binary_conv2d(x, wp, 1, 1)[0])


def test_config2_conv_full():
    c = synth.config2()
    alpha = oracle.alpha_mean_abs(c["w"])
    assert_f32_close(B.alpha_mean_abs(dev(c["w"])).cpu().numpy(), alpha)
    ri, rf = oracle.binary_conv2d(c["x"], c["w"], 1, 1, alpha)
    # automatic (the short-K FP4 matrix-core kernel with its filters in LDS; k5=5 names it),
    # register-stationary xor/popcount kernel, xor/popcount GEMM kernel, GEMM-shaped FP4 and
    # int8 matrix-core kernels
    for choice in (dict(), dict(k5=1), dict(k5=5), dict(k5=2), dict(k5=4), dict(k5=4, k7=2)):
        with tuned(**choice):
            got = run_conv(c["x"], c["w"], 1, 1, alpha=alpha)
            assert got.shape == (16, 64, 56, 56)
            assert_f32_close(got, rf)
            np.testing.assert_array_equal(run_conv(c["x"], c["w"], 1, 1, integer_out=True), ri)


@pytest.mark.parametrize("stride", [1, 2])
def test_config4_conv_full(stride):
    c = synth.config4(stride=stride)
    frac_pos = (c["x"] >= 0).mean()
    assert 0.60 < frac_pos < 0.635                     # skewed sign balance, P(|z| >= 0.5) = 0.617
    alpha = oracle.alpha_mean_abs(c["w"])
    ri, rf = oracle.binary_conv2d(c["x"], c["w"], stride, 1, alpha)
    # automatic (the short-K FP4 matrix-core kernel, 36 words of K), register-stationary
    # xor/popcount kernel, xor/popcount GEMM kernel, GEMM-shaped FP4 and int8 matrix-core kernels,
    # the 64 x 64 per wave FP4 kernel's convolution form
    for choice in (dict(), dict(k14=1), dict(k14=2), dict(k14=3), dict(k5=1), dict(k5=2), dict(k5=4), dict(k5=4, k7=2), dict(k5=6)):
        with tuned(**choice):
            got = run_conv(c["x"], c["w"], stride, 1, alpha=alpha)
            assert got.shape == (64, 256, 14 // stride, 14 // stride)
            assert_f32_close(got, rf)
            np.testing.assert_array_equal(run_conv(c["x"], c["w"], stride, 1, integer_out=True), ri)


# ------------------------------------------------------------------ alpha helper
@pytest.mark.parametrize("rows,cols", [(1, 1), (3, 7), (64, 576), (5, 9216)])
def test_alpha_mean_abs(rows, cols):
    rng = np.random.default_rng(rows + cols)
    w = rng.uniform(-1, 1, (rows, cols)).astype(np.float32)
    assert_f32_close(B.alpha_mean_abs(dev(w)).cpu().numpy(), oracle.alpha_mean_abs(w))


@pytest.mark.parametrize("rows,cols", [(5, 3), (1023, 2305), (1024, 4096), (7, 2303), (3, 9217), (2, 25086), (1230, 10243), (3100, 4095)])
def test_alpha_and_row_pack_any_start(rows, cols):
    """Rows that start on any dword, with a wave and with four per row, one trip and several, the sizes on both sides of what is
    read with the streaming hint (50 MB).  alpha against the mean in 64 bits: its own sum is one, so half an ulp of float is left."""
    w = torch.rand(rows * cols + 1, device="cuda")[1:].sub_(0.5).view(rows, cols)
    host = w.cpu().numpy()
    np.testing.assert_allclose(B.alpha_mean_abs(w).cpu().numpy(), np.abs(host.astype(np.float64)).mean(axis=1), rtol=2.0 ** -24 * 1.01, atol=0)
    np.testing.assert_array_equal(host_u64(B.binarize_pack(w, 1)), oracle.binarize_pack(host, 1))


def test_pack_more_rows_than_a_launch_counts():
    """2^30 + 70 rows of one value: two launches, the second from its own row on."""
    rows = (1 << 30) + 70
    x = torch.full((rows, 1), -1.0, device="cuda")
    at = torch.tensor([0, 5, (1 << 30) - 1, 1 << 30, (1 << 30) + 1, rows - 1], device="cuda")
    x[at] = 1.0
    out = B.binarize_pack(x, 1)
    assert out.shape == (rows, 1) and int(out.sum()) == len(at) and bool((out[at] == 1).all())


@pytest.mark.parametrize("K,cols,start", [(1, 1, 0), (15, 64, 0), (16, 65, 0), (17, 96, 1), (64, 63, 0), (65, 130, 3), (128, 1024, 0), (129, 1024, 1),
                                          (191, 320, 0), (1000, 515, 2), (3150, 4096, 0), (3150, 4100, 0)])
def test_pack_down_columns_tiles(K, cols, start):
    """Pack down the columns: rests of rows, words and columns, rows of whole 128-byte lines (below and above the size of the
    streaming hint) and tiles dealt out per XCD."""
    x = torch.rand(K * cols + start, device="cuda")[start:].sub_(0.5).view(K, cols)
    np.testing.assert_array_equal(host_u64(B.binarize_pack(x, 0)), oracle.binarize_pack(x.cpu().numpy(), 0))


@pytest.mark.parametrize("O,C,k", [(1, 1, 5), (3, 64, 5), (2, 65, 5), (5, 128, 5), (2, 129, 5), (70, 321, 5), (1, 1, 7), (3, 64, 7), (2, 65, 7), (9, 191, 7), (70, 449, 7)])
def test_conv_weight_pack_many_taps(O, C, k):
    """25 and 49 taps: channels around whole words, filters that start on any dword, one workgroup per filter (25, 49 and 50
    words, with their constant) and one per 64 channels."""
    w = torch.rand(O * C * k * k + 1, device="cuda")[1:].sub_(0.5).view(O, C, k, k)
    host = w.cpu().numpy()
    Wp, kwords = host_u64(B.pack_conv_weights(w)), k * k * ((C + 63) // 64)
    ref = oracle.binarize_pack(np.transpose(host, (0, 2, 3, 1)).reshape(O * k * k, C), 1).reshape(O, kwords)
    np.testing.assert_array_equal(Wp[:, :kwords], ref)
    short = kwords in (25, 49, 50)
    ldb = Wp.shape[1] - (2 if short else 0)
    assert (Wp[:, kwords:ldb] == 0).all()
    if short:
        ones = np.unpackbits(ref.view(np.uint8), axis=1).sum(axis=1, dtype=np.int64)
        consts = Wp[:, ldb:].copy().view(np.float32)
        np.testing.assert_array_equal(consts[:, 0], (C * k * k - 2 * ones).astype(np.float32))
        assert (consts[:, 1:] == 0).all()


# ------------------------------------------------------------------ k-bit GEMM
@pytest.mark.parametrize("bits", [1, 2, 3, 4, 8])
def test_quant_gemm_small(bits):
    rng = np.random.default_rng(bits)
    M, N, K = 37, 70, 333
    a = rng.uniform(0, 1, (M, K)).astype(np.float32)
    a[0, :6] = [1 / 6, 5 / 6, 0.5, 0.0, 1.0, 0.25]      # tie inputs of the quantiser
    a[1, :4] = [-0.5, 1.5, -0.0, 2.0]                   # clamped
    w = rng.standard_normal((N, K)).astype(np.float32)
    S, of = B.quant_gemm(dev(a), dev(w), bits)
    rS, r64, r32 = oracle.quant_gemm(a, w, bits)
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    assert_f32_close(of.cpu().numpy(), r64, atol=1e-9)
    assert_f32_close(of.cpu().numpy(), r32)


@pytest.mark.parametrize("bits", [1, 2])
@pytest.mark.parametrize("M,N,K", [(5, 3, 64), (7, 70, 1000), (6, 9, 1025), (3, 66, 2049), (9, 5, 5000), (2, 33, 16383), (3, 40, 17500)])
def test_quant_planes_by_thresholds(M, N, K, bits):
    """One- and two-bit activations as bit planes: floats on both sides of every level's threshold, rows of one to more
    than sixteen segments of 1024 values, whole and not, several of a workgroup's rows past the last."""
    rng = np.random.default_rng(K + bits)
    L = (1 << bits) - 1
    at = np.array([(i - 0.5) / L for i in range(1, L + 1)] + [0.0, 1.0], np.float32)
    near = np.concatenate([at] + [np.nextafter(at, s * np.float32(np.inf), dtype=np.float32) for s in (-1, 1)]
                          + [np.array([-0.0, -1e30, 1e30, np.inf, -np.inf], np.float32)])
    a = rng.uniform(-0.1, 1.1, (M, K)).astype(np.float32)
    pick = rng.random((M, K)) < 0.5
    a[pick] = rng.choice(near, int(pick.sum()))
    w = rng.standard_normal((N, K)).astype(np.float32)
    with tuned(k7=1):
        S, of = B.quant_gemm(dev(a), dev(w), bits)
    rS, r64, r32 = oracle.quant_gemm(a, w, bits)
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    assert_f32_close(of.cpu().numpy(), r32)


@pytest.mark.parametrize("M,N,K", [(513, 290, 1100), (513, 290, 1101), (994, 551, 1200), (700, 1300, 5000), (520, 513, 5003)])
def test_quant_bytes_forms(M, N, K):
    """The byte form's three sizes of C per wave and its splits of K: both sides of the lines that choose them."""
    rng = np.random.default_rng(M + N + K)
    a = rng.uniform(0, 1, (M, K)).astype(np.float32)
    w = np.tanh(rng.standard_normal((N, K))).astype(np.float32)
    S, of = B.quant_gemm(dev(a), dev(w), 4, bits_w=4)
    assert "gemm_i8_kernel" in B.last_kernel()
    rS, r64, r32 = oracle.quant_gemm(a, w, 4, 4)
    np.testing.assert_array_equal(S.cpu().numpy(), rS)


@pytest.mark.parametrize("engine", [0, 1])
@pytest.mark.parametrize("ba,bw", [(1, 2), (2, 2), (2, 3), (3, 2), (4, 4), (8, 8), (2, 8)])
def test_quant_gemm_kbit_weights(ba, bw, engine):
    """k-bit weights: w in [-1, 1] through the affine pair around Eq. 1.  Integer S exact, the
    float within 1e-6; tie and clamp inputs on both operands, ragged shapes, the matrix-core and
    the xor/popcount engine."""
    rng = np.random.default_rng(10 * ba + bw)
    M, N, K = 37, 45, 333
    a = rng.uniform(0, 1, (M, K)).astype(np.float32)
    a[0, :6] = [1 / 6, 5 / 6, 0.5, 0.0, 1.0, 0.25]
    w = rng.uniform(-1, 1, (N, K)).astype(np.float32)
    w[0, :8] = [0.0, -0.0, 1.0, -1.0, 1.5, -2.0, 1 / 3, -1 / 3]      # ties of u = 1/2, clamps
    rS, r64, r32 = oracle.quant_gemm(a, w, ba, bw)
    with tuned(k7=engine):
        S, of = B.quant_gemm(dev(a), dev(w), ba, bits_w=bw)
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    assert_f32_close(of.cpu().numpy(), r32)
    assert_f32_close(of.cpu().numpy(), r64, atol=1e-9)


@pytest.mark.parametrize("M,N,K", [(16, 16, 1), (32, 32, 256), (33, 65, 257), (31, 300, 2305), (512, 520, 770), (700, 2100, 100)])
@pytest.mark.parametrize("ba,bw", [(3, 1), (8, 1), (1, 2), (4, 4), (7, 7), (8, 3), (2, 8), (8, 8)])
def test_quant_gemm_bytes(M, N, K, ba, bw):
    """The int8 form: edges of its 32-row blocks and 256-wide k blocks, both tile sizes, with and
    without a K split, operands whose rows do not start 16-byte aligned, one output or both."""
    rng = np.random.default_rng(M + N + K + 10 * ba + bw)
    a = rng.uniform(-0.1, 1.1, (M, K + 1)).astype(np.float32)
    w = rng.uniform(-1.1, 1.1, (N, K + 3)).astype(np.float32)
    da, dw = dev(a)[:, :K], dev(w)[:, 3:] if bw > 1 else dev(w)[:, :K]
    a, w = a[:, :K].copy(), w[:, 3:].copy() if bw > 1 else w[:, :K].copy()
    rS, _, r32 = oracle.quant_gemm(a, w, ba, bw)
    with tuned(k7=3):
        S, of = B.quant_gemm(da, dw, ba, bits_w=bw)
        assert "gemm_i8_kernel" in B.last_kernel()
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    np.testing.assert_array_equal(of.cpu().numpy(), r32)  # (the division, to the last bit)
    S2, none = B.quant_gemm(dev(a), dev(w), ba, bits_w=bw, want_float=False)
    assert none is None
    np.testing.assert_array_equal(S2.cpu().numpy(), rS)


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (1, 1, 4), (16, 16, 31), (33, 70, 257), (64, 32, 320), (300, 200, 65), (600, 700, 40), (40, 30, 893), (5, 9, 7)])
@pytest.mark.parametrize("ba,bw", [(1, 1), (2, 1), (3, 1), (8, 1), (1, 2), (4, 4), (8, 7), (7, 8), (8, 8)])
def test_quant_gemm_one_launch(M, N, K, ba, bw):
    """The one-launch form, every pair of bit widths: K tails inside a lane's four values and inside
    a step, one and many waves per tile, rows and columns that do not fill a tile, operand rows further
    apart than their length and not 16-byte aligned, a caller's workspace or none."""
    rng = np.random.default_rng(M + N + K + 10 * ba + bw)
    a = rng.uniform(-0.1, 1.1, (M, K + 1)).astype(np.float32)
    w = rng.uniform(-1.1, 1.1, (N, K + 3)).astype(np.float32)
    rS, _, r32 = oracle.quant_gemm(a[:, :K].copy(), w[:, :K].copy(), ba, bw)
    S, of = B.quant_gemm(dev(a)[:, :K], dev(w)[:, :K], ba, bits_w=bw)
    assert ("quant_small_kernel" in B.last_kernel()) == (K >= 4)
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    assert_f32_close(of.cpu().numpy(), r32)
    ws = torch.empty(B.workspace_bytes(B.OP_QUANT_GEMM, (M, N, K, ba, bw)), dtype=torch.uint8, device="cuda")
    none, of = B.quant_gemm(dev(a)[:, :K], dev(w)[:, :K], ba, bits_w=bw, want_int=False, workspace=ws)
    assert none is None
    assert_f32_close(of.cpu().numpy(), r32)


@pytest.mark.parametrize("M,N,K", [(513, 580, 769), (545, 513, 1023), (33, 1100, 2817), (520, 300, 1025), (40, 3000, 1300), (70, 36, 4200), (16, 33, 3583), (200, 2100, 897)])
@pytest.mark.parametrize("ba,bw", [(1, 1), (2, 1), (4, 1), (3, 2), (1, 3), (4, 4)])
def test_quant_halves(M, N, K, ba, bw):
    """Two values a byte: K that ends in either half of a block of 256 and on its edge, rows that do not fill a block of 32, one
    and two blocks a wave, K split up to eight ways; ties, clamped values, NaN and infinities; operand rows apart."""
    rng = np.random.default_rng(M + N + K + 10 * ba + bw)
    a = rng.uniform(-0.1, 1.1, (M, K + 1)).astype(np.float32)
    w = rng.uniform(-1.1, 1.1, (N, K + 3)).astype(np.float32)
    a[rng.random(a.shape) < 0.01] = np.nan
    a[rng.random(a.shape) < 0.05] = 0.5
    a[rng.random(a.shape) < 0.01] = np.inf
    w[rng.random(w.shape) < 0.01] = -np.inf
    w[rng.random(w.shape) < 0.05] = -0.0
    # (NaN is level 0, which the oracle's conversion of it to a whole number does not define)
    rS, _, r32 = oracle.quant_gemm(np.where(np.isnan(a), np.float32(0), a)[:, :K].copy(), w[:, 3:].copy(), ba, bw)
    S, of = B.quant_gemm(dev(a)[:, :K], dev(w)[:, 3:], ba, bits_w=bw)
    assert "gemm_i8_kernel" in B.last_kernel() and "halves" in B.last_kernel(), B.last_kernel()
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    np.testing.assert_array_equal(of.cpu().numpy(), r32)  # (the division, to the last bit)


@pytest.mark.parametrize("M,N,K,form", [(16, 16, 1, "16 x 16"), (33, 47, 255, "16 x 16"), (31, 17, 257, "16 x 16"), (90, 70, 769, "16 x 16"),
                                        (16, 6144, 2049, "16 x 16"), (256, 384, 513, "16 x 16"), (17, 3073, 300, "1,1"), (176, 560, 600, "1,1")])
@pytest.mark.parametrize("ba,bw", [(1, 1), (4, 3), (2, 5), (7, 2), (8, 4), (3, 8), (8, 8)])
def test_quant_bytes_16_by_16(M, N, K, form, ba, bw):
    """Bytes of few tiles: 16 x 16 of the result a workgroup and the line to larger ones (384 and 385 of them); one step for a wave, one
    for some, several, a last one of padding; either half of the operands' blocks of 32 rows, part of one; operand rows apart."""
    rng = np.random.default_rng(M + N + K + 10 * ba + bw)
    a = rng.uniform(-0.1, 1.1, (M, K + 1)).astype(np.float32)
    w = rng.uniform(-1.1, 1.1, (N, K + 3)).astype(np.float32)
    rS, _, r32 = oracle.quant_gemm(a[:, :K].copy(), w[:, 3:].copy(), ba, bw)
    with tuned(k7=3 if ba > 2 or bw > 1 else 0):  # (the pair of launches; of few bits the engine pins the planes)
        S, of = B.quant_gemm(dev(a)[:, :K], dev(w)[:, 3:], ba, bits_w=bw)
        if ba > 2 or bw > 1:
            assert "gemm_i8_kernel<%s" % form in B.last_kernel(), B.last_kernel()
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    np.testing.assert_array_equal(of.cpu().numpy(), r32)  # (the division, to the last bit)


@pytest.mark.parametrize("M,N,K,form,bands", [(300, 40, 2200, "16 x 16", 8), (250, 70, 2500, "16 x 16", 4), (136, 40, 5300, "16 x 16", 4), (700, 150, 1000, "1,1", 8),
                                              (610, 330, 1100, "1,1", 4), (440, 640, 2800, "1,2", 2), (1500, 140, 1300, "1,2", 8),
                                              (256, 384, 513, "16 x 16", 1), (176, 560, 600, "1,1", 1), (700, 700, 5200, "1,2", 2)])
@pytest.mark.parametrize("ba,bw", [(4, 3), (8, 2)])
def test_quant_bytes_bands(M, N, K, form, bands, ba, bw):
    """The order of the tiles of a product of bytes in one band, two, four and eight, rows that do not come out even among them."""
    rng = np.random.default_rng(M + N + K + 10 * ba + bw)
    a, w = rng.uniform(-0.1, 1.1, (M, K)).astype(np.float32), rng.uniform(-1.1, 1.1, (N, K)).astype(np.float32)
    rS, _, r32 = oracle.quant_gemm(a, w, ba, bw)
    with tuned(k7=3):  # (the pair of launches)
        S, of = B.quant_gemm(dev(a), dev(w), ba, bits_w=bw)
        assert "gemm_i8_kernel<%s" % form in B.last_kernel() and B.last_kernel().endswith("bands %d" % bands), B.last_kernel()
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    np.testing.assert_array_equal(of.cpu().numpy(), r32)


@pytest.mark.parametrize("M,N,K,T", [(16, 16, 4, 16), (1, 1, 63, 16), (17, 31, 64, 16), (15, 33, 65, 16), (256, 256, 129, 16), (256, 257, 512, 16),
                                     (256, 257, 513, 32), (512, 1024, 128, 16), (512, 1025, 128, 32), (30, 50, 2816, 16), (16, 33, 3071, 16), (300, 240, 700, 32), (300, 240, 896, 32), (730, 1439, 31, 32)])
@pytest.mark.parametrize("ba,bw", [(1, 1), (8, 1), (2, 2), (4, 7), (8, 3), (1, 8), (8, 8)])
def test_quant_one_launch_tiles(M, N, K, T, ba, bw):
    """The one-launch form in tiles of 16 x 16 and 32 x 32, both sides of the lines between them, K around a step."""
    rng = np.random.default_rng(M + N + K + 10 * ba + bw)
    a = rng.uniform(-0.1, 1.1, (M, K)).astype(np.float32)
    w = rng.uniform(-1.1, 1.1, (N, K)).astype(np.float32)
    rS, _, r32 = oracle.quant_gemm(a, w, ba, bw)
    S, of = B.quant_gemm(dev(a), dev(w), ba, bits_w=bw)
    assert "quant_small_kernel" in B.last_kernel() and "<%d>" % T in B.last_kernel(), B.last_kernel()
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    np.testing.assert_array_equal(of.cpu().numpy(), r32)


@pytest.mark.parametrize("M,N,K,ba,bw,call,graph", [
    (119, 448, 1231, 1, 1, True, True), (119, 448, 1280, 1, 1, True, True), (119, 448, 1281, 1, 1, True, False), (119, 448, 1856, 1, 1, True, False),
    (119, 448, 1857, 1, 1, False, False), (119, 448, 2072, 1, 1, False, False), (119, 448, 2304, 1, 1, False, False), (119, 448, 2305, 1, 1, False, False),
    (119, 448, 1344, 8, 1, True, True), (119, 448, 1345, 8, 1, True, True), (119, 448, 1408, 8, 1, True, True), (119, 448, 1409, 8, 1, True, False),
    (119, 448, 1779, 8, 1, True, False), (119, 448, 1780, 8, 1, False, False), (119, 448, 1846, 8, 1, False, False), (119, 448, 2432, 8, 1, False, False),
    (119, 448, 2815, 8, 1, False, False), (119, 448, 2816, 8, 1, False, False),
    (30, 40, 2112, 4, 4, True, True), (30, 40, 2240, 4, 4, True, True), (30, 40, 2241, 4, 4, True, False), (30, 40, 2816, 4, 4, True, False),
    (30, 40, 3264, 4, 4, True, False), (30, 40, 3456, 4, 4, True, False), (30, 40, 3457, 4, 4, False, False), (30, 40, 2815, 4, 8, True, False),
    (90, 60, 2048, 2, 2, True, True), (90, 60, 2176, 2, 2, True, True), (90, 60, 2177, 2, 2, True, False), (90, 60, 2688, 2, 2, True, False),
    (90, 60, 2689, 2, 2, True, False), (90, 60, 3200, 2, 2, True, False), (90, 60, 3201, 2, 2, False, False),
    (241, 256, 1118, 2, 1, True, True), (241, 256, 1119, 2, 1, True, True), (241, 256, 1152, 2, 1, True, True), (241, 256, 1153, 2, 1, True, False),
    (241, 256, 1536, 2, 1, True, False), (241, 256, 1537, 2, 1, True, False), (241, 256, 1728, 2, 1, True, False), (241, 256, 1729, 2, 1, False, False),
    (1835, 24, 2158, 2, 8, True, True), (139, 256, 2432, 8, 1, False, False), (27, 21, 3264, 1, 2, True, False), (407, 125, 1792, 8, 1, True, False),
    (40, 64, 3072, 8, 8, True, False), (40, 64, 3073, 8, 8, False, False), (16, 2048, 8192, 8, 8, True, True), (16, 2048, 8193, 8, 8, False, False),
    (15, 17, 2816, 4, 4, True, True), (15, 17, 2817, 4, 4, False, False), (287, 256, 704, 2, 1, True, True),
    (287, 256, 705, 2, 1, True, False), (287, 256, 896, 2, 1, True, True), (287, 256, 928, 2, 1, True, False), (500, 512, 704, 8, 2, True, True),
    (500, 512, 736, 8, 2, True, False), (500, 512, 576, 8, 2, True, True), (500, 512, 575, 8, 2, True, True), (500, 512, 577, 8, 2, True, False),
    (600, 512, 288, 3, 3, True, True), (600, 512, 289, 3, 3, True, False), (1125, 1216, 128, 8, 1, True, True), (1125, 1216, 129, 8, 1, False, False)])
def test_quant_one_launch_or_two(M, N, K, ba, bw, call, graph):
    """The lines between one launch and two, for calls and for calls that are being captured, K up to where the choice ends; replays
    between calls give what the calls give."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K)
    a = torch.rand((M, K), device="cuda", generator=g)
    w = torch.rand((N, K), device="cuda", generator=g) * 2 - 1
    run = lambda: B.quant_gemm(a, w, ba, bits_w=bw)  # noqa: E731
    run()
    assert ("quant_small" in B.last_kernel()) == call, B.last_kernel()
    torch.cuda.synchronize()
    captured = torch.cuda.CUDAGraph()
    with torch.cuda.graph(captured):
        S, f = run()
        assert ("quant_small" in B.last_kernel()) == graph, B.last_kernel()
    for _ in range(3):
        a.uniform_(generator=g)
        captured.replay()
        S2, f2 = run()
        assert ("quant_small" in B.last_kernel()) == call, B.last_kernel()
        assert torch.equal(S, S2) and torch.equal(f, f2)
    rS, _, r32 = oracle.quant_gemm(a.cpu().numpy(), w.cpu().numpy(), ba, bw)
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    np.testing.assert_array_equal(f.cpu().numpy(), r32)


@pytest.mark.parametrize("M,N,K,words", [(700, 700, 2000, 32), (520, 520, 1300, 32)])  # words: of a row of planes
def test_quant_few_bits_workspace(M, N, K, words):
    """Few bits: with the workspace that the query names, two values a byte, in it and not beside it; with what the plane
    kernels need, the plane kernels; with less, refused."""
    rng = np.random.default_rng(9)
    a, w = rng.uniform(0, 1, (M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    rS, _, _ = oracle.quant_gemm(a, w, 1, 1)
    full = B.workspace_bytes(B.OP_QUANT_GEMM, (M, N, K, 1, 1))
    up = lambda n, to: (n + to - 1) // to * to
    planes = up(M * words * 8, 256) + up(N * up(up(K, 64) // 64, 2) * 8, 256) + up(M * 4, 256)
    assert planes < full == (up(M, 32) + up(N, 32)) * up(K, 256) // 2
    for size, kernel in ((full, "gemm_i8_kernel"), (full - 256, "gemm_fp4_kernel"), (planes, "gemm_fp4_kernel")):
        room = torch.full((4 * full,), 0xa5, dtype=torch.uint8, device="cuda")
        S, _ = B.quant_gemm(dev(a), dev(w), 1, want_float=False, workspace=room[full:full + size])
        assert kernel in B.last_kernel(), (size, B.last_kernel())
        np.testing.assert_array_equal(S.cpu().numpy(), rS)
        assert bool((room[:full] == 0xa5).all()) and bool((room[full + size:] == 0xa5).all())  # nothing beside it is written
    with pytest.raises(B.BmxError) as e:
        B.quant_gemm(dev(a), dev(w), 1, want_float=False, workspace=torch.empty(planes - 256, dtype=torch.uint8, device="cuda"))
    assert e.value.status == -6


def test_config5_quant_gemm():
    c = synth.config5(small=True)
    S, of = B.quant_gemm(dev(c["a"]), dev(c["w"]), 2)
    rS, r64, r32 = oracle.quant_gemm(c["a"], c["w"], 2)
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    assert_f32_close(of.cpu().numpy(), r64, atol=1e-9)
    assert_f32_close(of.cpu().numpy(), r32)


def test_config5_quant_gemm_full_size():
    """Full 1024 x 1024 x 4096, 2-bit activations x 1-bit weights: every element of S and of the
    scaled output against the oracle, on every GEMM engine."""
    c = synth.config5()
    rS, r64, r32 = oracle.quant_gemm(c["a"], c["w"], 2)
    assert (np.abs(rS) <= 3 * 4096).all()
    for engine in GEMM_ENGINES:
        with tuned(**engine):
            S, of = B.quant_gemm(dev(c["a"]), dev(c["w"]), 2)
        np.testing.assert_array_equal(S.cpu().numpy(), rS)
        assert_f32_close(of.cpu().numpy(), r64, atol=1e-9)
        assert_f32_close(of.cpu().numpy(), r32)


def test_quant_gemm_long_k_leaves_fp4_range():
    """K * (2^bits - 1) >= 2^24: fp32 sums could round, so the launcher must take the int8 form
    (int32 accumulation); the result stays exact."""
    M, N, K = 2, 3, 5_700_000
    rng = np.random.default_rng(77)
    a = rng.uniform(0, 1, (M, K)).astype(np.float32)
    a[0] = 1.0                                  # q = 3 everywhere: the largest possible sums
    w = rng.standard_normal((N, K)).astype(np.float32)
    w[0] = 1.0
    S, of = B.quant_gemm(dev(a), dev(w), 2)
    rS, r64, r32 = oracle.quant_gemm(a, w, 2)
    assert rS[0, 0] == 3 * K and 3 * K > (1 << 24)
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    assert_f32_close(of.cpu().numpy(), r32)


# ------------------------------------------------------------------ determinism, empties
def test_repeatable_and_empty():
    c = synth.config2(small=True)
    alpha = oracle.alpha_mean_abs(c["w"])
    a = run_conv(c["x"], c["w"], 1, 1, alpha=alpha)
    b = run_conv(c["x"], c["w"], 1, 1, alpha=alpha)
    assert a.tobytes() == b.tobytes()
    e = B.binarize_pack(torch.empty((0, 64), dtype=torch.float32, device="cuda"), 1)
    assert e.shape == (0, 1)
    z = B.xnor_gemm(torch.empty((0, 1), dtype=torch.int64, device="cuda"),
                    torch.empty((5, 1), dtype=torch.int64, device="cuda"), 64)
    assert z.shape == (0, 5)


# ------------------------------------------------------------------ GEMM kernel shapes
@pytest.mark.parametrize("rows_per_wave", [8, 16, 32])
@pytest.mark.parametrize("ksplit", [1, 2, 3, 8])
def test_gemm_every_kernel_shape(rows_per_wave, ksplit):
    """Every (rows per wave, K split, workgroup order) the launcher can pick, forced through
    the tuning hook, on shapes with ragged rows, columns, K tails and bit planes."""
    L = B.lib()
    rng = np.random.default_rng(rows_per_wave * 10 + ksplit)
    try:
        assert L.bmx_tune_set(7, 1) == 0  # the xor/popcount engine
        for order in (0, 1):
            assert L.bmx_tune_set(2, rows_per_wave) == 0
            assert L.bmx_tune_set(3, ksplit) == 0
            assert L.bmx_tune_set(4, order) == 0
            for (M, N, K) in [(37, 70, 5000), (8, 64, 1024), (100, 129, 3072 + 64)]:
                A = oracle.binarize_pack(rng.standard_normal((M, K)).astype(np.float32), 1)
                Bm = oracle.binarize_pack(rng.standard_normal((N, K)).astype(np.float32), 1)
                got = B.xnor_gemm(dev(A.view(np.int64)), dev(Bm.view(np.int64)), K).cpu().numpy()
                np.testing.assert_array_equal(got, oracle.xnor_gemm(A, Bm, K))
            x = rng.standard_normal((19, 2500)).astype(np.float32)
            w = rng.uniform(-1, 1, (75, 2500)).astype(np.float32)
            alpha = oracle.alpha_mean_abs(w)
            ri, rf = oracle.binary_fc(x, w, alpha)
            Wp = B.binarize_pack(dev(w), 1)
            np.testing.assert_array_equal(B.binary_fc(dev(x), Wp, integer_out=True).cpu().numpy(), ri)
            assert_f32_close(B.binary_fc(dev(x), Wp, alpha=dev(alpha)).cpu().numpy(), rf)
            for bits in (1, 3):
                if rows_per_wave < bits:
                    continue
                a = rng.uniform(0, 1, (21, 2200)).astype(np.float32)
                wq = rng.standard_normal((70, 2200)).astype(np.float32)
                S, f = B.quant_gemm(dev(a), dev(wq), bits)
                rS, r64, r32 = oracle.quant_gemm(a, wq, bits)
                np.testing.assert_array_equal(S.cpu().numpy(), rS)
                assert_f32_close(f.cpu().numpy(), r32)
    finally:
        for key in (2, 3, 4, 7):
            L.bmx_tune_set(key, 0)


@pytest.mark.parametrize("engine", [2, 3])
@pytest.mark.parametrize("ksplit", [0, 1, 2, 3, 8])
def test_gemm_matrix_core_engine(ksplit, engine):
    """The matrix-core kernel (bits expanded in registers to int8, engine 2, or to FP4 nibbles,
    engine 3), forced through the tuning hook: ragged tiles in M and N, K tails inside and at
    the end of a 1024-bit step, every K split, every output kind."""
    L = B.lib()
    rng = np.random.default_rng(100 + ksplit)
    try:
        assert L.bmx_tune_set(7, engine) == 0
        assert L.bmx_tune_set(8, ksplit) == 0
        for (M, N, K) in [(37, 70, 5000), (8, 64, 1024), (100, 129, 3072 + 64), (1, 1, 1), (64, 64, 63),
                          (65, 33, 1025), (130, 200, 2048 + 128),
                          # enough tiles for the 64 x 64 per wave variant
                          (700, 801, 1100), (1031, 640, 2048 + 64)]:
            A = oracle.binarize_pack(rng.standard_normal((M, K)).astype(np.float32), 1)
            Bm = oracle.binarize_pack(rng.standard_normal((N, K)).astype(np.float32), 1)
            # rows padded to an even number of words: the kernel's 16-byte pieces need it
            ld = (A.shape[1] + 1) // 2 * 2
            Ad = np.zeros((M, ld), dtype=np.uint64); Ad[:, :A.shape[1]] = A
            Bd = np.zeros((N, ld), dtype=np.uint64); Bd[:, :A.shape[1]] = Bm
            got = B.xnor_gemm(dev(Ad.view(np.int64)), dev(Bd.view(np.int64)), K).cpu().numpy()
            np.testing.assert_array_equal(got, oracle.xnor_gemm(A, Bm, K))
        for (batch, fin, fout) in [(19, 2500, 75), (70, 4096, 130)]:
            x = rng.standard_normal((batch, fin)).astype(np.float32)
            w = rng.uniform(-1, 1, (fout, fin)).astype(np.float32)
            alpha = oracle.alpha_mean_abs(w)
            ri, rf = oracle.binary_fc(x, w, alpha)
            Wp = B.binarize_pack(dev(w), 1)
            np.testing.assert_array_equal(B.binary_fc(dev(x), Wp, integer_out=True).cpu().numpy(), ri)
            assert_f32_close(B.binary_fc(dev(x), Wp, alpha=dev(alpha)).cpu().numpy(), rf)
            assert_f32_close(B.binary_fc(dev(x), Wp).cpu().numpy(), ri.astype(np.float32))
        # k-bit activations (1 and 2 bit planes assembled into the int8 operand)
        for bits in (1, 2):
            for (M, N, K) in [(21, 70, 2200), (1, 1, 1), (33, 65, 1024), (100, 130, 4096 + 200)]:
                a = rng.uniform(0, 1, (M, K)).astype(np.float32)
                a[rng.random(a.shape) < 0.05] = 0.5  # a rounding tie of Eq. 1 for k = 2
                wq = rng.standard_normal((N, K)).astype(np.float32)
                Sg, fg = B.quant_gemm(dev(a), dev(wq), bits)
                rS, r64, r32 = oracle.quant_gemm(a, wq, bits)
                np.testing.assert_array_equal(Sg.cpu().numpy(), rS)
                assert_f32_close(fg.cpu().numpy(), r32)
    finally:
        L.bmx_tune_set(7, 0)
        L.bmx_tune_set(8, 0)


# ------------------------------------------------------------------ convolution kernel paths
BIG_K_CONV_CASES = [
    # K beyond the 36 words the register-stationary kernel holds: runs on the GEMM kernel
    # N, C, H, W, O, k, s, p
    (1, 320, 6, 7, 20, 3, 1, 1),      # 45 words, 24-dword chunks
    (2, 128, 9, 9, 33, 5, 2, 2),      # 50 words
    (1, 64, 12, 12, 5, 7, 1, 3),      # 49 words
    (2, 500, 5, 5, 70, 1, 1, 0),      # 8 words, 1x1, ragged channels
    (1, 1024, 4, 4, 17, 3, 1, 1),     # 144 words, many chunks
    (3, 200, 12, 12, 64, 5, 1, 0),    # the paper's efficiency shape (5x5, 64 filters, 8x8 out)
]


@pytest.mark.parametrize("N,C,H,W,O,k,s,p", BIG_K_CONV_CASES)
def test_conv_big_k(N, C, H, W, O, k, s, p):
    rng = np.random.default_rng(N + 10 * C + 100 * H + 1000 * O + k + s + p)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    np.testing.assert_array_equal(run_conv(x, w, s, p, integer_out=True), ri)
    assert_f32_close(run_conv(x, w, s, p, alpha=alpha), rf)


@pytest.mark.parametrize("path", [1, 2, 3, 4])
def test_conv_every_path(path):
    """The four convolution kernels (register-stationary, GEMM kernel, one-thread-per-output,
    matrix cores), each forced through the tuning hook on the shapes it accepts, with every K
    split."""
    L = B.lib()
    try:
        assert L.bmx_tune_set(5, path) == 0
        for ksplit in ((0, 2, 3) if path in (2, 4) else (0,)):
            L.bmx_tune_set(3, ksplit)
            L.bmx_tune_set(8, ksplit)
            L.bmx_tune_set(7, 2 if (path == 4 and ksplit == 2) else 0)  # int8 form once, FP4 otherwise
            for (N, C, H, W, O, k, s, p) in (CONV_CASES if path == 4 else CONV_CASES[:10]) + BIG_K_CONV_CASES[:2]:
                rng = np.random.default_rng(N + 10 * C + 100 * H + 1000 * O + k + s + p + path)
                x = rng.standard_normal((N, C, H, W)).astype(np.float32)
                w = rng.standard_normal((O, C, k, k)).astype(np.float32)
                alpha = oracle.alpha_mean_abs(w)
                ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
                np.testing.assert_array_equal(run_conv(x, w, s, p, integer_out=True), ri)
                assert_f32_close(run_conv(x, w, s, p, alpha=alpha), rf)
    finally:
        L.bmx_tune_set(5, 0)
        L.bmx_tune_set(3, 0)
        L.bmx_tune_set(8, 0)
        L.bmx_tune_set(7, 0)


WS_CONV_CASES = [
    # N, C, H, W, O, s, p   (3x3 with 9, 18, 27 or 36 words of K: the short-K matrix-core kernel)
    (1, 1, 3, 3, 1, 1, 0),
    (2, 3, 5, 5, 4, 1, 1),
    (1, 20, 8, 5, 3, 2, 1),
    (2, 64, 5, 8, 5, 1, 1),
    (3, 33, 7, 9, 70, 1, 2),
    (2, 64, 56, 56, 64, 1, 1),
    (1, 32, 57, 57, 130, 2, 0),
    (2, 128, 28, 28, 128, 2, 1),
    (3, 100, 9, 11, 33, 1, 1),
    (1, 256, 14, 14, 19, 1, 2),
    (5, 200, 9, 9, 256, 1, 1),
    (64, 256, 14, 14, 40, 2, 1),
    (2, 192, 14, 14, 70, 1, 1),
    (3, 130, 9, 11, 33, 2, 1),
    (70, 200, 14, 14, 250, 1, 1),     # 429 blocks x 8 filter tiles: a wave per block at four waves per SIMD
]


@pytest.mark.parametrize("N,C,H,W,O,s,p", WS_CONV_CASES)
def test_conv_short_k_matrix_core(N, C, H, W, O, s, p):
    """The convolution kernel that reads pre-expanded FP4 filters from LDS and streams pixel
    blocks through the matrix cores, forced through the tuning hook: ragged filter and pixel
    tiles, both filter-tile heights, several blocks per wave (a fixed count, and an uneven deal
    of the blocks over 101 waves), every output kind."""
    L = B.lib()
    rng = np.random.default_rng(N + 10 * C + 100 * H + 1000 * O + s + p)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    x[rng.random(x.shape) < 0.05] = 0.0
    w = rng.standard_normal((O, C, 3, 3)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    # (narrow = 1: pixel words fetched 8 bytes at a time also where an even number of channel
    # words lets the kernel fetch 16)
    # (narrow = 2: 16 at a time, but not in the form for channel-word counts that are multiples
    # of four, which those cases take by themselves)
    # (narrow = 3: never the form that holds one block per wave in 128 registers)
    for tile, per_wave, narrow in ((0, 0, 0), (2, 3, 0), (0, 7, 0), (0, 101, 0), (0, 0, 1), (0, 3, 1), (0, 0, 2), (0, 3, 2),
                                   (0, 0, 3)):
        with tuned(k5=5, k9=tile, k1=per_wave, k14=narrow):
            np.testing.assert_array_equal(run_conv(x, w, s, p, integer_out=True), ri)
            assert_f32_close(run_conv(x, w, s, p, alpha=alpha), rf)
            np.testing.assert_array_equal(run_conv(x, w, s, p), ri.astype(np.float32))


@pytest.mark.parametrize("N,C,H,W,O,s,p", [(1, 1, 5, 5, 1, 1, 0), (2, 64, 12, 12, 64, 1, 0), (3, 20, 9, 11, 70, 2, 2),
                                           (200, 64, 12, 12, 64, 1, 0), (2, 50, 30, 17, 33, 1, 4),
                                           (2, 100, 13, 9, 40, 1, 2), (200, 128, 12, 12, 64, 1, 0)])
def test_conv_short_k_matrix_core_5x5(N, C, H, W, O, s, p):
    """5 x 5 kernels over one or two channel words (K = 25 and 50 words, the first two points of
    the paper's Sec. 3.1 sweep) on the same kernel: an odd word count, several blocks per wave,
    every output kind."""
    rng = np.random.default_rng(N + 10 * C + 100 * H + 1000 * O + s + p)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((O, C, 5, 5)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    for per_wave, narrow in ((0, 0), (3, 0), (101, 0), (0, 1), (3, 1)):
        with tuned(k5=5, k1=per_wave, k14=narrow):
            np.testing.assert_array_equal(run_conv(x, w, s, p, integer_out=True), ri)
            assert_f32_close(run_conv(x, w, s, p, alpha=alpha), rf)
    Wp, xp = B.pack_conv_weights(dev(w)), B.pack_nchw(dev(x), p)
    img = B.binary_conv2d_bits(xp, C, Wp, O, 5, 5, s, p, alpha=dev(alpha), out_pad=2)
    np.testing.assert_array_equal(host_u64(img), packed_image(rf >= 0.0, 2))


@pytest.mark.parametrize("N,C,H,W,O,s,p", [(1, 1, 7, 7, 1, 1, 0), (2, 64, 15, 14, 70, 1, 3), (3, 3, 40, 33, 64, 2, 3)])
def test_conv_short_k_matrix_core_7x7(N, C, H, W, O, s, p):
    """7 x 7 kernels over one channel word (K = 49 words; the first layer of a ResNet has this
    shape class) on the short-K kernel, forced, several blocks per wave."""
    rng = np.random.default_rng(N + 10 * C + 100 * H + 1000 * O + s + p)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((O, C, 7, 7)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    for per_wave in (0, 2, 101):
        with tuned(k5=5, k1=per_wave):
            np.testing.assert_array_equal(run_conv(x, w, s, p, integer_out=True), ri)
            assert_f32_close(run_conv(x, w, s, p, alpha=alpha), rf)
    Wp, xp = B.pack_conv_weights(dev(w)), B.pack_nchw(dev(x), p)
    img = B.binary_conv2d_bits(xp, C, Wp, O, 7, 7, s, p, alpha=dev(alpha), out_pad=1)
    np.testing.assert_array_equal(host_u64(img), packed_image(rf >= 0.0, 1))


def test_conv_weight_rows_are_zero_padded():
    """Packed filter rows are as long as bmx_conv_weight_row_words says: the bits (zero past the
    data up to a whole register chunk), and for the K the short-K matrix-core kernel takes
    (9, 18, 25, 27, 36, 49 or 50 words) two more words holding the float K - 2 * popcount(filter)
    and zeros."""
    rng = np.random.default_rng(3)
    for (O, C, k) in [(3, 64, 3), (2, 256, 3), (2, 130, 5), (4, 1, 1), (5, 100, 3), (3, 40, 5), (3, 130, 3), (3, 70, 5), (2, 20, 7)]:
        w = rng.standard_normal((O, C, k, k)).astype(np.float32)
        Wp = host_u64(B.pack_conv_weights(dev(w)))
        kwords = k * k * ((C + 63) // 64)
        assert Wp.shape == (O, B.lib().bmx_conv_weight_row_words(C, k, k)) and Wp.shape[1] >= kwords
        ref = oracle.binarize_pack(np.transpose(w, (0, 2, 3, 1)).reshape(O * k * k, C), 1)
        ref = ref.reshape(O, kwords)
        np.testing.assert_array_equal(Wp[:, :kwords], ref)
        if kwords not in (9, 18, 25, 27, 36, 49, 50):
            assert (Wp[:, kwords:] == 0).all()
            continue
        ldb = Wp.shape[1] - 2
        assert ldb >= kwords and (Wp[:, kwords:ldb] == 0).all() and Wp.shape[1] % 2 == 0
        consts = Wp[:, ldb:].copy().view(np.float32)
        pc = np.array([[bin(int(v)).count("1") for v in row] for row in ref]).sum(axis=1)
        np.testing.assert_array_equal(consts[:, 0], (C * k * k - 2 * pc).astype(np.float32))
        assert (consts[:, 1:] == 0).all()


# ------------------------------------------------------------------ chained FC on packed bits
@pytest.mark.parametrize("small", [True, False])
def test_fc_packed_chain(small):
    """Two chained binary layers that hand packed sign bits to each other: the bits must be
    exactly what packing the first layer's fp32 output gives, and the second layer's output
    the same as through the fp32 route."""
    c = synth.config3(small=small)
    x, w1, w2 = c["x"], c["w1"], c["w2"]
    a1, a2 = oracle.alpha_mean_abs(w1), oracle.alpha_mean_abs(w2)
    r1i, r1f = oracle.binary_fc(x, w1, a1)
    r2i, r2f = oracle.binary_fc(r1f, w2, a2)
    W1p, W2p = B.binarize_pack(dev(w1), 1), B.binarize_pack(dev(w2), 1)
    Xp = B.binarize_pack(dev(x), 1)
    bits1 = B.binary_fc_packed(Xp, x.shape[1], W1p, alpha=dev(a1), mode="bits")
    np.testing.assert_array_equal(host_u64(bits1), oracle.binarize_pack(r1f, 1))
    np.testing.assert_array_equal(B.binary_fc_packed(Xp, x.shape[1], W1p, mode="i32").cpu().numpy(), r1i)
    h2 = B.binary_fc_packed(bits1, w1.shape[0], W2p, alpha=dev(a2), mode="f32")
    assert_f32_close(h2.cpu().numpy(), r2f)
    np.testing.assert_array_equal(B.binary_fc_packed(bits1, w1.shape[0], W2p, mode="i32").cpu().numpy(), r2i)


@pytest.mark.parametrize("engine", [1, 2, 3])
@pytest.mark.parametrize("batch,fin,fout", [(1, 1, 1), (5, 27, 3), (3, 180, 70), (66, 1000, 130), (9, 2100, 64),
                                            (300, 1100, 700)])
def test_fc_packed_bits_ragged(batch, fin, fout, engine):
    """Ragged shapes, poisoned output, and scales of either sign and zero: the bit is the
    IEEE compare (alpha * dot >= 0) of the fp32 product, as bmx_binarize_pack would see it.
    Every GEMM engine (xor/popcount, int8 and FP4 matrix cores), forced through the tuning hook; rows
    are padded to an even word count, which the matrix-core kernel needs to take the problem."""
    rng = np.random.default_rng(batch + fin + fout)
    x = rng.standard_normal((batch, fin)).astype(np.float32)
    w = rng.uniform(-1, 1, (fout, fin)).astype(np.float32)
    alpha = rng.standard_normal(fout).astype(np.float32)
    alpha[::3] = 0.0
    _, rf = oracle.binary_fc(x, w, alpha)

    def even_rows(a):
        p = oracle.binarize_pack(a, 1)
        out = np.zeros((p.shape[0], (p.shape[1] + 1) // 2 * 2), dtype=np.uint64)
        out[:, :p.shape[1]] = p
        return dev(out.view(np.int64))

    Xp, Wp = even_rows(x), even_rows(w)
    L = B.lib()
    try:
        assert L.bmx_tune_set(7, engine) == 0
        out = dev(np.full((batch, (fout + 63) // 64 + 1), -1, dtype=np.int64))   # one spare word
        B.binary_fc_packed(Xp, fin, Wp, alpha=dev(alpha), mode="bits", out=out)
        got = host_u64(out)
        np.testing.assert_array_equal(got[:, :-1], oracle.binarize_pack(rf, 1))
        assert (got[:, -1] == np.uint64(0xFFFFFFFFFFFFFFFF)).all()              # spare word untouched
        nob = B.binary_fc_packed(Xp, fin, Wp, mode="bits")                       # no scale: sign of dot
        ri, _ = oracle.binary_fc(x, w)
        np.testing.assert_array_equal(host_u64(nob), oracle.binarize_pack(ri.astype(np.float32), 1))
        # a folded BatchNorm threshold per feature: bit = (alpha * dot >= thr) in fp32
        thr = (rng.standard_normal(fout) * np.sqrt(fin)).astype(np.float32)
        thr[1::4] = 0.0
        tb = B.binary_fc_packed(Xp, fin, Wp, alpha=dev(alpha), mode="bits", thr=dev(thr))
        want = np.where(rf >= thr[None, :], 1.0, -1.0).astype(np.float32)
        np.testing.assert_array_equal(host_u64(tb), oracle.binarize_pack(want, 1))
    finally:
        L.bmx_tune_set(7, 0)


# ------------------------------------------------------------------ convolutions chained on packed images
def packed_image(bits_nchw, out_pad):
    """[N, O, Ho, Wo] booleans -> the packed image bmx_pack_nchw would hand the next layer:
    [N, Ho + 2*out_pad, Wo + 2*out_pad, ceil(O/64)] words, halo = every real channel set."""
    N, O, Ho, Wo = bits_nchw.shape
    rows = np.where(bits_nchw.transpose(0, 2, 3, 1).reshape(-1, O), 1.0, -1.0).astype(np.float32)
    words = oracle.binarize_pack(rows, 1)
    halo = oracle.binarize_pack(np.ones((1, O), dtype=np.float32), 1)[0]
    img = np.empty((N, Ho + 2 * out_pad, Wo + 2 * out_pad, words.shape[1]), dtype=np.uint64)
    img[:] = halo
    img[:, out_pad:out_pad + Ho, out_pad:out_pad + Wo, :] = words.reshape(N, Ho, Wo, -1)
    return img


CONV_BITS_CASES = [c + (op,) for c, op in zip(
    [(N, C, H, W, O, 3, s, p) for (N, C, H, W, O, s, p) in WS_CONV_CASES] + CONV_CASES,
    [1, 0, 2, 1, 3, 1, 0, 1, 2, 1, 1, 6, 1, 2, 1] + [1, 0, 1, 2, 1, 0, 1, 1, 3, 1, 1, 0, 2])]


@pytest.mark.parametrize("N,C,H,W,O,k,s,p,out_pad", CONV_BITS_CASES)
def test_conv_packed_bits(N, C, H, W, O, k, s, p, out_pad):
    """The convolution that hands the next one its packed image: bit o of a pixel is the fp32
    compare (alpha * dot >= thr), thr folded from a BatchNorm or absent, scales of either sign
    and zero; the halo carries the +1 of the next layer's zero padding; the image is written
    whole (poisoned beforehand).  3 x 3 kernels over up to 256 channels take the kernel that
    writes the bits itself, the rest go through the fp32 result and the channel pack."""
    rng = np.random.default_rng(7 + N + 10 * C + 100 * H + 1000 * O + k + s + p)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha = rng.standard_normal(O).astype(np.float32)
    alpha[::5] = 0.0
    thr = (rng.standard_normal(O) * np.sqrt(C * k * k)).astype(np.float32)
    thr[1::4] = 0.0
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    Ho, Wo = ri.shape[2:]
    Wp = B.pack_conv_weights(dev(w))
    xp = B.pack_nchw(dev(x), p)
    shape = (N, Ho + 2 * out_pad, Wo + 2 * out_pad, (O + 63) // 64)
    # (four channel words: also the general form of the 16-byte pixel loads)
    for narrow in ((0, 2) if k == 3 and 192 < C <= 256 else (0,)):
        for al, th, ref in ((alpha, thr, rf >= thr[None, :, None, None]),
                            (alpha, None, rf >= 0.0),
                            (None, thr, ri.astype(np.float32) >= thr[None, :, None, None]),
                            (None, None, ri >= 0)):
            out = dev(np.full(shape, -1, dtype=np.int64))
            with tuned(k14=narrow):
                B.binary_conv2d_bits(xp, C, Wp, O, k, k, s, p, alpha=None if al is None else dev(al),
                                     thr=None if th is None else dev(th), out_pad=out_pad, out=out)
            np.testing.assert_array_equal(host_u64(out), packed_image(ref, out_pad))


@pytest.mark.parametrize("N,C,H,W,O1,O2,s1", [(2, 64, 20, 20, 64, 48, 1), (3, 100, 17, 13, 130, 70, 2),
                                               (16, 64, 56, 56, 64, 64, 1)])
def test_conv_chain_on_packed_images(N, C, H, W, O1, O2, s1):
    """Two binary blocks chained without an fp32 feature map in between: the second layer reads
    the image the first wrote, and matches the oracle run on the +-1 feature map (zero padded
    before the sign, like every layer input)."""
    rng = np.random.default_rng(N + C + H + O1 + O2)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w1 = rng.standard_normal((O1, C, 3, 3)).astype(np.float32)
    w2 = rng.standard_normal((O2, O1, 3, 3)).astype(np.float32)
    a1, a2 = oracle.alpha_mean_abs(w1), oracle.alpha_mean_abs(w2)
    thr = (rng.standard_normal(O1) * 5.0).astype(np.float32)
    _, r1 = oracle.binary_conv2d(x, w1, s1, 1, a1)
    h1 = np.where(r1 >= thr[None, :, None, None], 1.0, -1.0).astype(np.float32)
    r2i, r2f = oracle.binary_conv2d(h1, w2, 1, 1, a2)
    W1p, W2p = B.pack_conv_weights(dev(w1)), B.pack_conv_weights(dev(w2))
    xp = B.pack_nchw(dev(x), 1)
    img = B.binary_conv2d_bits(xp, C, W1p, O1, 3, 3, s1, 1, alpha=dev(a1), thr=dev(thr), out_pad=1)
    np.testing.assert_array_equal(host_u64(img), packed_image(h1 > 0, 1))
    got = B.binary_conv2d_packed(img, O1, W2p, O2, 3, 3, 1, 1, alpha=dev(a2))
    assert_f32_close(got.cpu().numpy(), r2f)
    goti = B.binary_conv2d_packed(img, O1, W2p, O2, 3, 3, 1, 1, integer_out=True)
    np.testing.assert_array_equal(goti.cpu().numpy(), r2i)


# ------------------------------------------------------------------ seeded random shapes
def _random_conv_shapes(seed, count):
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < count:
        k = int(rng.choice([1, 3, 3, 3, 5, 7]))
        s = int(rng.choice([1, 2]))
        p = int(rng.integers(0, k))
        C = int(rng.choice([1, 3, 31, 64, 65, 100, 128, 200, 256, 300]))
        H, W = int(rng.integers(1, 13)), int(rng.integers(1, 13))
        if H + 2 * p < k or W + 2 * p < k:
            continue
        out.append((int(rng.integers(1, 4)), C, H, W, int(rng.choice([1, 2, 31, 32, 33, 64, 70, 130])), k, s, p))
    return out


@pytest.mark.parametrize("N,C,H,W,O,k,s,p", _random_conv_shapes(2024, 48))
def test_conv_random_shapes(N, C, H, W, O, k, s, p):
    """Seeded random layer shapes across every kernel the dispatcher can pick (1x1 to 7x7, one
    to five channel words, ragged filter and pixel counts): integer output exact, scaled output
    within tolerance, and the packed-image output equal to packing the float one."""
    rng = np.random.default_rng(N + 7 * C + 11 * H + 13 * W + 17 * O + k + s + p)
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    np.testing.assert_array_equal(run_conv(x, w, s, p, integer_out=True), ri)
    assert_f32_close(run_conv(x, w, s, p, alpha=alpha), rf)
    Wp, xp = B.pack_conv_weights(dev(w)), B.pack_nchw(dev(x), p)
    img = B.binary_conv2d_bits(xp, C, Wp, O, k, k, s, p, alpha=dev(alpha), out_pad=1)
    np.testing.assert_array_equal(host_u64(img), packed_image(rf >= 0.0, 1))


@pytest.mark.parametrize("seed", range(24))
def test_fc_random_shapes(seed):
    """Seeded random fully connected layers through the fp32 entry point (pack + GEMM) and the
    packed one, every output kind."""
    rng = np.random.default_rng(900 + seed)
    batch, fin, fout = int(rng.integers(1, 300)), int(rng.integers(1, 3000)), int(rng.integers(1, 400))
    x = rng.standard_normal((batch, fin)).astype(np.float32)
    w = rng.standard_normal((fout, fin)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(w)
    ri, rf = oracle.binary_fc(x, w, alpha)
    Wp = B.binarize_pack(dev(w), 1)
    np.testing.assert_array_equal(B.binary_fc(dev(x), Wp, integer_out=True).cpu().numpy(), ri)
    assert_f32_close(B.binary_fc(dev(x), Wp, alpha=dev(alpha)).cpu().numpy(), rf)
    Xp = B.binarize_pack(dev(x), 1)
    np.testing.assert_array_equal(B.binary_fc_packed(Xp, fin, Wp, mode="i32").cpu().numpy(), ri)
    bits = B.binary_fc_packed(Xp, fin, Wp, alpha=dev(alpha), mode="bits")
    np.testing.assert_array_equal(host_u64(bits), oracle.binarize_pack(rf, 1))


# ------------------------------------------------------------------ 32-bit BINARY_WORD rows
def words32(x, ld_dw=None, fill=0xCDCDCDCD):
    """Rows of 32-bit words straight from the definition (element k = bit k % 32 of dword k / 32,
    numpy.packbits, little bit order), ld_dw dwords apart, spare dwords poisoned."""
    bits = (x >= 0).astype(np.uint8)
    R, K = bits.shape
    Kd = (K + 31) // 32
    padded = np.zeros((R, Kd * 32), dtype=np.uint8)
    padded[:, :K] = bits
    w = np.packbits(padded, axis=1, bitorder="little").view("<u4").reshape(R, Kd)
    out = np.full((R, Kd if ld_dw is None else ld_dw), fill, dtype=np.uint32)
    out[:, :Kd] = w
    return out


@pytest.mark.parametrize("K", [1, 32, 33, 64, 96, 100, 333, 1000, 1024, 2048 + 32, 4096 + 96])
@pytest.mark.parametrize("layout", ["tight", "wide_odd", "wide_even", "offset"])
def test_words32_gemm_and_fc(K, layout):
    """Operands stored as rows of 32-bit words (Sec. 2.2.1, the 32-bit BINARY_WORD flavour): odd
    and even dword counts, odd and even strides with garbage behind the rows, and a base that is
    only 4-byte aligned.  The GEMM must equal the oracle's float layer on the unpacked signs."""
    rng = np.random.default_rng(K * 7 + len(layout))
    M, N = 37, 70
    a = rng.standard_normal((M, K)).astype(np.float32)
    b = rng.standard_normal((N, K)).astype(np.float32)
    alpha = oracle.alpha_mean_abs(b)
    ri, rf = oracle.binary_fc(a, b, alpha)
    Kd = (K + 31) // 32
    ld = {"tight": Kd, "wide_odd": Kd + 1 + (Kd & 1), "wide_even": Kd + 2 - (Kd & 1), "offset": Kd + 1}[layout]
    A32, B32 = words32(a, ld), words32(b, ld)

    def put(w):
        if layout != "offset":
            return dev(w.view(np.int32))
        flat = torch.empty(w.size + 1, dtype=torch.int32, device="cuda")   # rows start one dword in
        flat[1:] = dev(w.view(np.int32)).flatten()
        return flat[1:].view(w.shape)

    Ad, Bd = put(A32), put(B32)
    got = B.xnor_gemm_w32(Ad, Bd, K).cpu().numpy()
    np.testing.assert_array_equal(got, ri)
    # widened rows feed every call that takes packed operands
    Aw, Bw = B.widen_words32(Ad, K), B.widen_words32(Bd, K)
    np.testing.assert_array_equal(host_u64(Aw), oracle.binarize_pack(a, 1))
    np.testing.assert_array_equal(B.xnor_gemm(Aw, Bw, K).cpu().numpy(), ri)
    f = B.binary_fc_packed(Aw, K, Bw, alpha=dev(alpha), mode="f32").cpu().numpy()
    assert_f32_close(f, rf)
    bits = B.binary_fc_packed(Aw, K, Bw, alpha=dev(alpha), mode="bits")
    np.testing.assert_array_equal(host_u64(bits), oracle.binarize_pack(rf, 1))
    if Kd % 2 == 0 and layout in ("tight", "wide_even"):
        # whole 64-bit words already: the same memory read in place through the 64-bit entry point
        as64 = Ad.view(torch.int64) if layout == "tight" else None
        if as64 is not None:
            np.testing.assert_array_equal(B.xnor_gemm(as64, Bd.view(torch.int64), K).cpu().numpy(), ri)


# ------------------------------------------------------------------ 64 x 64 per wave FP4 kernel (LDS-staged operands)
def test_gemm_fp4_chip_filling_problem_exact():
    """A GEMM large enough to keep every SIMD busy with several waves for many segments
    (4096 x 4096 x 4096: 4096 tiles of 64 x 64, 8 segments each, no K split), repeated so that
    the LDS queues stay long: every element against the popcount engine (an independent kernel),
    96 sampled rows against the oracle.  A wave's staging area is overwritten by the next
    segment's loads; the kernel has to wait for its LDS reads to complete before it requests them,
    and under this load a missing wait shows as a few wrong counts."""
    rng = np.random.default_rng(4096)
    M = N = K = 4096
    A = rng.integers(0, 2 ** 63, size=(M, K // 64), dtype=np.int64) * 2 + rng.integers(0, 2, size=(M, K // 64), dtype=np.int64)
    Bm = rng.integers(0, 2 ** 63, size=(N, K // 64), dtype=np.int64) * 2 + rng.integers(0, 2, size=(N, K // 64), dtype=np.int64)
    Ad, Bd = dev(A), dev(Bm)
    with tuned(k7=1):
        ref = B.xnor_gemm(Ad, Bd, K)
        assert "gemm_kernel" in B.last_kernel()
    # the automatic choice at this size (rows staged once per workgroup, 64 x 64 per wave); the 64 x 64 per wave kernel that
    # stages its own rows, pinned by its tile order: bands that leave a rest, as many rows as C, its own choice; and shared
    # rows with 128 x 64 per wave
    for band, tall in ((0, 0), (3, 0), (1000, 0), (16, 0), (0, 2), (3, 2)):
        with tuned(k12=band, k13=tall):
            for rep in range(6):
                got = B.xnor_gemm(Ad, Bd, K)
                assert "gemm_fp4_kernel<%d,2,1" % (4 if tall else 2) in B.last_kernel() and "K split 1," in B.last_kernel()
                assert B.last_kernel().startswith("block::") == (band == 0 or tall > 0)
                assert torch.equal(got, ref), "band %d tall %d repetition %d: %d elements differ" % (
                    band, tall, rep, int((got != ref).sum()))
    rows = np.sort(rng.choice(M, size=96, replace=False))
    want = oracle.xnor_gemm(A[rows].view(np.uint64), Bm.view(np.uint64), K)
    np.testing.assert_array_equal(ref[torch.from_numpy(rows).cuda()].cpu().numpy(), want)


def test_gemm_fp4_tall_tile():
    """The kernel that stages rows once per workgroup with 128 x 64 of C per wave, 256 x 128 per workgroup (the
    automatic choice only for chip-filling products), forced on small and ragged problems by the key's older
    number, beside the other kernel's keys: fewer rows than a tile, ragged
    tiles in M and N, rows that end inside a 64-byte segment, strides wider than the rows with
    garbage behind them, int32, xnor-count and scaled fp32 results."""
    rng = np.random.default_rng(1313)
    with tuned(k7=5, k10=1, k13=2):
        for (M, N, K) in [(1, 1, 1), (37, 70, 5000), (127, 64, 1024), (128, 129, 3072 + 64), (129, 64, 63),
                          (65, 33, 1025), (130, 200, 2048 + 128), (700, 801, 1100), (256, 512, 9216),
                          (300, 190, 64 * 7), (33, 65, 64 * 9), (513, 128, 64 * 10), (5, 300, 64 * 11),
                          (70, 70, 64 * 12 + 1), (257, 64, 64 * 13), (64, 65, 64 * 14), (191, 66, 64 * 15)]:
            a = rng.standard_normal((M, K)).astype(np.float32)
            b = rng.standard_normal((N, K)).astype(np.float32)
            A, Bm = oracle.binarize_pack(a, 1), oracle.binarize_pack(b, 1)
            ld = (A.shape[1] + 1) // 2 * 2 + 2 * (K % 3)            # even, sometimes wider than the row
            Ad = np.full((M, ld), POISON, dtype=np.uint64); Ad[:, :A.shape[1]] = A
            Bd = np.full((N, ld), POISON, dtype=np.uint64); Bd[:, :A.shape[1]] = Bm
            want = oracle.xnor_gemm(A, Bm, K)
            got = B.xnor_gemm(dev(Ad.view(np.int64)), dev(Bd.view(np.int64)), K).cpu().numpy()
            assert "gemm_fp4_kernel<4,2,1" in B.last_kernel() and B.last_kernel().startswith("block::")
            np.testing.assert_array_equal(got, want)
            cnt = B.xnor_gemm(dev(Ad.view(np.int64)), dev(Bd.view(np.int64)), K, count=True).cpu().numpy()
            np.testing.assert_array_equal(2 * cnt - K, want)
        for (batch, fin, fout) in [(19, 2500, 75), (200, 4096, 130), (256, 1100, 300)]:
            x = rng.standard_normal((batch, fin)).astype(np.float32)
            w = rng.uniform(-1, 1, (fout, fin)).astype(np.float32)
            alpha = rng.standard_normal(fout).astype(np.float32)
            alpha[::3] = 0.0
            ri, rf = oracle.binary_fc(x, w, alpha)
            Wp = B.binarize_pack(dev(w), 1)
            if Wp.shape[1] % 2:                                      # 16-byte rows for the matrix-core kernels
                Wp = torch.cat([Wp, torch.zeros_like(Wp[:, :1])], dim=1).contiguous()
            np.testing.assert_array_equal(B.binary_fc(dev(x), Wp, integer_out=True).cpu().numpy(), ri)
            assert "gemm_fp4_kernel<4,2,1" in B.last_kernel() and B.last_kernel().startswith("block::")
            assert_f32_close(B.binary_fc(dev(x), Wp, alpha=dev(alpha)).cpu().numpy(), rf)
            assert "gemm_fp4_kernel<4,2,1" in B.last_kernel() and B.last_kernel().startswith("block::")


@pytest.mark.parametrize("form", [2, 3])
@pytest.mark.parametrize("M,N,K,pad", [(1, 1, 1, 0), (127, 129, 63, 0), (128, 128, 256, 1), (129, 127, 257, 0), (255, 65, 512, 2),
                                       (256, 128, 513, 0), (257, 130, 1024, 1), (300, 260, 1025, 3), (513, 200, 1536 + 200, 2),
                                       (64, 400, 3072, 0), (385, 390, 64 * 33, 1), (200, 129, 64 * 18 + 30, 4)])
def test_gemm_fp4_block_form(form, M, N, K, pad):
    """The kernel that stages operand rows once per workgroup, forced on one to a dozen workgroups: ragged tiles in M and N,
    one to five segments of K and ends inside them, rows 16-byte aligned and on any dword (64-bit and 32-bit words, an
    operand that starts between two words), garbage behind the rows; dot products, counts and scaled fp32 results."""
    rng = np.random.default_rng(1000 * M + K + form)
    A = oracle.binarize_pack(rng.standard_normal((M, K)).astype(np.float32), 1)
    Bm = oracle.binarize_pack(rng.standard_normal((N, K)).astype(np.float32), 1)
    want = oracle.xnor_gemm(A, Bm, K)
    w = A.shape[1]
    with tuned(k17=1, k19=form):
        for ld in (w + pad, (w + 1) // 2 * 2 + 2 * pad):  # as it comes; 16-byte aligned
            Ad = np.full((M, ld), POISON, dtype=np.uint64); Ad[:, :w] = A
            Bd = np.full((N, ld), POISON, dtype=np.uint64); Bd[:, :w] = Bm
            a, b = dev(Ad.view(np.int64)), dev(Bd.view(np.int64))
            np.testing.assert_array_equal(B.xnor_gemm(a, b, K).cpu().numpy(), want)
            short = K <= 96 and ld % 2  # (rows of less than 16 bytes that the next begins in)
            assert "gemm_fp4_kernel<%s" % ("4,2,1,xnor,i32,block>" if form == 2 and not short else "2,2,1,xnor,i32,block") in B.last_kernel()
            np.testing.assert_array_equal(2 * B.xnor_gemm(a, b, K, count=True).cpu().numpy() - K, want)
        dw = -(-K // 32)
        A32 = np.full(M * (dw + 1) + 1, 0xCDCDCDCD, dtype=np.uint32)
        rows = A32[1:].reshape(M, dw + 1)
        rows[:, :dw] = A.view(np.uint32)[:, :dw]
        B32 = np.ascontiguousarray(Bm.view(np.uint32)[:, :dw])
        a32 = dev(A32.view(np.int32))[1:].view(M, dw + 1)
        np.testing.assert_array_equal(B.xnor_gemm_w32(a32, dev(B32.view(np.int32)), K).cpu().numpy(), want)
        assert "xnor,i32,block of dwords>" in B.last_kernel() if K <= 96 else "xnor,i32,block>" in B.last_kernel()
        x = rng.standard_normal((M, K)).astype(np.float32)
        wt = rng.uniform(-1, 1, (N, K)).astype(np.float32)
        alpha = rng.standard_normal(N).astype(np.float32)
        _, rf = oracle.binary_fc(x, wt, alpha)
        with tuned(k15=1, k17=1, k19=form):
            for Wp in (B.binarize_pack(dev(wt), 1), torch.nn.functional.pad(B.binarize_pack(dev(wt), 1), (0, w % 2))):
                assert_f32_close(B.binary_fc(dev(x), Wp.contiguous(), alpha=dev(alpha)).cpu().numpy(), rf)
                assert "f32,block" in B.last_kernel()


@pytest.mark.parametrize("form", [2, 3])
def test_gemm_fp4_block_form_longest_k(form):
    """The block form just below its bound on K, where a sum of 13/16 K in steps of 1/4 (the sign plane's products) fills fp32: rows
    all set, all clear and mixed on both sides; dot products and counts."""
    K = (1 << 22) - 1
    rng = np.random.default_rng(form)
    def rows(n):
        r = rng.integers(0, 2 ** 64, (n, (K + 63) // 64), dtype=np.uint64)
        r[:n // 3], r[n // 3:n // 2] = ~np.uint64(0), 0
        r[n // 2:n // 2 + 4] |= r[n // 2 + 4:n // 2 + 8] | rng.integers(0, 2 ** 64, (4, r.shape[1]), dtype=np.uint64)  # (mostly set)
        r[:, -1] &= ~np.uint64(0) >> np.uint64(1)
        return r
    A, W = rows(130), rows(70)
    want = np.stack([K - 2 * np.bitwise_count(a ^ W).sum(1, dtype=np.int64) for a in A])
    a, w = dev(A.view(np.int64)), dev(W.view(np.int64))
    with tuned(k17=1, k19=form):
        np.testing.assert_array_equal(B.xnor_gemm(a, w, K).cpu().numpy(), want)
        assert "i32,block>" in B.last_kernel(), B.last_kernel()
        np.testing.assert_array_equal(B.xnor_gemm(a, w, K, count=True).cpu().numpy(), (want + K) // 2)


@pytest.mark.parametrize("M,N,K,kind,block", [
    # rows of an odd number of 32-bit words like others
    (1032, 1995, 3995, "w32", False), (2137, 971, 3163, "w32", False), (1142, 1962, 987, "w32", False),
    (1535, 1317, 3163, "w32", False), (2041, 1020, 3995, "w32", False), (64, 32000, 7003, "w32", False), (900, 1500, 29979, "w32", False),
    (129, 10300, 9003, "w32", False), (2690, 3130, 2019, "w32", True),
    # to 1280 tiles of 64 x 64 never; to 2048 from 140 dwords on, fp32 from 100, up to 512 tiles of 128 x 128; past that from 64 dwords
    # on, where rows of results are whole lines from 38
    (2048, 2048, 3499, "f32", False), (2000, 2040, 3500, "f32", False), (1900, 2500, 1664, "f32", False),
    (1900, 2500, 3584, "f32", False), (2041, 4090, 1664, "f32", False), (2690, 3130, 1664, "f32", False), (1900, 2500, 1664, "i32", False),
    (2041, 4090, 2048, "f32", False), (2053, 4090, 2048, "f32", True), (2053, 4090, 1984, "f32", False), (2053, 4064, 1280, "i32", True),
    (2053, 4064, 1152, "i32", False), (2053, 3090, 7680, "i32", True), (2041, 3070, 7680, "i32", True), (2053, 3090, 7616, "i32", True),
    (4480, 1792, 5343, "i32", True), (2041, 3070, 4480, "i32", True), (2041, 3070, 4416, "i32", False), (2041, 3070, 3200, "f32", True),
    (2041, 3070, 3136, "f32", False), (2041, 2560, 7680, "f32", False), (2041, 2590, 7680, "f32", True), (1472, 5568, 7680, "i32", False),
    (2041, 3070, 4447, "w32", False), (2041, 3070, 4449, "w32", True)])
def test_block_form_lines(M, N, K, kind, block):
    """Both sides of the lines between the kernel that stages rows once per workgroup and the 64 x 64 per wave kernel: the
    form that runs, and the same results from the other."""
    rng = np.random.default_rng(M + N + K)
    A = B.binarize_pack(dev(rng.standard_normal((M, K)).astype(np.float32)), 1)
    W = B.binarize_pack(dev(rng.standard_normal((N, K)).astype(np.float32)), 1)
    if kind == "w32":
        A, W = (t.view(torch.int32)[:, :-(-K // 32)].contiguous() for t in (A, W))
        call = lambda: B.xnor_gemm_w32(A, W, K)  # noqa: E731
    else:
        A, W = (torch.nn.functional.pad(t, (0, t.shape[1] % 2)) for t in (A, W))  # (rows 16-byte aligned)
        alpha = dev(rng.standard_normal(N).astype(np.float32)) if kind == "f32" else None
        call = lambda: B.binary_fc_packed(A, K, W, alpha=alpha, mode=kind)  # noqa: E731
    got = call()
    assert ("block" in B.last_kernel()) == block, B.last_kernel()
    assert "gemm_fp4_kernel" in B.last_kernel(), B.last_kernel()  # (as they are, not widened)
    with tuned(k19=1 if block else 3):
        want = call()
        assert ("block" in B.last_kernel()) != block, B.last_kernel()
    assert torch.equal(got, want)


@pytest.mark.parametrize("M,N,tall", [(8192, 8192, True), (8130, 8160, True), (8192, 8190, False), (8064, 8064, False)])
def test_block_form_shape_line(M, N, tall):
    """256 x 128 of C per workgroup from 4096 tiles of 128 x 128 on where C's rows are whole lines; the same results from
    128 x 128."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N)
    A, W = (torch.randint(-2 ** 62, 2 ** 62, (rows, 64), device="cuda", generator=g) for rows in (M, N))
    got = B.xnor_gemm(A, W, 4096)
    assert ("gemm_fp4_kernel<4,2,1,xnor,i32,block>" in B.last_kernel()) == tall, B.last_kernel()
    with tuned(k19=3 if tall else 2):
        want = B.xnor_gemm(A, W, 4096)
        assert ("gemm_fp4_kernel<4,2,1,xnor,i32,block>" in B.last_kernel()) != tall, B.last_kernel()
    assert torch.equal(got, want)


def test_gemm_fp4_block_form_past_4_gib_of_results():
    """33000 x 33024 int32: rows of C past 4 GiB, the last tile in part past both edges, against the 64 x 64 per wave kernel; where it is
    chosen, and pinned at a shorter K."""
    M, N = 33000, 33024
    for words, K, pin in ((11, 704, 3), (11, 700, 3), (21, 1340, 0)):
        A = torch.randint(-2 ** 62, 2 ** 62, (M, 22), device="cuda")[:, :words]
        Bm = torch.randint(-2 ** 62, 2 ** 62, (N, 22), device="cuda")[:, :words]
        with tuned(k19=pin):
            got = B.xnor_gemm(A, Bm, K)
            assert "block" in B.last_kernel(), B.last_kernel()
        with tuned(k7=1):
            want = B.xnor_gemm(A[-1000:], Bm, K)
        assert torch.equal(got[-1000:], want)
        with tuned(k19=1):
            want = B.xnor_gemm(A, Bm, K)
            assert "block" not in B.last_kernel()
        assert torch.equal(got, want)
        del got, want


@pytest.mark.parametrize("split,partials", [(0, 0), (1, 0), (2, 0), (3, 0), (5, 0), (7, 0), (8, 0), (8, 2), (3, 2)])
def test_gemm_fp4_lds_staged_kernel(split, partials):
    """The matrix-core GEMM kernel with 64 x 64 of C per wave, operands staged through LDS by the
    load unit and K split over the waves of a workgroup, forced through the tuning hook whatever
    the size: ragged tiles in M and N, rows that end inside a 64-byte segment (every residue of
    the word count mod 8), row strides wider than the rows with garbage behind them, every K
    split, partial tiles crossing LDS as fp16 pairs (where a wave's sums stay exact in them) and as
    fp32 (partials = 2 forces it), every output kind, and the plane form with 1 and 2 bit planes."""
    rng = np.random.default_rng(300 + split)
    with tuned(k7=5, k10=split, k11=partials):
        for (M, N, K) in [(1, 1, 1), (37, 70, 5000), (8, 64, 1024), (100, 129, 3072 + 64), (64, 64, 63),
                          (65, 33, 1025), (130, 200, 2048 + 128), (700, 801, 1100), (256, 512, 9216),
                          (31, 190, 64 * 7), (33, 65, 64 * 9), (64, 128, 64 * 10), (5, 300, 64 * 11),
                          (70, 70, 64 * 12 + 1), (129, 64, 64 * 13), (64, 65, 64 * 14), (66, 66, 64 * 15)]:
            a = rng.standard_normal((M, K)).astype(np.float32)
            b = rng.standard_normal((N, K)).astype(np.float32)
            A, Bm = oracle.binarize_pack(a, 1), oracle.binarize_pack(b, 1)
            ld = (A.shape[1] + 1) // 2 * 2 + 2 * (K % 3)            # even, sometimes wider than the row
            Ad = np.full((M, ld), POISON, dtype=np.uint64); Ad[:, :A.shape[1]] = A
            Bd = np.full((N, ld), POISON, dtype=np.uint64); Bd[:, :A.shape[1]] = Bm
            want = oracle.xnor_gemm(A, Bm, K)
            got = B.xnor_gemm(dev(Ad.view(np.int64)), dev(Bd.view(np.int64)), K).cpu().numpy()
            assert B.last_kernel().startswith("gemm_fp4_kernel<2,2,1,xnor")
            np.testing.assert_array_equal(got, want)
            cnt = B.xnor_gemm(dev(Ad.view(np.int64)), dev(Bd.view(np.int64)), K, count=True).cpu().numpy()
            np.testing.assert_array_equal(2 * cnt - K, want)
        for (batch, fin, fout) in [(19, 2500, 75), (70, 4096, 130), (256, 1100, 300)]:
            x = rng.standard_normal((batch, fin)).astype(np.float32)
            w = rng.uniform(-1, 1, (fout, fin)).astype(np.float32)
            alpha = rng.standard_normal(fout).astype(np.float32)
            alpha[::3] = 0.0
            ri, rf = oracle.binary_fc(x, w, alpha)
            Wp = B.binarize_pack(dev(w), 1)
            if Wp.shape[1] % 2:                                      # 16-byte rows for the matrix-core kernels
                Wp = torch.cat([Wp, torch.zeros_like(Wp[:, :1])], dim=1).contiguous()
            np.testing.assert_array_equal(B.binary_fc(dev(x), Wp, integer_out=True).cpu().numpy(), ri)
            assert "gemm_fp4_kernel" in B.last_kernel()
            assert_f32_close(B.binary_fc(dev(x), Wp, alpha=dev(alpha)).cpu().numpy(), rf)
            Xp = B.binarize_pack(dev(x), 1)
            if Xp.shape[1] % 2:
                Xp = torch.cat([Xp, torch.zeros_like(Xp[:, :1])], dim=1).contiguous()
            thr = (rng.standard_normal(fout) * np.sqrt(fin)).astype(np.float32)
            out = dev(np.full((batch, (fout + 63) // 64 + 1), -1, dtype=np.int64))
            B.binary_fc_packed(Xp, fin, Wp, alpha=dev(alpha), mode="bits", thr=dev(thr), out=out)
            assert "gemm_fp4_kernel" in B.last_kernel()
            want = np.where(rf >= thr[None, :], 1.0, -1.0).astype(np.float32)
            got = host_u64(out)
            np.testing.assert_array_equal(got[:, :-1], oracle.binarize_pack(want, 1))
            assert (got[:, -1] == np.uint64(0xFFFFFFFFFFFFFFFF)).all()
        for bits in (1, 2):
            for (M, N, K) in [(21, 70, 2200), (1, 1, 1), (33, 65, 1024), (100, 130, 4096 + 200), (256, 256, 64 * 9)]:
                a = rng.uniform(0, 1, (M, K)).astype(np.float32)
                a[rng.random(a.shape) < 0.05] = 0.5
                wq = rng.standard_normal((N, K)).astype(np.float32)
                Sg, fg = B.quant_gemm(dev(a), dev(wq), bits)
                # (the sign-packed weight rows of the workspace are ceil(K/64) words: an odd count is
                # not 16-byte aligned and goes to the xor/popcount kernel)
                assert "gemm_fp4_kernel" in B.last_kernel() or ((K + 63) // 64) % 2 == 1
                rS, r64, r32 = oracle.quant_gemm(a, wq, bits)
                np.testing.assert_array_equal(Sg.cpu().numpy(), rS)
                assert_f32_close(fg.cpu().numpy(), r32)


@pytest.mark.parametrize("split", [2, 4, 5, 8])
@pytest.mark.parametrize("K", [65535, 65536])
def test_gemm_fp4_largest_16_bit_sums(K, split):
    """Partial sums and counts that cross LDS as 16-bit whole numbers, where they are largest: rows all set, so that the full sum
    and both counts are K (65535 still fits, 65536 takes fp32 partials), all clear and mixed; a tile that reaches past C in both
    directions, with rows of C that are whole lines and that are not; the two planes of 2-bit activations, whose sums reach 3 K."""
    rng = np.random.default_rng(K + split)
    with tuned(k7=5, k10=split):
        for M, N in [(67, 96), (67, 70)]:
            a, b = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
            a[:40], b[:50] = 1.0, 1.0
            a[40:50], b[50:60] = -1.0, -1.0
            A, Bm = B.binarize_pack(dev(a), 1), B.binarize_pack(dev(b), 1)
            want = (a.clip(-1, 1) >= 0).astype(np.float64) * 2 - 1
            want = (want @ ((b >= 0).astype(np.float64) * 2 - 1).T).astype(np.int32)
            np.testing.assert_array_equal(B.xnor_gemm(A, Bm, K).cpu().numpy(), want)
            assert ("16-bit partials" in B.last_kernel()) == (K <= 65535), B.last_kernel()
            np.testing.assert_array_equal(B.xnor_gemm(A, Bm, K, count=True).cpu().numpy(), (want + K) // 2)
        k = (K + 2) // 3
        a, w = rng.uniform(0, 1, (67, k)).astype(np.float32), rng.standard_normal((70, k)).astype(np.float32)
        a[:40], w[:50] = 1.0, 1.0
        S, f = B.quant_gemm(dev(a), dev(w), 2)
        assert "planes,S" in B.last_kernel() and "K split %d" % split in B.last_kernel(), B.last_kernel()
        assert ("16-bit partials" in B.last_kernel()) == (3 * k <= 65535), B.last_kernel()
        rS, _, r32 = oracle.quant_gemm(a, w, 2)
        np.testing.assert_array_equal(S.cpu().numpy(), rS)
        np.testing.assert_array_equal(f.cpu().numpy(), rS.astype(np.float32) / np.float32(3))


@pytest.mark.parametrize("tm,tn,words,split", [(16, 16, 18, 1), (16, 16, 20, 1), (16, 16, 21, 3), (16, 16, 28, 3), (16, 17, 20, 1), (16, 17, 23, 3),
                                               (16, 32, 28, 3), (16, 32, 27, 3), (19, 27, 27, 1), (16, 16, 29, 4), (16, 16, 60, 4), (16, 16, 59, 4),
                                               (16, 16, 61, 8), (16, 32, 32, 4), (19, 27, 28, 1), (19, 27, 30, 4), (24, 32, 33, 4), (32, 33, 33, 4), (24, 32, 34, 4), (24, 33, 34, 1),
                                               (24, 33, 76, 1), (32, 32, 98, 1), (32, 33, 34, 4), (32, 40, 34, 4), (32, 41, 34, 1)])
def test_gemm_fp4_split_lines(tm, tn, words, split):
    """Both sides of the lines between the waves that share a tile's K, by the tiles and words (an odd number of words: rows that start
    on any word); a last tile of one row and one column; the same results undivided."""
    g = torch.Generator(device="cuda")
    g.manual_seed(tm * tn + words)
    A, W = (torch.randint(-2 ** 62, 2 ** 62, (64 * n - 63, words), device="cuda", generator=g) for n in (tm, tn))
    with tuned(k17=1, k19=1):
        got = B.xnor_gemm(A, W, 64 * words)
        assert "K split %d" % split in B.last_kernel(), B.last_kernel()
    with tuned(k7=5, k10=1 if split > 1 else 4):
        want = B.xnor_gemm(A, W, 64 * words)
        assert "K split %d" % split not in B.last_kernel(), B.last_kernel()
    assert torch.equal(got, want)


@pytest.mark.parametrize("M,N,words,ldc,kernel", [(2048, 2560, 64, 1 << 20, "block"), (2048, 2560, 64, 1 << 19, "gemm_fp4_kernel<2,2,1,xnor,i32> "),
                                                  (32, 32768, 6, 3 << 23, "gemm_small"), (2048, 2560, 10, 1 << 20, "block"),
                                                  (2048, 2560, 9, 1 << 20, "block"), (1472, 1472, 5, 3 << 19, "block"), (2048, 2560, 1, 1 << 20, "block"),
                                                  (1408, 1472, 5, 3 << 19, "gemm_mfma")])
def test_rows_of_c_far_apart(M, N, words, ldc, kernel):
    """Results in a matrix whose rows are further apart than gemm_fp4.hip's 32-bit indices reach: the kernels that would leave it
    such a product take it themselves, as they did."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    A, W = (torch.randint(-2 ** 62, 2 ** 62, (n, words), device="cuda", generator=g) for n in (M, N))
    room = torch.empty((M, ldc), dtype=torch.int32, device="cuda")
    B.xnor_gemm(A, W, 64 * words, out=room[:, :N])
    assert kernel in B.last_kernel(), B.last_kernel()
    with tuned(k7=1):
        want = B.xnor_gemm(A, W, 64 * words)
    assert torch.equal(room[:, :N], want)
    if kernel == "block":  # rows on any dword are not widened first
        a32, w32 = (t.view(torch.int32)[:, :2 * words - 1].contiguous() for t in (A, W))
        B.xnor_gemm_w32(a32, w32, 64 * words - 32, out=room[:, :N])
        assert kernel in B.last_kernel(), B.last_kernel()
        with tuned(k7=1):
            assert torch.equal(room[:, :N], B.xnor_gemm_w32(a32, w32, 64 * words - 32))


@pytest.mark.parametrize("words,split", [(20, 1), (22, 3), (28, 3), (29, 4), (60, 4), (61, 8)])
@pytest.mark.parametrize("bits", [1, 2])
def test_plane_gemm_split_lines(bits, words, split):
    """The same lines for bit planes, 136 tiles."""
    rng = np.random.default_rng(words + bits)
    a, w = rng.uniform(0, 1, (1030, 64 * words - 3)).astype(np.float32), rng.standard_normal((500, 64 * words - 3)).astype(np.float32)
    with tuned(k7=3):
        S, f = B.quant_gemm(dev(a), dev(w), bits)
        assert "planes,S" in B.last_kernel() and "K split %d" % split in B.last_kernel(), B.last_kernel()
    rS, _, _ = oracle.quant_gemm(a, w, bits)
    np.testing.assert_array_equal(S.cpu().numpy(), rS)
    np.testing.assert_array_equal(f.cpu().numpy(), rS.astype(np.float32) / np.float32(2 ** bits - 1))


@pytest.mark.parametrize("M,N,words,small", [(1024, 1216, 6, True), (1024, 1280, 6, True), (1024, 4032, 2, False), (1024, 1024, 28, True),
                                             (1024, 960, 30, False), (1024, 1024, 32, True), (1024, 1024, 34, False), (512, 512, 126, True),
                                             (512, 512, 130, False), (1024, 960, 32, False), (1024, 960, 31, False), (1024, 768, 46, False), (1024, 704, 47, False), (1024, 704, 53, False), (1024, 960, 39, False), (1024, 1024, 43, False),
                                             (1024, 1024, 51, False), (1024, 1920, 24, True), (1024, 1728, 30, False), (1024, 1280, 20, True), (1024, 1216, 20, True),
                                             (3200, 1024, 7, False), (3200, 1024, 9, False), (2560, 1024, 9, False), (1024, 1700, 8, True), (1024, 1760, 8, True),
                                             (1024, 960, 4, True), (1024, 1024, 4, True), (1000, 1024, 4, True), (1000, 1728, 3, True), (1000, 1792, 3, True),
                                             (1024, 1536, 6, True), (1024, 1600, 6, False), (1024, 1984, 3, True), (1024, 2048, 3, False), (1000, 1984, 7, True), (1000, 2048, 7, False), (1000, 2700, 7, True), (1000, 2800, 7, False),
                                             (1000, 3136, 3, True), (1000, 3200, 3, False), (1000, 3210, 3, True), (1024, 1984, 6, False), (1024, 2048, 6, False), (1024, 1920, 28, False)])
def test_gemm_small_lines(M, N, words, small):
    """Both sides of the lines between the kernel of 32 x 32 and those of larger tiles, rows of an even and of an odd number of words; the same results from the popcount kernel."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + words)
    A, W = (torch.randint(-2 ** 62, 2 ** 62, (n, words), device="cuda", generator=g) for n in (M, N))
    got = B.xnor_gemm(A, W, 64 * words)
    assert ("gemm_small" in B.last_kernel()) == small, B.last_kernel()
    with tuned(k7=1):
        assert torch.equal(got, B.xnor_gemm(A, W, 64 * words))


@pytest.mark.parametrize("M,N,words,small", [(1024, 1984, 6, True), (1024, 2048, 6, False), (1000, 1984, 7, True), (1000, 2048, 7, False), (1000, 2700, 7, True),
                                             (1000, 2800, 7, False), (1000, 3136, 3, True), (1000, 3200, 3, False), (1000, 3210, 3, True)])
def test_gemm_small_lines_of_fp32(M, N, words, small):
    """The same for fp32 results, scaled by a power of two per column."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + words)
    A, W = (torch.randint(-2 ** 62, 2 ** 62, (n, words), device="cuda", generator=g) for n in (M, N))
    alpha = 2.0 ** torch.randint(-3, 4, (N,), device="cuda", generator=g).float()
    got = B.binary_fc_packed(A, 64 * words, W, alpha=alpha)
    assert ("gemm_small" in B.last_kernel()) == small, B.last_kernel()
    with tuned(k7=1):
        assert torch.equal(got, B.xnor_gemm(A, W, 64 * words).float() * alpha)


@pytest.mark.parametrize("O", [5, 33, 63, 64, 70])
@pytest.mark.parametrize("C,k", [(64, 3), (100, 3), (64, 5)])
def test_conv_bits_decisions(C, k, O):
    """Packed results of the short-K convolution, decisions shifted in as carries: filters that end inside a word and inside its
    halves, thresholds that results meet exactly, infinities and NaN on either side."""
    rng = np.random.default_rng(C + 10 * k + O)
    x, w = rng.standard_normal((9, C, 13, 11)).astype(np.float32), rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha = rng.choice([0.5, -0.25, 1.0, 0.0, np.inf, np.nan], O, p=[0.4, 0.2, 0.2, 0.1, 0.05, 0.05]).astype(np.float32)
    thr = (rng.choice([0.5, -0.25, 1.0], O) * rng.integers(-20, 20, O) * 2).astype(np.float32)
    thr[::7], thr[3::7], thr[5::7] = 0.0, rng.choice([np.inf, -np.inf]), np.nan
    Wp, xp = B.pack_conv_weights(dev(w)), B.pack_nchw(dev(x), k // 2)
    with tuned(k18=1):
        got = B.binary_conv2d_bits(xp, C, Wp, O, k, k, 1, k // 2, alpha=dev(alpha), thr=dev(thr), out_pad=1)
        assert "conv_mfma_ws" in B.last_kernel(), B.last_kernel()
    f = B.binary_conv2d_packed(xp, C, Wp, O, k, k, 1, k // 2, integer_out=True).cpu().numpy().astype(np.float32)
    with np.errstate(invalid="ignore"):
        want = np.where(alpha[None, :, None, None] * f >= thr[None, :, None, None], np.float32(1), np.float32(-1))
    assert torch.equal(got, B.pack_nchw(dev(want), 1))


FP4_CONV_CASES = [
    # N, C, H, W, O, k, s, p   (an even number of channel words: 16-byte pieces never straddle two taps)
    (2, 128, 9, 9, 33, 5, 2, 2),
    (3, 100, 9, 11, 70, 3, 1, 1),
    (1, 256, 14, 14, 19, 3, 1, 2),
    (2, 500, 5, 5, 70, 1, 1, 0),
    (1, 1024, 4, 4, 17, 3, 1, 1),
    (3, 200, 12, 12, 64, 5, 1, 0),
    (2, 128, 28, 28, 128, 3, 2, 1),
    (2, 66, 9, 8, 3, 7, 1, 3),
    (5, 256, 14, 14, 256, 3, 1, 1),
    (1, 70, 1, 1, 1, 1, 1, 0),
]


@pytest.mark.parametrize("split", [0, 1, 2, 3, 8])
def test_conv_fp4_lds_staged_kernel(split):
    """The convolution form of the 64 x 64 per wave matrix-core kernel (im2col rows gathered piece
    by piece from the packed image by the load unit), forced through the tuning hook: ragged
    filter and pixel tiles, pixel tiles that straddle images, strides, halos, K that ends inside
    a 64-byte segment, every K split, both output kinds."""
    for (N, C, H, W, O, k, s, p) in FP4_CONV_CASES:
        rng = np.random.default_rng(N + 10 * C + 100 * H + 1000 * O + k + s + p + split)
        x = rng.standard_normal((N, C, H, W)).astype(np.float32)
        x[rng.random(x.shape) < 0.05] = 0.0
        w = rng.standard_normal((O, C, k, k)).astype(np.float32)
        alpha = rng.standard_normal(O).astype(np.float32)
        ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
        with tuned(k5=6, k10=split):
            got_i = run_conv(x, w, s, p, integer_out=True)
            assert "gemm_fp4_kernel" in B.last_kernel() and "conv" in B.last_kernel(), B.last_kernel()
            np.testing.assert_array_equal(got_i, ri)
            assert_f32_close(run_conv(x, w, s, p, alpha=alpha), rf)
            np.testing.assert_array_equal(run_conv(x, w, s, p), ri.astype(np.float32))


@pytest.mark.parametrize("M,N,K,off", [(512, 1024, 4096 - 64, 0), (700, 1900, 1, 0), (650, 2000, 129, 0), (520, 600, 64 * 49 - 3, 0),
                                       (1100, 1700, 64 * 7, 0), (640, 1300, 4096, 1), (333, 4001, 64 * 61, 1)])
def test_gemm_fp4_rows_through_registers(M, N, K, off):
    """(Through registers they went once.)  Operand rows of an odd number of words, or an even number behind a base that is only 8-byte
    aligned, on the 64 x 64 per wave kernel: with and without a K split, K tails inside a segment,
    output rows that are whole 128-byte lines and that are not; int32, fp32 and packed bits."""
    rng = np.random.default_rng(M + N + K)
    a, w = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    alpha, thr = rng.standard_normal(N).astype(np.float32), rng.standard_normal(N).astype(np.float32)

    def rows(m):
        words = (K + 63) // 64
        flat = torch.full((m.shape[0] * words + off,), -1, dtype=torch.int64, device="cuda")
        return B.binarize_pack(dev(m), 1, out=flat[off:].view(m.shape[0], words))

    A, W = rows(a), rows(w)
    ri, rf = oracle.binary_fc(a, w, alpha)
    with tuned(k7=5):
        np.testing.assert_array_equal(B.xnor_gemm(A, W, K).cpu().numpy(), ri)
        assert "gemm_fp4_kernel" in B.last_kernel() or K <= 96  # (rows of less than 16 bytes stay with gemm_mfma.hip)
        np.testing.assert_array_equal(B.binary_fc_packed(A, K, W, alpha=dev(alpha)).cpu().numpy(), rf)
        bits = B.binary_fc_packed(A, K, W, alpha=dev(alpha), mode="bits", thr=dev(thr))
    ref = np.where(rf >= thr[None, :], np.float32(1), np.float32(-1))
    np.testing.assert_array_equal(bits.cpu().numpy(), B.binarize_pack(dev(ref), 1).cpu().numpy())
    np.testing.assert_array_equal(B.xnor_gemm(A, W, K, count=True).cpu().numpy(), (ri + K) // 2)


@pytest.mark.parametrize("form", ["undivided", "divided", "block"])
@pytest.mark.parametrize("dwords", list(range(4, 37)) + [95, 129, 160])
def test_rows_on_any_dword_end_with_their_buffer(dwords, form):
    """Rows of every length mod 16 dwords (a last segment of one to four pieces, the last one whole or of one to three dwords), as many
    dwords apart and some more, from every dword of 16 bytes on, the last row's end the buffer's end: on the 64 x 64 per wave kernel, K
    undivided and divided, and on the one that stages rows once per workgroup.  (The results, the parts of pieces that are cleared among
    them; that nothing behind a row is read is test_row_pieces.py's.)"""
    K, M, N = 32 * dwords - dwords % 5, 70, 67
    pins = {"undivided": dict(k7=5, k10=1), "divided": dict(k7=5, k10=4), "block": dict(k17=1, k19=2 + dwords % 2)}[form]
    g = torch.Generator(device="cuda")
    g.manual_seed(dwords)
    mask = torch.full((dwords,), -1, dtype=torch.int32, device="cuda")
    if K % 32:
        mask[-1] = (1 << K % 32) - 1

    def rows(n, apart, first):
        flat = torch.randint(-2 ** 31, 2 ** 31, (first + (n - 1) * apart + dwords,), device="cuda", generator=g).to(torch.int32)
        t = flat.as_strided((n, dwords), (apart, 1), first)
        t &= mask
        return t

    def signs(t):
        return ((t[:, :, None] >> torch.arange(32, device="cuda")) & 1).reshape(t.shape[0], -1)[:, :K].float() * 2 - 1

    for first in range(4):
        A, W = rows(M, dwords + dwords % 3, first), rows(N, dwords, 3 - first)
        with tuned(**pins):
            got = B.xnor_gemm_w32(A, W, K)
            assert "gemm_fp4_kernel<" in B.last_kernel() and ("block" in B.last_kernel()) == (form == "block"), B.last_kernel()
        assert torch.equal(got, (signs(A) @ signs(W).T).to(torch.int32))


@pytest.mark.parametrize("M,N,words", [(64, 64, 1), (63, 65, 2), (1, 4096, 3), (4096, 1, 5), (130, 191, 8), (129, 64, 33), (700, 1000, 11)])
def test_gemm_fp4_bits_of_undivided_tiles(M, N, words):
    """Packed decisions of a tile that one wave finishes, a word a row: tiles that end in every direction, columns past the last without
    a bit, thresholds met exactly, infinities and NaN in scale and threshold; rows of the result further apart than their words."""
    rng = np.random.default_rng(M + N + words)
    K = 64 * words - (words > 1)
    a, w = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    alpha = rng.choice([0.5, -0.25, 1.0, 0.0, np.inf, np.nan], N, p=[0.4, 0.2, 0.2, 0.1, 0.05, 0.05]).astype(np.float32)
    thr = (rng.choice([0.5, -0.25, 1.0], N) * rng.integers(-6, 7, N)).astype(np.float32)
    thr[::7], thr[3::7], thr[5::7] = 0.0, -np.inf, np.nan
    dot = oracle.binary_fc(a, w, None)[0].astype(np.float32)
    even = words + words % 2 if words < 2 else words  # (rows of one word 16 bytes apart)
    A, W = (torch.nn.functional.pad(B.binarize_pack(dev(t), 1), (0, even - words)) for t in (a, w))
    out = dev(np.full((M, -(-N // 64) + 1), -1, dtype=np.int64))
    with tuned(k7=5, k10=1):
        B.binary_fc_packed(A, K, W, alpha=dev(alpha), mode="bits", thr=dev(thr), out=out)
        assert "gemm_fp4_kernel<2,2,1,xnor,bits>" in B.last_kernel() and "K split 1" in B.last_kernel(), B.last_kernel()
    with np.errstate(invalid="ignore"):
        want = np.where(alpha * dot >= thr, np.float32(1), np.float32(-1))
    got = host_u64(out)
    np.testing.assert_array_equal(got[:, :-1], oracle.binarize_pack(want, 1))
    assert (got[:, -1] == np.uint64(0xFFFFFFFFFFFFFFFF)).all()


@pytest.mark.parametrize("word", [32, 64])
@pytest.mark.parametrize("M,N,K,off", [(1, 1, 1, 0), (33, 31, 33, 1), (5, 70, 65, 0), (40, 33, 97, 1), (32, 64, 128, 0), (31, 65, 256, 1),
                                       (70, 130, 257, 0), (64, 100, 1000, 1), (100, 90, 2017, 1), (3, 40, 4096, 0), (2, 33, 16385, 1),
                                       (1100, 2000, 4000, 1), (400, 700, 8161, 0)])
def test_gemm_small_and_rows_on_any_dword(M, N, K, off, word):
    """The kernel for small products (1 to 16 waves per tile, rows shorter than a 16-byte piece, pieces
    past the row's end) and the 64 x 64 per wave kernel beyond its range, on rows of 64-bit and of 32-bit
    words, odd numbers of them, behind a base that is aligned to one word only."""
    rng = np.random.default_rng(M + N + K)
    a, w = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    words = -(-K // word)

    def rows(m):
        flat = torch.full((m.shape[0] * words + off,), -1, dtype=torch.int64 if word == 64 else torch.int32, device="cuda")
        full = B.binarize_pack(dev(m), 1)
        flat[off:].view(m.shape[0], words).copy_(full.view(flat.dtype)[:, :words])
        return flat[off:].view(m.shape[0], words)

    A, W = rows(a), rows(w)
    alpha, thr = rng.standard_normal(N).astype(np.float32), rng.standard_normal(N).astype(np.float32)
    ri, rf = oracle.binary_fc(a, w, alpha)
    large = M >= 1000 or K == 8161
    if word == 32:
        np.testing.assert_array_equal(B.xnor_gemm_w32(A, W, K).cpu().numpy(), ri)
        assert ("gemm_small_kernel" in B.last_kernel()) != large
        with tuned(k19=1):  # (1100 x 2000 x 4000 is past the line from which the form of shared rows is ahead)
            np.testing.assert_array_equal(B.xnor_gemm_w32(A, W, K).cpu().numpy(), ri)
            assert not large or "gemm_fp4_kernel" in B.last_kernel()
        return
    np.testing.assert_array_equal(B.xnor_gemm(A, W, K).cpu().numpy(), ri)
    assert ("gemm_small_kernel" in B.last_kernel()) != large
    np.testing.assert_array_equal(B.xnor_gemm(A, W, K, count=True).cpu().numpy(), (ri + K) // 2)
    np.testing.assert_array_equal(B.binary_fc_packed(A, K, W, alpha=dev(alpha)).cpu().numpy(), rf)
    bits = B.binary_fc_packed(A, K, W, alpha=dev(alpha), mode="bits", thr=dev(thr))
    ref = np.where(rf >= thr[None, :], np.float32(1), np.float32(-1))
    np.testing.assert_array_equal(bits.cpu().numpy(), B.binarize_pack(dev(ref), 1).cpu().numpy())


@pytest.mark.parametrize("N,C,H,W,O,k,s,p", [(6, 300, 20, 21, 80, 3, 1, 1), (30, 150, 17, 18, 130, 5, 2, 2), (12, 140, 24, 25, 70, 7, 1, 0),
                                             (40, 190, 20, 20, 64, 1, 1, 0), (3, 420, 40, 41, 200, 3, 1, 0)])
def test_conv_fp4_odd_channel_words(N, C, H, W, O, k, s, p):
    """The 64 x 64 per wave convolution where the image has an odd number of channel words (its
    16-byte pieces straddle taps and kernel rows), at sizes the dispatch sends there."""
    rng = np.random.default_rng(N + C + H + O)
    x, w = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha = rng.standard_normal(O).astype(np.float32)
    Wp = B.pack_conv_weights(dev(w))
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    with tuned(k16=1, k18=1):
        np.testing.assert_array_equal(B.binary_conv2d(dev(x), Wp, O, k, k, s, p, integer_out=True).cpu().numpy(), ri)
        assert "conv,reg" in B.last_kernel()
        np.testing.assert_array_equal(B.binary_conv2d(dev(x), Wp, O, k, k, s, p, alpha=dev(alpha)).cpu().numpy(), rf)


@pytest.mark.parametrize("M,N,K", [(256, 1001, 70), (257, 1001, 200), (320, 831, 64), (1000, 500, 65), (40, 8300, 130), (9000, 33, 64)])
def test_gemm_small_parts_of_lines(M, N, K):
    """The small product where tiles side by side share lines of the result: 256 tiles and more, eighths that do not come out even."""
    rng = np.random.default_rng(M + N + K)
    a, w = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    alpha = rng.standard_normal(N).astype(np.float32)
    ri, rf = oracle.binary_fc(a, w, alpha)
    A, W = B.binarize_pack(dev(a), 1), B.binarize_pack(dev(w), 1)
    got = B.xnor_gemm(A, W, K)
    assert "gemm_small_kernel" in B.last_kernel(), B.last_kernel()
    np.testing.assert_array_equal(got.cpu().numpy(), ri)
    np.testing.assert_array_equal(B.binary_fc_packed(A, K, W, alpha=dev(alpha)).cpu().numpy(), rf)


@pytest.mark.parametrize("M,N,K", [(3000, 2001, 64), (3001, 1990, 61), (60000, 70, 33), (70, 60000, 64), (9000, 33, 1)])
def test_bits_of_one_word_rows_of_many_tiles(M, N, K):
    """Packed decisions of rows of one word, a word apart, past the small kernel's lines for other rows: it takes them whatever the size."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    x, w = (torch.randint(0, 2, (n, K), device="cuda", generator=g).float() * 2 - 1 for n in (M, N))
    thr = torch.randint(-K, K + 1, (N,), device="cuda", generator=g).float()
    alpha = torch.rand(N, device="cuda", generator=g) - 0.25
    A, W = B.binarize_pack(x, 1), B.binarize_pack(w, 1)
    out = torch.full((M, -(-N // 64) + 1), -1, dtype=torch.int64, device="cuda")
    B.binary_fc_packed(A, K, W, alpha=alpha, mode="bits", thr=thr, out=out)
    assert "gemm_small_kernel<bits>" in B.last_kernel(), B.last_kernel()
    want = B.binarize_pack((alpha * (x @ w.T) >= thr).float() * 2 - 1, 1)  # (whole numbers, exact in fp32)
    assert torch.equal(out[:, :-1], want) and bool((out[:, -1] == -1).all())


@pytest.mark.parametrize("N,C,H,W,O", [(1, 300, 3, 9, 40), (1, 300, 14, 16, 33), (1, 300, 15, 15, 70), (1, 300, 15, 17, 260), (1, 300, 16, 16, 130),
                                       (7, 300, 14, 14, 300), (3, 300, 27, 29, 100)])
def test_conv_small_runs_of_pixels(N, C, H, W, O):
    """The small convolution: one block of pixels and less than eight, whole eighths, one block more; the halo written by blocks in the
    grid's order, and by runs per XCD that do not come out even (74 blocks)."""
    rng = np.random.default_rng(N + H + W + O)
    x, w = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((O, C, 3, 3)).astype(np.float32)
    alpha, thr = rng.standard_normal(O).astype(np.float32), rng.standard_normal(O).astype(np.float32)
    ri, rf = oracle.binary_conv2d(x, w, 1, 1, alpha)
    Wp, xp = B.pack_conv_weights(dev(w)), B.pack_nchw(dev(x), 1)
    got = B.binary_conv2d_packed(xp, C, Wp, O, 3, 3, 1, 1, integer_out=True)
    assert "conv_small_kernel" in B.last_kernel(), B.last_kernel()
    np.testing.assert_array_equal(got.cpu().numpy(), ri)
    np.testing.assert_array_equal(B.binary_conv2d_packed(xp, C, Wp, O, 3, 3, 1, 1, alpha=dev(alpha)).cpu().numpy(), rf)
    ref = B.pack_nchw(dev(np.where(rf >= thr[None, :, None, None], np.float32(1), np.float32(-1))), 1)
    out = torch.full(ref.shape, -1, dtype=ref.dtype, device="cuda")
    got = B.binary_conv2d_bits(xp, C, Wp, O, 3, 3, 1, 1, alpha=dev(alpha), thr=dev(thr), out_pad=1, out=out)
    assert "conv_small_kernel" in B.last_kernel(), B.last_kernel()
    np.testing.assert_array_equal(got.cpu().numpy(), ref.cpu().numpy())


@pytest.mark.parametrize("N,C,H,W,O,grid", [(3, 130, 10, 10, 64, 10), (1, 130, 47, 32, 33, 47), (1, 130, 48, 32, 33, 48), (1, 130, 683, 3, 70, 72),
                                            (1, 130, 683, 3, 480, 65), (8, 130, 23, 21, 100, 128)])
def test_conv_small_order(N, C, H, W, O, grid):
    """Pixels in runs per XCD, eight of one length, from 48 blocks on, and in the grid's order below and where a CU would have more."""
    rng = np.random.default_rng(N + H + W + O)
    x, w = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((O, C, 1, 1)).astype(np.float32)
    ri, _ = oracle.binary_conv2d(x, w, 1, 0)
    got = B.binary_conv2d_packed(B.pack_nchw(dev(x), 0), C, B.pack_conv_weights(dev(w)), O, 1, 1, 1, 0, integer_out=True)
    assert "conv_small_kernel<i32> grid %d x" % grid in B.last_kernel(), B.last_kernel()
    np.testing.assert_array_equal(got.cpu().numpy(), ri)


@pytest.mark.parametrize("N,C,H,W,O,k,s,p,shift", [
    (3, 190, 13, 12, 70, 3, 1, 1, 0),   # runs of 9 words: two meet in one segment, and a last word alone
    (3, 60, 12, 13, 40, 3, 2, 1, 0),    # runs of 3, shorter than half a segment
    (2, 60, 15, 14, 65, 7, 1, 0, 0),    # runs of 7: in every segment
    (2, 320, 9, 11, 129, 1, 2, 0, 0),   # one run, in one segment
    (4, 300, 11, 9, 64, 5, 1, 2, 0),    # 5 runs of 25
    (2, 420, 10, 10, 66, 7, 1, 3, 0),   # 7 runs of 49
    (3, 250, 12, 11, 67, 3, 1, 1, 1),   # an even number of channel words in an image that starts on an odd word
    (3, 190, 12, 11, 67, 3, 1, 1, 1),   # an odd one
])
def test_conv_odd_runs(N, C, H, W, O, k, s, p, shift):
    """The 64 x 64 per wave convolution and the one that stages a row once per workgroup, where 16-byte pieces of a patch cross
    from one kernel row to the next, or the image is 8-byte aligned only: every way of dividing K, every kind of result."""
    rng = np.random.default_rng(N + C + H + O + k)
    x, w = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha, thr = rng.standard_normal(O).astype(np.float32), rng.standard_normal(O).astype(np.float32)
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    ref_bits = B.pack_nchw(dev(np.where(rf >= thr[None, :, None, None], np.float32(1), np.float32(-1))), 1)
    Wp, packed = B.pack_conv_weights(dev(w)), B.pack_nchw(dev(x), p)
    flat = torch.empty(packed.numel() + shift, dtype=packed.dtype, device="cuda")
    xp = flat[shift:].view(packed.shape).copy_(packed)
    for pin in ({"k10": 1}, {"k10": 4}, {"k10": 8}, {"k20": 2}, {"k20": 3}):
        with tuned(k18=1, **(pin if "k20" in pin else {"k5": 6, **pin})):
            got = B.binary_conv2d_packed(xp, C, Wp, O, k, k, s, p, integer_out=True)
            assert "gemm_fp4_kernel" in B.last_kernel()
            np.testing.assert_array_equal(got.cpu().numpy(), ri)
            got = B.binary_conv2d_packed(xp, C, Wp, O, k, k, s, p, alpha=dev(alpha))
            np.testing.assert_array_equal(got.cpu().numpy(), rf)
            got = B.binary_conv2d_bits(xp, C, Wp, O, k, k, s, p, alpha=dev(alpha), thr=dev(thr), out_pad=1)
            np.testing.assert_array_equal(got.cpu().numpy(), ref_bits.cpu().numpy())


@pytest.mark.parametrize("form", [1, 2, 3])
@pytest.mark.parametrize("N,C,H,W,O,k,s,p,opad", [
    (1, 1, 1, 1, 1, 1, 1, 0, 0),        # one word, one pixel
    (2, 500, 9, 8, 65, 1, 1, 0, 1),     # whole segment, a filter past the tile
    (3, 130, 13, 11, 129, 3, 1, 1, 1),  # odd number of channel words, three segments and a half
    (2, 384, 14, 10, 128, 3, 2, 1, 2),  # even, stride 2
    (5, 300, 8, 7, 63, 5, 1, 2, 0),     # many segments, images that end inside a tile
    (1, 640, 23, 24, 200, 3, 1, 0, 1),  # several tiles each way
    (9, 70, 9, 8, 31, 7, 1, 3, 3),      # halo as wide as the image's rest
    (4, 256, 16, 16, 64, 1, 1, 0, 6),
    (300, 130, 1, 1, 70, 1, 1, 0, 0),   # a pixel an image: a tile holds as many images as pixels
    (130, 200, 3, 3, 130, 3, 2, 1, 1),  # four
    (37, 320, 7, 1, 65, 1, 1, 0, 1)])   # seven: tiles begin and end inside an image
def test_conv_long_k_kernels(form, N, C, H, W, O, k, s, p, opad):
    """Convolutions of packed images on the kernels for long K, whatever the size: rows staged once per workgroup (2: 128
    filters x 128 pixels, 3: 64 x 256), and 64 x 64 per wave (1; with and without K divided).  fp32, int32, and the next
    convolution's image with its halo, thresholds and negative scales included."""
    rng = np.random.default_rng(N + C + H + O)
    x, w = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha, thr = rng.standard_normal(O).astype(np.float32), (rng.standard_normal(O) * np.sqrt(C) * k).astype(np.float32)
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    xp, Wp = B.pack_nchw(dev(x), p), B.pack_conv_weights(dev(w))
    ref = np.where(rf >= thr[None, :, None, None], np.float32(1), np.float32(-1))
    want = B.pack_nchw(dev(ref), opad)
    for split in ((0, 1, 3, 8) if form == 1 else (0,)):
        pins = dict(k18=1, k5=6, k10=split) if form == 1 else dict(k18=1, k20=form)
        with tuned(**pins):
            np.testing.assert_array_equal(B.binary_conv2d_packed(xp, C, Wp, O, k, k, s, p, integer_out=True).cpu().numpy(), ri)
            assert "gemm_fp4_kernel" in B.last_kernel() and ("block" in B.last_kernel()) == (form > 1)
            np.testing.assert_array_equal(B.binary_conv2d_packed(xp, C, Wp, O, k, k, s, p, alpha=dev(alpha)).cpu().numpy(), rf)
            if form > 1 or k * k * -(-C // 64) not in (9, 18, 25, 27, 36, 49, 50):  # (those words' kernel writes the image itself)
                out = torch.full_like(want, -1)
                B.binary_conv2d_bits(xp, C, Wp, O, k, k, s, p, alpha=dev(alpha), thr=dev(thr), out_pad=opad, out=out)
                assert "gemm_fp4_kernel" in B.last_kernel() and "bits" in B.last_kernel()
                assert torch.equal(out, want)
    if k > 1:  # images of one row and one column of padding more, on the general route
        with tuned(k5=3):
            assert torch.equal(B.binary_conv2d_bits(xp, C, Wp, O, k, k, s, p, alpha=dev(alpha), thr=dev(thr), out_pad=opad), want)


@pytest.mark.parametrize("N,C,H,W,O,k,f32", [(44, 250, 25, 26, 391, 3, False), (21, 60, 32, 33, 384, 7, True), (20, 128, 31, 33, 449, 5, True),
                                             (43, 250, 25, 26, 127, 3, False)])
def test_conv_short_k_many_filters(N, C, H, W, O, k, f32):
    """36, 49 and 50 words with so many filters and pixels that the rows are staged once per workgroup: as the kernel for
    short K has it (by its tests against the oracle), as packed image and, from 49 words on, fp32."""
    rng = np.random.default_rng(O)
    x, w = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha, thr = dev(rng.standard_normal(O).astype(np.float32)), dev((rng.standard_normal(O) * 40).astype(np.float32))
    xp, Wp = B.pack_nchw(dev(x), k // 2), B.pack_conv_weights(dev(w))
    runs = [lambda: B.binary_conv2d_bits(xp, C, Wp, O, k, k, 1, k // 2, alpha=alpha, thr=thr, out_pad=1)]
    runs += [lambda: B.binary_conv2d_packed(xp, C, Wp, O, k, k, 1, k // 2, alpha=alpha),
             lambda: B.binary_conv2d_packed(xp, C, Wp, O, k, k, 1, k // 2, integer_out=True)]
    for i, run in enumerate(runs):
        got = run()
        assert ("gemm_fp4_kernel" in B.last_kernel()) == (O >= 128 and (f32 or i == 0)), B.last_kernel()
        with tuned(k20=1):
            assert torch.equal(got, run())
            assert "conv_mfma_ws_kernel" in B.last_kernel()


@pytest.mark.parametrize("N,C,H,W,O,k,s,p,opad", [
    (1, 1, 1, 1, 1, 1, 1, 0, 0), (3, 300, 5, 7, 33, 1, 2, 0, 2), (2, 128, 9, 8, 70, 3, 1, 1, 1), (2, 131, 6, 5, 32, 3, 2, 2, 0), (1, 70, 8, 9, 95, 5, 1, 4, 3),
    (5, 64, 7, 7, 64, 7, 1, 3, 1), (2, 260, 6, 11, 129, 3, 1, 1, 6), (1, 512, 9, 9, 31, 7, 2, 6, 1), (40, 200, 12, 13, 100, 3, 1, 0, 1), (9, 50, 40, 41, 64, 1, 1, 0, 1)])
def test_conv_small(N, C, H, W, O, k, s, p, opad):
    """The kernel for small convolutions of packed images: 1 to 16 waves per tile, odd and even numbers of
    channel words, patches that end inside a step, tiles that straddle images and are not full, an odd
    number of 32-filter tiles (the upper half of the last word is written), halos of the result."""
    rng = np.random.default_rng(N + C + H + O + k)
    x, w = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((O, C, k, k)).astype(np.float32)
    alpha, thr = rng.standard_normal(O).astype(np.float32), rng.standard_normal(O).astype(np.float32)
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    xp, Wp = B.pack_nchw(dev(x), p), B.pack_conv_weights(dev(w))
    got = B.binary_conv2d_bits(xp, C, Wp, O, k, k, s, p, alpha=dev(alpha), thr=dev(thr), out_pad=opad)
    assert "conv_small_kernel<bits>" in B.last_kernel()
    ref = np.where(rf >= thr[None, :, None, None], np.float32(1), np.float32(-1))
    np.testing.assert_array_equal(got.cpu().numpy(), B.pack_nchw(dev(ref), opad).cpu().numpy())
    np.testing.assert_array_equal(B.binary_conv2d_packed(xp, C, Wp, O, k, k, s, p, integer_out=True).cpu().numpy(), ri)
    assert ("conv_small_kernel<i32>" in B.last_kernel()) == (C > 64 or k > 1)
    np.testing.assert_array_equal(B.binary_conv2d_packed(xp, C, Wp, O, k, k, s, p, alpha=dev(alpha)).cpu().numpy(), rf)


@pytest.mark.parametrize("N,O,off,small", [(12, 64, 0, False), (10, 64, 0, True), (24, 30, 0, True), (28, 30, 0, False), (12, 64, 1, True)])
def test_conv_small_lines(N, O, off, small):
    """Both sides of the line to the 64 x 64 kernel at 45 words and 12 steps a tile, for filters that fill its tiles and for such as
    leave them half empty, and filters that are 8-byte aligned, which it does not take; the same results from the popcount kernel."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N + O)
    x, w = torch.randn((N, 320, 40, 40), device="cuda", generator=g), torch.randn((O, 320, 3, 3), device="cuda", generator=g)
    xp, Wp = B.pack_nchw(x, 1), B.pack_conv_weights(w)
    room = torch.empty(Wp.numel() + off, dtype=Wp.dtype, device="cuda")[off:].view(Wp.shape)
    got = B.binary_conv2d_packed(xp, 320, room.copy_(Wp), O, 3, 3, 1, 1, integer_out=True)
    assert ("conv_small_kernel" in B.last_kernel()) == small, B.last_kernel()
    with tuned(k7=1):
        assert torch.equal(got, B.binary_conv2d_packed(xp, 320, Wp, O, 3, 3, 1, 1, integer_out=True))


@pytest.mark.parametrize("parts,N,C,H,W,O,k,s,p", [
    (1, 1, 1, 1, 1, 1, 1, 1, 0), (1, 3, 17, 9, 11, 33, 1, 2, 0), (1, 12, 390, 24, 26, 83, 1, 1, 0), (2, 2, 64, 10, 9, 32, 3, 1, 1),
    (2, 5, 42, 29, 28, 31, 3, 2, 2), (4, 7, 130, 29, 27, 70, 3, 2, 1), (4, 1, 33, 7, 6, 65, 5, 1, 4), (8, 2, 211, 8, 20, 19, 3, 1, 0),
    (8, 1, 256, 5, 5, 40, 5, 2, 2), (8, 3, 65, 13, 13, 29, 7, 1, 6), (1, 2, 16, 40, 130, 20, 3, 1, 1), (1, 40, 31, 12, 12, 200, 3, 1, 1)])
def test_conv_one_launch(parts, N, C, H, W, O, k, s, p):
    """The one-launch convolution: K split over 1 to 8 waves, patches that end inside a step of four
    words, channels that end inside sixteen or inside a word, a filter tile and a pixel block that are
    not full, the last band shorter than the others, bands that lie in the padding alone, strides."""
    rng = np.random.default_rng(N + C + H + O + k)
    x, w = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((O, C, k, k)).astype(np.float32)
    x[rng.random(x.shape) < 0.05] = 0.0
    alpha = rng.standard_normal(O).astype(np.float32)
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    np.testing.assert_array_equal(run_conv(x, w, s, p, integer_out=True), ri)
    assert "conv_one_kernel" in B.last_kernel() and "%d parts of K" % parts in B.last_kernel(), B.last_kernel()
    np.testing.assert_array_equal(run_conv(x, w, s, p, alpha=alpha), rf)
    np.testing.assert_array_equal(run_conv(x, w, s, p), ri.astype(np.float32))


@pytest.mark.parametrize("waves,parts,N,C,H,W,O,k,s,p", [
    (4, 2, 1, 16, 3, 3, 5, 3, 1, 1), (4, 1, 40, 40, 20, 22, 30, 1, 1, 0), (4, 2, 3, 15, 8, 8, 20, 3, 1, 1), (4, 4, 1, 190, 17, 4, 20, 3, 1, 1),
    (8, 2, 60, 130, 16, 18, 20, 3, 1, 1), (8, 4, 2, 113, 25, 30, 70, 3, 1, 1), (8, 8, 1, 460, 16, 16, 512, 3, 1, 1), (8, 4, 4, 129, 20, 20, 129, 3, 1, 1),
    (12, 4, 2, 320, 6, 23, 300, 3, 2, 1), (12, 8, 20, 320, 19, 11, 20, 5, 1, 2), (16, 2, 100, 130, 11, 3, 200, 3, 1, 1),
    (16, 4, 1, 4101, 5, 5, 300, 1, 1, 0), (16, 4, 2, 1000, 30, 31, 33, 1, 1, 0)])
def test_conv_one_launch_waves(waves, parts, N, C, H, W, O, k, s, p):
    """The one-launch convolution in workgroups of 4 to 16 waves: items of the pack that do not divide by them, channels that
    end in each sixteenth of a word (the words behind are cleared), patches of up to 64 words a wave; NaN, zeros and
    infinities among the values."""
    rng = np.random.default_rng(C + H + O)
    x, w = rng.standard_normal((N, C, H, W)).astype(np.float32), rng.standard_normal((O, C, k, k)).astype(np.float32)
    x[rng.random(x.shape) < 0.02] = -0.0
    x[rng.random(x.shape) < 0.02] = np.nan
    x[rng.random(x.shape) < 0.02] = -np.inf
    alpha = rng.standard_normal(O).astype(np.float32)
    ri, rf = oracle.binary_conv2d(x, w, s, p, alpha)
    with tuned(k16=2):
        np.testing.assert_array_equal(run_conv(x, w, s, p, integer_out=True), ri)
        assert "conv_one_kernel" in B.last_kernel() and "x %d," % (64 * waves) in B.last_kernel(), B.last_kernel()
        assert "%d parts of K" % parts in B.last_kernel(), B.last_kernel()
        np.testing.assert_array_equal(run_conv(x, w, s, p, alpha=alpha), rf)


@pytest.mark.parametrize("N,C,H,W,O,k,s,p,call,graph", [
    (25, 40, 21, 21, 320, 5, 2, 2, False, False), (126, 107, 42, 44, 18, 3, 1, 1, False, False), (136, 128, 16, 16, 458, 1, 1, 0, False, False),
    (2, 142, 50, 50, 64, 3, 2, 1, True, False), (3, 256, 25, 25, 128, 3, 1, 1, True, False), (7, 130, 29, 27, 70, 3, 2, 1, True, True), (1, 64, 8, 8, 64, 1, 1, 0, True, True),
    (123, 445, 11, 10, 18, 1, 2, 0, True, True)])
def test_conv_one_launch_or_two(N, C, H, W, O, k, s, p, call, graph):
    """Layers that look short to a model that counts workgroups by the chip and not by its XCDs, or bytes and not loads, take two
    launches; layers whose two launches are held up by the host alone take one as a call and two in a graph; replays between
    calls give what the calls give."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N + C)
    x = torch.randn((N, C, H, W), device="cuda", generator=g)
    w = torch.randn((O, C, k, k), device="cuda", generator=g)
    Wp, alpha = B.pack_conv_weights(w), B.alpha_mean_abs(w)
    run = lambda: B.binary_conv2d(x, Wp, O, k, k, s, p, alpha=alpha)  # noqa: E731
    run()
    assert ("conv_one" in B.last_kernel()) == call, B.last_kernel()
    torch.cuda.synchronize()
    captured = torch.cuda.CUDAGraph()
    with torch.cuda.graph(captured):
        out = run()
        assert ("conv_one" in B.last_kernel()) == graph, B.last_kernel()
    for _ in range(3):
        x.normal_(generator=g)
        captured.replay()
        want = run()
        assert ("conv_one" in B.last_kernel()) == call, B.last_kernel()
        assert torch.equal(out, want)
        with tuned(k16=1):
            assert torch.equal(run(), want)


# ------------------------------------------------------------------ ties of the quantiser
@pytest.mark.parametrize("bits", range(1, 9))
@pytest.mark.parametrize("rows,engine", [(300, {}), (300, {"k7": 3}), (40, {"k7": 1}), (5, {})])
def test_quantiser_ties_on_every_form(bits, rows, engine):
    """Values around every tie of Eq. 1: the level is that of the fp32 product L * x, rounded half away from zero, and
    not of the exact product (at 5 and 7 bits they differ for some floats).  One launch, bytes and planes; the planes'
    own choice below 256 results."""
    L = np.float32((1 << bits) - 1)
    x = ((np.arange(1 << bits) + 0.5) / float(L)).astype(np.float32)
    at = [x]
    for way in (np.float32(0), np.float32(2)):
        v = x
        for _ in range(3):
            v = np.nextafter(v, way)
            at.append(v)
    x = np.concatenate(at)
    x = np.resize(x[x <= 1], max(2048, x.size))
    a = np.stack([np.roll(x, 7 * r) for r in range(rows)])
    w = np.random.default_rng(bits).choice(np.float32([-1, 1]), (40, x.size)) if rows > 5 else np.eye(40, x.size, dtype=np.float32) * 2 - 1
    for bw in (1, bits):
        wb = w if bw == 1 else np.stack([np.roll(2 * x - 1, 11 * r) for r in range(40)])
        rS, _, _ = oracle.quant_gemm(a, wb, bits, bw)
        with tuned(**engine):
            S, _ = B.quant_gemm(dev(a), dev(wb), bits, bw, want_float=False)
        np.testing.assert_array_equal(S.cpu().numpy(), rS, err_msg=B.last_kernel())


@pytest.mark.parametrize("bits", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("M,N,K,engine", [(70, 60, 1100, {"k7": 1}), (300, 290, 2100, {"k7": 3}), (300, 290, 2100, {}), (5, 9, 130, {})])
def test_quantiser_takes_nan_as_zero(M, N, K, engine, bits):
    """NaN of either sign is level 0 of an activation and of a k-bit weight, and -1 as a one-bit weight, on every form: planes
    (the popcount and the FP4 kernels), bytes, one launch."""
    rng = np.random.default_rng(M + K + bits)
    a, w = rng.uniform(-0.1, 1.1, (M, K)).astype(np.float32), rng.uniform(-1, 1, (N, K)).astype(np.float32)
    for t in (a, w):
        t[rng.random(t.shape) < 0.1] = np.nan
        t[rng.random(t.shape) < 0.1] = -np.nan
    for bw in (1, bits):
        rS, _, _ = oracle.quant_gemm(np.nan_to_num(a, nan=0.0), np.nan_to_num(w, nan=-1.0), bits, bw)
        with tuned(**engine):
            S, _ = B.quant_gemm(dev(a), dev(w), bits, bw, want_float=False)
        np.testing.assert_array_equal(S.cpu().numpy(), rS, err_msg=B.last_kernel())


# ------------------------------------------------------------------ few bits: bytes or planes
@pytest.mark.parametrize("M,N,K,bits_a,bytes_form", [
    (16, 2048, 8192, 2, False), (32, 1900, 8192, 2, False), (16, 200, 16384, 1, False), (100, 32, 10000, 2, True),
    (16, 900, 4096, 2, True), (475, 1088, 832, 2, True), (360, 4096, 832, 1, False), (130, 300, 4097, 1, True),
    (100, 900, 10000, 2, True), (100, 900, 8192, 2, False)])
def test_few_bits_on_the_byte_form_or_the_plane_form(M, N, K, bits_a, bytes_form):
    rng = np.random.default_rng(K + M)
    a = rng.uniform(-0.2, 1.2, (M, K)).astype(np.float32)
    w = rng.standard_normal((N, K)).astype(np.float32)
    S, _ = B.quant_gemm(dev(a), dev(w), bits_a, 1, want_float=False)
    assert ("gemm_i8_kernel" in B.last_kernel()) == bytes_form, B.last_kernel()
    with tuned(k7=3):
        P, _ = B.quant_gemm(dev(a), dev(w), bits_a, 1, want_float=False)
        assert "gemm_i8_kernel" not in B.last_kernel() and "quant_small" not in B.last_kernel()
    assert torch.equal(S, P)
    q = np.floor((np.float32((1 << bits_a) - 1) * np.clip(a, 0, 1)).astype(np.float64) + 0.5)  # half away from zero
    at = rng.integers(0, M, 8)
    np.testing.assert_array_equal(S.cpu().numpy()[at], (q[at] @ np.where(w >= 0, 1.0, -1.0).T).astype(np.int32))


# ------------------------------------------------------------------ matrices given with more dimensions
@pytest.mark.parametrize("N", [1, 5])
def test_contiguous_tensors_of_more_dimensions_are_rows(N):
    rng = np.random.default_rng(N)
    H, W, C, F = 3, 4, 128, 24
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = rng.standard_normal((F, H * W * C)).astype(np.float32)
    img, Wp = B.pack_nchw(dev(x), 0), B.binarize_pack(dev(w), 1)
    flat = img.view(N, -1)
    want = B.binary_fc_packed(flat, H * W * C, Wp, mode="i32")
    rows = oracle.binarize_pack(np.ascontiguousarray(np.transpose(x, (0, 2, 3, 1)).reshape(N, -1)), 1)
    np.testing.assert_array_equal(host_u64(flat), rows)
    np.testing.assert_array_equal(want.cpu().numpy(), oracle.xnor_gemm(rows, host_u64(Wp), H * W * C))
    assert img.dim() == 4
    assert torch.equal(B.binary_fc_packed(img, H * W * C, Wp, mode="i32"), want)
    assert torch.equal(B.binary_fc_packed(img, H * W * C, Wp.view(F, H, -1), mode="f32"), want.float())
    bits = torch.empty((N, 1, 1), dtype=torch.int64, device="cuda")
    assert torch.equal(B.binary_fc_packed(img, H * W * C, Wp, mode="bits", out=bits).view(N, 1),
                       B.binary_fc_packed(flat, H * W * C, Wp, mode="bits"))
    out = torch.empty((N, 4, 6), dtype=torch.int32, device="cuda")
    assert B.xnor_gemm(img, Wp, H * W * C, out=out) is out and torch.equal(out.view(N, F), want)
    dense = dev(rng.standard_normal((N, 300)).astype(np.float32))
    wd = B.binarize_pack(dev(rng.standard_normal((F, 300)).astype(np.float32)), 1)
    fout = torch.empty((N, 2, 12), dtype=torch.float32, device="cuda")
    assert torch.equal(B.binary_fc(dense, wd, out=fout).view(N, F), B.binary_fc(dense, wd))
    as32 = img.view(torch.int32)
    out.zero_()
    assert torch.equal(B.xnor_gemm_w32(as32, Wp.view(torch.int32).view(F, H, -1), H * W * C, out=out).view(N, F), want)
    assert torch.equal(B.unpack_pm1(img, H * W * C), B.unpack_pm1(flat, H * W * C))


def test_rows_of_one_word_as_a_vector_and_what_stays_refused():
    rng = np.random.default_rng(3)
    A, W = (B.binarize_pack(dev(rng.standard_normal((n, 50)).astype(np.float32)), 1) for n in (9, 7))
    want = B.xnor_gemm(A, W, 50)
    assert torch.equal(B.xnor_gemm(A.view(9), W.view(7), 50), want)
    with pytest.raises(ValueError):
        B.xnor_gemm(A.view(3, 3, 1).transpose(0, 1), W, 50)      # more dimensions, not contiguous
    with pytest.raises(ValueError):
        B.xnor_gemm(A[0, 0], W, 50)                              # no rows at all
    with pytest.raises(ValueError):
        B.binary_fc(torch.zeros((2, 5, 10), device="cuda"), W)   # fp32 rows have two dimensions
    img = B.pack_nchw(dev(rng.standard_normal((2, 40, 6, 6)).astype(np.float32)), 1)
    Wp = B.pack_conv_weights(dev(rng.standard_normal((5, 40, 3, 3)).astype(np.float32)))
    assert torch.equal(B.binary_conv2d_packed(img.view(2, 8, 8), 40, Wp, 5, 3, 3, 1, 1),
                       B.binary_conv2d_packed(img, 40, Wp, 5, 3, 3, 1, 1))
    with pytest.raises(B.BmxError):
        B.xnor_gemm(A.view(9), W, 65)                            # a row of one word holds 64 values
