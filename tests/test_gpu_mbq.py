"""GPU parity, scheme M: bit planes bit-exact, header within 1e-6 * sum|alpha| (the sums
are reduced in a different order), decoded values within 1e-6 * sum|alpha| and bit-exact
when the decoder is fed the oracle's own header and payload."""
import numpy as np
import pytest

import synthetic_inputs as si
from oracle import accept_oracle as orc

from gpu_util import bytes_to_dev, dev_bytes, first_mismatch, out_to_numpy, to_dev, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    torch = torch_mod()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2311_05827_amd as pkg
    return pkg


def run_case(A, x, k, n, m, t=1, alpha_prev=None, in_bf16=False, out_bf16=False, tag=""):
    torch = torch_mod()
    print("case", tag, "k", k, "n", n, "m", m, "t", t, "bf16", in_bf16, out_bf16, flush=True)
    xd, bits = to_dev(x, in_bf16)
    xin = orc.widen_bf16(bits) if in_bf16 else np.asarray(x, np.float32).reshape(-1)
    if alpha_prev is None:
        alpha_prev, _ = orc.mbq_residue_init(xin, k)
    ad = torch.from_numpy(np.asarray(alpha_prev, np.float32)).cuda()
    d = A.make_desc(A.MBQ, k, n, m, in_dtype=A.BF16 if in_bf16 else A.F32,
                    out_dtype=A.BF16 if out_bf16 else A.F32, t=t)
    header, payload = A.accept_compress(d, xd, alpha_prev=ad)
    xh = A.accept_decompress(d, header, payload)
    torch.cuda.synchronize()
    oh, op = orc.mbq_compress(bits if in_bf16 else x, k, n, m, alpha_prev, t, in_bf16)
    mm = first_mismatch(dev_bytes(payload), op.tobytes())
    assert mm is None, "payload differs: " + mm
    gh = np.frombuffer(dev_bytes(header), dtype="<f4")
    ohf = np.frombuffer(oh, dtype="<f4")
    scale = float(np.sum(np.abs(ohf[:k])))
    assert np.all(np.abs(gh.astype(np.float64) - ohf.astype(np.float64)) <= 1e-6 * scale), (gh, ohf)
    # decoder fed the oracle's header and payload: bit-exact
    xh2 = A.accept_decompress(d, bytes_to_dev(oh), bytes_to_dev(op.tobytes()))
    torch.cuda.synchronize()
    oxh = orc.mbq_decompress(oh, op, k, n, m, out_bf16)
    got2 = out_to_numpy(xh2)
    assert got2.tobytes() == oxh.tobytes()
    # decoder fed the GPU's own header: within tolerance of the oracle's output
    got = out_to_numpy(xh)
    if out_bf16:
        g32, o32 = orc.widen_bf16(got), orc.widen_bf16(oxh)
        assert np.all(np.abs(g32.astype(np.float64) - o32.astype(np.float64)) <= 2.0 ** -7 * np.abs(o32) + 1e-6 * scale)
    else:
        assert np.all(np.abs(got.astype(np.float64) - oxh.astype(np.float64)) <= 1e-6 * scale)
    return gh, ohf


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8])
def test_small_shapes_every_k(A, k):
    for n, m in [(8, 1), (16, 5), (3, 7), (9, 4), (1, 1), (64, 36), (13, 260), (24, 1030)]:
        x = si.make_shape("relu_normal", (n, m), 1000 + 10 * k + n)
        run_case(A, x, k, n, m, t=3, tag="small")


@pytest.mark.parametrize("k", [2, 3, 4])
@pytest.mark.parametrize("t", [0, 1, 50, 100])
def test_multi_block_shapes(A, k, t):
    # several workgroups, row-group boundary inside a wavefront, n not a multiple of 8
    x = si.make_shape("relu_lognormal", (21, 4100), 2000 + k)
    run_case(A, x, k, 21, 4100, t=t, tag="21x4100")
    x = si.make_shape("relu_normal", (256, 1024), 2001 + k)
    run_case(A, x, k, 256, 1024, t=t, tag="256x1024")
    x = si.make_shape("student_t3", (12, 4099), 2002 + k)  # m not a multiple of 4: scalar path
    run_case(A, x, k, 12, 4099, t=t, tag="12x4099")


@pytest.mark.parametrize("k", [2, 3, 4])
def test_config1_activation_both_views(A, k):
    x = si.make("cfg1_act")
    run_case(A, x, k, 4, 65536, t=1, tag="cfg1 n=4 (padded to 8 rows)")
    run_case(A, x, k, 256, 1024, t=1, tag="cfg1 as 256x1024")


@pytest.mark.parametrize("k", [2, 4, 6])
@pytest.mark.parametrize("in_bf16,out_bf16", [(True, False), (False, True), (True, True)])
def test_bf16_io(A, k, in_bf16, out_bf16):
    x = si.make_shape("relu_lognormal", (16, 2056), 3000 + k)
    run_case(A, x, k, 16, 2056, in_bf16=in_bf16, out_bf16=out_bf16, tag="bf16 vec8")
    x = si.make_shape("relu_lognormal", (10, 1004), 3001 + k)  # 1004 % 8 != 0: scalar path
    run_case(A, x, k, 10, 1004, in_bf16=in_bf16, out_bf16=out_bf16, tag="bf16 scalar")


def test_alpha_carried_across_batches(A):
    """Feed header[0..k) back as alpha_prev for a few batches, oracle and GPU each on
    their own chain; the chains must stay within tolerance of each other."""
    torch = torch_mod()
    k, n, m = 3, 32, 2048
    a_gpu = a_orc = None
    for t in range(4):
        x = si.make_shape("relu_normal", (n, m), 4000 + t)
        if t == 0:
            a_orc, _ = orc.mbq_residue_init(x, k)
            a_gpu = a_orc.copy()
        xd, _ = to_dev(x)
        d = A.make_desc(A.MBQ, k, n, m, t=t)
        header, payload = A.accept_compress(d, xd, alpha_prev=torch.from_numpy(a_gpu).cuda())
        torch.cuda.synchronize()
        oh, op = orc.mbq_compress(x, k, n, m, a_orc, t)
        a_gpu = np.frombuffer(dev_bytes(header), dtype="<f4")[:k].copy()
        a_orc = np.frombuffer(oh, dtype="<f4")[:k].copy()
        assert np.all(np.abs(a_gpu - a_orc) <= 4e-6 * np.sum(np.abs(a_orc)))
        differing = np.count_nonzero(np.frombuffer(dev_bytes(payload), np.uint8) != op)
        assert differing <= 0.001 * op.size  # only elements within an ulp of a threshold may move


def test_singular_gram_and_special_values(A):
    # constant input: every element takes the same level, B^T B is singular -> alpha stays
    x = np.full((8, 64), 5.0, np.float32)
    gh, ohf = run_case(A, x, 2, 8, 64, alpha_prev=np.array([1.0, 0.5], np.float32), tag="singular")
    assert gh[:2].tolist() == [1.0, 0.5]
    # duplicate levels (alpha_0 == alpha_1) and a zero coefficient
    x = si.make_shape("relu_normal", (16, 260), 5000)
    run_case(A, x, 2, 16, 260, alpha_prev=np.array([0.5, 0.5], np.float32), tag="dup-levels")
    run_case(A, x, 3, 16, 260, alpha_prev=np.array([0.7, 0.0, 0.2], np.float32), tag="zero-alpha")
    # positive and negative denormals must fall on their own side of the zero threshold;
    # exact threshold values go to the lower level
    a = np.array([0.75, 0.25], np.float32)
    _, _, tau = orc.mbq_levels(a)
    vals = np.concatenate([tau, [1e-40, -1e-40, 0.0, -0.0, 1e-45, -1e-45]]).astype(np.float32)
    x = np.resize(vals, (8, 36)).astype(np.float32)
    run_case(A, x, 2, 8, 36, alpha_prev=a, tag="thresholds+denormals")


@pytest.mark.parametrize("k,alpha", [(3, [1.0, 0.03, 0.02]), (4, [1.0, 0.5, 0.03, 0.02]), (4, [0.6, 0.58, 0.3, 0.29])])
def test_two_thresholds_per_bucket(A, k, alpha):
    """Levels closer than the width of a bucket of the level search's float-prefix table: the
    encoder then compares against two thresholds per element.  The shapes give whole pipelined
    rounds, a last incomplete round and a ragged last row group; values sit on and next to the
    thresholds as well."""
    a = np.asarray(alpha, np.float32)
    _, _, tau = orc.mbq_levels(a)
    for n, m, bf in [(8, 8 * 1024 * 100 + 4 * 37, False), (19, 400004, False), (16, 800008, True), (5, 1003, False)]:
        x = si.make_shape("student_t3", (n, m), 7100 + n)
        x = (x * np.float32(0.8 / x.std())).astype(np.float32)
        edge = np.concatenate([tau, np.nextafter(tau, np.float32(np.inf)), np.nextafter(tau, np.float32(-np.inf))])
        x.reshape(-1)[: edge.size * 5 : 5] = edge.astype(np.float32)
        run_case(A, x, k, n, m, alpha_prev=a, in_bf16=bf, tag="two-per-bucket")


@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_residue_init(A, k):
    torch = torch_mod()
    for shape, bf in [((16, 1000), False), ((7, 333), False), ((16, 1000), True)]:
        x = si.make_shape("relu_lognormal", shape, 6000 + k)
        xd, bits = to_dev(x, bf)
        xin = orc.widen_bf16(bits) if bf else x
        d = A.make_desc(A.MBQ, k, shape[0], shape[1], in_dtype=A.BF16 if bf else A.F32)
        a0 = A.accept_mbq_init(d, xd)
        torch.cuda.synchronize()
        exp, _ = orc.mbq_residue_init(xin, k)
        got = a0.cpu().numpy()
        assert np.all(np.abs(got.astype(np.float64) - exp.astype(np.float64)) <= 1e-6 * float(np.sum(np.abs(exp)))), (got, exp)


@pytest.mark.parametrize("k", [1, 2, 3, 4, 6])
def test_batch0_compress(A, k):
    """accept_mbq_compress_first: header [alpha^0, m_q] within 1e-6 * sum|alpha| of the oracle's,
    bit planes of B^0 bit-exact for the GPU's own alpha^0 bits, and the decoder reads the pair
    like any other batch."""
    torch = torch_mod()
    # in one kernel (k <= 4), then, from 32769 items of eight rows on, in a kernel for every pass: single columns, and vectors for k = 1
    # and 6 (k = 2 to 4 of vectors: test_batch0_held)
    for shape, bf in [((16, 1000), False), ((7, 333), False), ((21, 4100), False), ((24, 2056), True), ((10, 1004), True),
                      ((64, 8192 + 4), False),
                      ((21, 43700), False), ((13, 16387), False), ((10, 131080), True), ((9, 16389), True), ((16, 65540), False)]:
        n, m = shape
        print("batch0 k", k, "shape", shape, "bf16", bf, flush=True)
        x = si.make_shape("relu_lognormal", shape, 6500 + k)
        x.reshape(-1)[::97] = 0.0
        xd, bits = to_dev(x, bf)
        xin = orc.widen_bf16(bits) if bf else x
        d = A.make_desc(A.MBQ, k, n, m, in_dtype=A.BF16 if bf else A.F32)
        header, payload = A.accept_mbq_compress_first(d, xd)
        xh = A.accept_decompress(d, header, payload)
        torch.cuda.synchronize()
        gh = np.frombuffer(dev_bytes(header), dtype="<f4")
        oh, _ = orc.mbq_compress_first(xin, k, n, m)
        ohf = np.frombuffer(oh, dtype="<f4")
        scale = float(np.sum(np.abs(ohf[:k])))
        assert np.all(np.abs(gh.astype(np.float64) - ohf.astype(np.float64)) <= 1e-6 * scale), (gh, ohf)
        op = orc.mbq_pack(orc.mbq_residue_signs(xin, gh[:k]), k, n, m)
        mm = first_mismatch(dev_bytes(payload), op.tobytes())
        assert mm is None, "B^0 planes differ: " + mm
        ref = orc.mbq_decompress(dev_bytes(header), op, k, n, m)
        assert out_to_numpy(xh).tobytes() == ref.tobytes()
        # the stand-alone initialisation gives the same alpha^0 bits
        a0 = A.accept_mbq_init(d, xd)
        torch.cuda.synchronize()
        assert a0.cpu().numpy().tobytes() == gh[:k].tobytes()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("k", [1, 2, 4, 5])
@pytest.mark.parametrize("bad", ["nan", "negative nan", "inf", "-inf"])
def test_batch0_planes_with_values_that_are_not_finite(A, k, bf16, bad):
    """b_j = +1 where rho_j >= 0, which a residue that is not a number is not, whatever its sign bit.  The last two
    shapes take a kernel for every pass (the last one for k = 2 and 4 is kept in registers: test_batch0_held_values_that_are_not_finite goes beyond)."""
    torch = torch_mod()
    for n, m in ((16, 1000), (7, 333), (9, 16389), (13, 131200)):
        x = si.make_shape("student_t3", (n, m), 7700 + k)
        x.reshape(-1)[::53] = {"nan": np.nan, "negative nan": -np.nan, "inf": np.inf, "-inf": -np.inf}[bad]
        x.reshape(-1)[::61] = 0.0
        xd = torch.from_numpy(x.reshape(-1)).cuda()
        xd = xd.to(torch.bfloat16) if bf16 else xd
        d = A.make_desc(A.MBQ, k, n, m, in_dtype=A.BF16 if bf16 else A.F32)
        header, payload = A.accept_mbq_compress_first(d, xd)
        torch.cuda.synchronize()
        with np.errstate(invalid="ignore"):
            oh, op = orc.mbq_compress_first(xd.float().cpu().numpy(), k, n, m)
        gh, ohf = np.frombuffer(dev_bytes(header), dtype="<f4"), np.frombuffer(oh, dtype="<f4")
        assert np.array_equal(np.isnan(gh), np.isnan(ohf)) and np.array_equal(np.isinf(gh), np.isinf(ohf)), (gh, ohf)
        mm = first_mismatch(dev_bytes(payload), op.tobytes())
        assert mm is None, "B^0 planes differ: " + mm


@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_bf16_every_value(A, k):
    """bfloat16 and k <= 4 go through a table of all 65536 values: every finite one, with
    coefficients whose levels lie far apart, close together, on top of each other and among the
    smallest numbers.  (The header is a least-squares solution, ill-conditioned for the odd
    coefficients: checked for the first set, where it is not.)"""
    torch = torch_mod()
    bits = np.arange(65536, dtype=np.uint32)
    bits = bits[(bits & 0x7F80) != 0x7F80].astype(np.uint16)      # 65280 finite values
    values = orc.widen_bf16(bits)
    for n, m in ((16, 4080), (15, 4351)):                          # whole vectors; odd rows and a partial row group
        x = values[: n * m].reshape(n, m)
        tame = np.where(np.abs(x) > 4, np.sign(x) * np.float32(3), x).astype(np.float32)
        run_case(A, tame, k, n, m, alpha_prev=np.array([1.0, 0.5, 0.25, 0.125][:k], np.float32), in_bf16=True, tag="every value")
        xd, xb = to_dev(x, True)
        d = A.make_desc(A.MBQ, k, n, m, in_dtype=A.BF16, t=1)
        for alpha in ([1.0, 1.0, 1.0, 1.0], [0.7, 0.699, 0.0007, 1e-30], [2e-38, 1e-38, 5e-39, 3e-39], [-3.0, 2.0, 1e5, 0.0]):
            a = np.array(alpha[:k], np.float32)
            _, payload = A.accept_compress(d, xd, alpha_prev=torch.from_numpy(a).cuda())
            torch.cuda.synchronize()
            want = orc.mbq_pack(orc.mbq_assign(orc.widen_bf16(xb), a), k, n, m)
            assert first_mismatch(dev_bytes(payload), want.tobytes()) is None, (n, m, alpha)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("kind", ["outliers", "cancelling", "wide"])
@pytest.mark.parametrize("k", [2, 3, 4])
def test_header_of_values_that_differ_much(A, k, kind, bf16):
    """The header against the sums in 64 bits, with terms of very different size.  An item's sums are
    float32: at most 64 terms, in 32 steps (two-term dot products) or 64, each good to an ulp of the
    largest number in it, so to 2^-23 of the item's sum |x|; they add up in float64.  With E = 64 * 2^-23 *
    sum |x| the plane sums H and S_x are within E, B^T x = 2 H - S_x within 3 E, and the bounds of alpha_t
    and m_q follow (plus their own rounding to float32)."""
    torch = torch_mod()
    rng = np.random.default_rng(7500 + k)
    for n, m in ((64, 2048), (13, 1003)):
        x = rng.standard_normal((n, m))
        if kind == "outliers":
            x *= np.where(rng.random((n, m)) < 0.01, 1e3, 1.0)
        elif kind == "cancelling":
            x = np.where(rng.random((n, m)) < 0.05, np.sign(x) * 1e4, x)
        else:
            x *= np.exp2(rng.integers(-20, 20, (n, m)))
        xd, bits = to_dev(x.astype(np.float32), bf16)
        x32 = orc.widen_bf16(bits) if bf16 else x.astype(np.float32).reshape(-1)
        alpha = (np.median(np.abs(x32)) * 0.5 ** np.arange(k)).astype(np.float32)
        d = A.make_desc(A.MBQ, k, n, m, in_dtype=A.BF16 if bf16 else A.F32, t=0)
        header, _ = A.accept_compress(d, xd, alpha_prev=torch.from_numpy(alpha).cuda())
        torch.cuda.synchronize()
        got = np.frombuffer(dev_bytes(header), dtype="<f4").astype(np.float64)
        G, h, Sb, Sx = orc.mbq_stats(x32, orc.mbq_assign(x32, alpha), k)
        beta, N = orc.beta(0), n * m
        want = beta * alpha.astype(np.float64) + (1 - beta) * np.linalg.solve(G, h)
        E = 64 * 2.0 ** -23 * np.abs(x32.astype(np.float64)).sum()
        d_alpha = (1 - beta) * np.abs(np.linalg.inv(G)).sum(axis=1) * 3 * E + 2.0 ** -23 * np.abs(want)
        mq = (want @ Sb - Sx) / N
        d_mq = (np.abs(Sb) @ d_alpha + E) / N + 2.0 ** -23 * abs(mq)
        assert np.all(np.abs(got[:k] - want) <= d_alpha), (got, want, d_alpha)
        assert abs(got[k] - mq) <= d_mq, (got[k], mq, d_mq)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 23])
def test_rows_at_any_alignment(A, n, bf16):
    """Rows that are not whole 16-byte vectors, from the narrowest that can go in vectors (64 of them) on,
    and just below it; complete and partial row groups.  The sizes from which the encoder takes vectors at any
    alignment stand in the next test."""
    vec = 8 if bf16 else 4
    for i, m in enumerate([64 * vec - 1, 64 * vec, 64 * vec + 1, 65 * vec - 1, 1024 + 3, 128 * vec + 2, 40 * 64 * vec + vec - 1]):
        k = 1 + (i + n) % 4
        x = si.make_shape("student_t3" if i % 2 else "relu_normal", (n, m), 7300 + 10 * n + i)
        run_case(A, x, k, n, m, t=2, in_bf16=bf16, out_bf16=bf16, tag="ragged")
    # levels that share a bucket of the search table: two of them, and more
    for alpha in ([1.0, 0.52, 0.26, 0.1301], [1.0, 0.99, 0.011, 0.01]):
        m = 40 * 64 * vec + 3
        x = si.make_shape("student_t3", (n, m), 7400 + n)
        d = A.make_desc(A.MBQ, 4, n, m, in_dtype=A.BF16 if bf16 else A.F32, t=1)
        xd, bits = to_dev(x, bf16)
        a = np.array(alpha, np.float32)
        torch = torch_mod()
        _, payload = A.accept_compress(d, xd, alpha_prev=torch.from_numpy(a).cuda())
        torch.cuda.synchronize()
        want = orc.mbq_pack(orc.mbq_assign(orc.widen_bf16(bits) if bf16 else x, a), 4, n, m)
        assert first_mismatch(dev_bytes(payload), want.tobytes()) is None, (n, m, alpha)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n,m", [(16, 65535), (16, 65539), (8 * 511, 257 + 256), (9, 196607), (9, 196613), (8 * 768 + 5, 513),
                                 (8 * 255 + 5, 4103), (8 * 256 + 5, 4103), (8 * 4100 + 3, 513),
                                 (16, 196607), (16, 196613), (4, 16383), (4, 16387), (7, 16391), (1, 131075)])
def test_rows_at_any_alignment_large(A, n, m, bf16):
    """Both sides of the sizes from which such rows go in vectors: in columns of all row groups 393216 (bfloat16 without a
    partial group 131072, fewer than eight rows 16384 in the encoder), more for narrow rows of float32."""
    torch = torch_mod()
    x = si.make_shape("student_t3", (n, m), 7600 + n % 100)
    run_case(A, x, 3, n, m, t=2, in_bf16=bf16, out_bf16=bf16, tag="ragged large")
    d = A.make_desc(A.MBQ, 4, n, m, in_dtype=A.BF16 if bf16 else A.F32, t=1)
    xd, bits = to_dev(x, bf16)
    xin = orc.widen_bf16(bits) if bf16 else x
    for alpha in ([1.0, 0.52, 0.26, 0.1301], [1.0, 0.99, 0.011, 0.01]):   # levels that share a bucket: two, and more
        a = np.array(alpha, np.float32)
        _, payload = A.accept_compress(d, xd, alpha_prev=torch.from_numpy(a).cuda())
        torch.cuda.synchronize()
        want = orc.mbq_pack(orc.mbq_assign(xin, a), 4, n, m)
        assert first_mismatch(dev_bytes(payload), want.tobytes()) is None, alpha


# Encode kernels of at most 64 workgroups solve for the coefficients themselves, in the workgroup that ends last.
@pytest.mark.parametrize("n,m,bf16,one", [
    (8, 40, False, True),                    # one workgroup, too narrow for wave-items
    (64, 8 * 64 * 4 * 8, False, True),       # 64 workgroups
    (64, 8 * 64 * 4 * 8 + 4, False, False),  # one wave-item more per row group: 65
    (64, 8 * 64 * 8 * 8, True, True),
    (5, 256 * 64 * 4, False, True),          # a partial row group only, four wave-items to a workgroup
    (5, 256 * 64 * 4 + 4, False, False),     # one wave-item more: one to a workgroup
    (13, 4096, True, True),                  # complete and partial
    (13, 4100, True, False),                 # the same in single columns: 65 for the partial one
])
def test_encoder_that_solves_itself(A, n, m, bf16, one):
    torch = torch_mod()
    k = 4 if n != 13 else 3
    d = A.make_desc(A.MBQ, k, n, m, in_dtype=A.BF16 if bf16 else A.F32, t=7)
    assert (A.accept_stage_name(d, 0, 1) is None) == one
    x = si.make_shape("relu_lognormal", (n, m), 900 + n)
    run_case(A, x, k, n, m, t=7, in_bf16=bf16, out_bf16=bf16, tag="solves itself")
    # one workspace, other numbers of workgroups in between, and replays of a captured call: the counters are back at 0
    xd, bits = to_dev(x, bf16)
    alpha, _ = orc.mbq_residue_init(orc.widen_bf16(bits) if bf16 else x.reshape(-1), k)
    ad = torch.from_numpy(np.asarray(alpha, np.float32)).cuda()
    header, payload, ws = A.alloc_outputs(d, "cuda")
    big = A.make_desc(A.MBQ, 2, 64, 40000, t=3)
    xb = torch.randn(64 * 40000, device="cuda")
    A.accept_compress(d, xd, alpha_prev=ad, header=header, payload=payload, workspace=ws)
    torch.cuda.synchronize()
    want = dev_bytes(header), dev_bytes(payload)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        A.accept_compress(d, xd, alpha_prev=ad, header=header, payload=payload, workspace=ws)
    for _ in range(3):
        A.accept_compress(big, xb, alpha_prev=ad[:2].clone(), workspace=ws)
        payload.zero_()
        header.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert (dev_bytes(header), dev_bytes(payload)) == want


# Batch 0 of at most 64 workgroups of 512 items (8 rows, a 16-byte vector or a column): one kernel, the passes in registers.
@pytest.mark.parametrize("n,m,k,bf16", [
    (8, 64, 2, False),              # one workgroup
    (128, 160, 4, False),           # two, the second not full
    (5, 333, 3, True),              # single columns, a partial row group
    (64, 64 * 64 * 4, 3, False),    # 64 workgroups
    (64, 64 * 64 * 4 + 4, 4, False),  # one item more: a kernel for every pass
    (31, 16384, 4, True),
    (40, 6553, 2, False),           # 64 of single columns
])
def test_batch0_in_one_kernel(A, n, m, k, bf16):
    torch = torch_mod()
    x = si.make_shape("relu_lognormal", (n, m), 950 + k)
    xd, bits = to_dev(x, bf16)
    xf = orc.widen_bf16(bits).reshape(n, m) if bf16 else x
    d = A.make_desc(A.MBQ, k, n, m, in_dtype=A.BF16 if bf16 else A.F32)
    header, payload, ws = A.alloc_outputs(d, "cuda")
    oh = np.frombuffer(orc.mbq_compress_first(xf, k, n, m)[0], dtype="<f4")
    seen = set()
    for polls in (64, 0, 1, 64):  # seen by each other; workgroups add up each other's parts
        print("case", n, m, k, bf16, polls, flush=True)
        header.zero_()
        payload.zero_()
        A.accept_compress_polls(d, xd, header, payload, ws, polls)
        torch.cuda.synchronize()
        gh = np.frombuffer(dev_bytes(header), dtype="<f4")
        assert np.all(np.abs(gh.astype(np.float64) - oh) <= 1e-6 * np.abs(oh[:k]).sum()), (gh, oh, polls)
        op = orc.mbq_pack(orc.mbq_residue_signs(xf, gh[:k]), k, n, m)
        assert first_mismatch(dev_bytes(payload), op.tobytes()) is None, polls
        seen.add(gh.tobytes())
    assert len(seen) == 1  # the same bits, whoever added up
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        A.accept_mbq_compress_first(d, xd, header=header, payload=payload, workspace=ws)
    for _ in range(3):
        A.accept_compress(d, xd, alpha_prev=header.view(torch.float32)[:k].clone(), workspace=ws)  # eager, same workspace
        header.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert dev_bytes(header) in seen


@pytest.mark.parametrize("n,m,k,bf16", [(5, 64 * 4 * 2048 + 516, 4, False), (1, 64 * 4 * 2050, 3, False), (3, 64 * 8 * 2048 + 1032, 2, True)])
def test_few_rows_and_more_wave_items_than_wavefronts(A, n, m, k, bf16):
    """A tensor of fewer than eight rows: some wavefronts have a second wave-item, asked for while the first is used."""
    x = si.make_shape("student_t3", (n, m), 970 + n)
    run_case(A, x, k, n, m, t=5, in_bf16=bf16, out_bf16=bf16, tag="few rows")


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("wave_items", [2041, 2048, 2049, 2180, 2304, 2305, 2399, 3840, 3841, 4097])
def test_shares_of_the_work_queue(A, wave_items, bf16):
    """256 workgroups, in 32 groups that take four wave-items each out of a sweep of 128 (2305 to 3840 wave-items: 64 out of 2048): fewer
    wave-items than wavefronts, as many, and last sweeps that not all groups, or not all of a group, have a part of."""
    m = wave_items * 64 * (8 if bf16 else 4)
    x = si.make_shape("relu_normal", (8, m), 9800 + wave_items)
    run_case(A, x, 2, 8, m, in_bf16=bf16, out_bf16=bf16, tag="shares")


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n,m,k", [(9, 512, 2), (15, 4096, 3), (12, 20000, 4), (14, 1000, 5), (12, 520192, 2), (15, 526336, 3),
                                   (15, 200003, 3), (23, 173913, 4), (9, 393217, 1),
                                   (9, 1001, 2), (135, 1001, 3), (143, 1001, 3),
                                   (9, 20008, 6), (9, 1001, 5), (15, 20001, 8)])
def test_partial_row_group_in_the_queue(A, n, m, k, bf16):
    """The partial row group's wave-items are the last of the work queue: one of them, fewer than wavefronts, more; rows at any
    alignment; single columns, in the queue up to 16 complete groups and beside it above.  Levels that lie close (two thresholds
    in a bucket) as well."""
    x = si.make_shape("relu_lognormal", (n, m), 9900 + n + m)
    run_case(A, x, k, n, m, in_bf16=bf16, out_bf16=bf16, tag="partial")
    if k in (3, 4) and not bf16:
        run_case(A, x, k, n, m, alpha_prev=np.array([1.0, 0.5, 0.03, 0.02], np.float32) if k == 4 else
                 np.array([1.0, 0.03, 0.02], np.float32), tag="partial, two thresholds")


# Batch 0 with the tensor in the registers of 256 workgroups: up to one, two, four items per thread; beyond, a kernel for every pass.
@pytest.mark.parametrize("n,m,k,bf16", [
    (8, 4 * 131072, 2, False),       # one item per thread, all of them
    (8, 4 * 131073, 3, False),       # one item more: a chunk of one
    (13, 4 * 50001, 4, False),       # a chunk with lanes of both row groups, a partial row group
    (3, 8 * 100001, 4, True),        # nothing but a partial row group
    (21, 8 * 50000, 2, True),
    (9, 8 * 196608, 3, True),        # four items in some wavefronts
    (8, 4 * 524288, 3, False),       # the largest
    (8, 4 * 524289, 2, False),       # one item more: a kernel for every pass
    (9, 4 * 262147, 3, False), (15, 4 * 262145, 4, False),         # the same, with a partial row group
    (9, 8 * 262147, 2, True), (15, 8 * 262145, 3, True), (12, 8 * 262145, 4, True),
    (300005, 4, 2, False), (300003, 8, 3, True), (70001, 12, 4, False), (52003, 40, 4, True),  # a wavefront's items in many row groups
    (2, 4 * 262144, 3, False), (2, 4 * 262145, 3, False), (3, 4 * 524288, 2, False),                      # few rows: both sides
    (1, 8 * 196608, 2, True), (7, 8 * 196609, 3, True),                                                   # of the lines
    (5, 8 * 65536, 4, True), (5, 8 * 65537, 4, True), (6, 8 * 81920, 2, True), (7, 8 * 81921, 3, True),
])
def test_batch0_held(A, n, m, k, bf16):
    torch = torch_mod()
    x = si.make_shape("relu_lognormal", (n, m), 960 + k)
    xd, bits = to_dev(x, bf16)
    xf = orc.widen_bf16(bits).reshape(n, m) if bf16 else x
    d = A.make_desc(A.MBQ, k, n, m, in_dtype=A.BF16 if bf16 else A.F32)
    header, payload, ws = A.alloc_outputs(d, "cuda")
    oh = np.frombuffer(orc.mbq_compress_first(xf, k, n, m)[0], dtype="<f4")
    want = None
    for polls in (64, 0, 1, 64):  # seen by each other; workgroups add up each other's parts
        print("case", n, m, k, bf16, polls, flush=True)
        header.zero_()
        payload.zero_()
        A.accept_compress_polls(d, xd, header, payload, ws, polls)
        torch.cuda.synchronize()
        gh = np.frombuffer(dev_bytes(header), dtype="<f4")
        assert np.all(np.abs(gh.astype(np.float64) - oh) <= 1e-6 * np.abs(oh[:k]).sum()), (gh, oh, polls)
        got = (gh.tobytes(), dev_bytes(payload))
        if want is None:
            op = orc.mbq_pack(orc.mbq_residue_signs(xf, gh[:k]), k, n, m)
            assert first_mismatch(got[1], op.tobytes()) is None
            want = got
        assert got == want, polls  # the same bits, whoever added up
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        A.accept_mbq_compress_first(d, xd, header=header, payload=payload, workspace=ws)
    for _ in range(3):
        A.accept_compress(d, xd, alpha_prev=header.view(torch.float32)[:k].clone(), workspace=ws)  # eager, same workspace
        header.zero_()
        payload.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert (dev_bytes(header), dev_bytes(payload)) == want


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("bad", [np.nan, -np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("n,m", [(13, 8 * 20001), (9, 8 * 262147)])
def test_batch0_held_values_that_are_not_finite(A, n, m, bad, bf16):
    """Kept in registers; in a kernel for every pass.  A partial row group both times."""
    torch = torch_mod()
    k = 3
    x = si.make_shape("student_t3", (n, m), 970)
    x.reshape(-1)[::53001] = bad
    x.reshape(-1)[::61] = 0.0
    xd = torch.from_numpy(x.reshape(-1)).cuda()
    xd = xd.to(torch.bfloat16) if bf16 else xd
    d = A.make_desc(A.MBQ, k, n, m, in_dtype=A.BF16 if bf16 else A.F32)
    header, payload = A.accept_mbq_compress_first(d, xd)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        oh, op = orc.mbq_compress_first(xd.float().cpu().numpy(), k, n, m)
    gh, ohf = np.frombuffer(dev_bytes(header), dtype="<f4"), np.frombuffer(oh, dtype="<f4")
    assert np.array_equal(np.isnan(gh), np.isnan(ohf)) and np.array_equal(np.isinf(gh), np.isinf(ohf)), (gh, ohf)
    assert first_mismatch(dev_bytes(payload), op.tobytes()) is None


@pytest.mark.parametrize("n,m,k,bf16", [
    (64, 2048, 1, False), (64, 2048, 1, True), (64, 2048, 2, False),   # by comparisons
    (7, 4096, 2, True), (8, 4096, 2, True),                            # by comparisons; through a table
    (24, 255, 3, False), (24, 256, 3, False), (24, 511, 4, True),      # too narrow for wave-items; wide; too narrow
    (3, 100, 4, False), (520, 63, 4, False), (524281, 3, 3, False),    # few rows; 64 workgroups of single columns; more than 64
    (4096, 511, 1, True), (4104, 511, 1, True), (4099, 511, 1, True),  # narrow: two columns for a thread; more, through a table
])
def test_levels_by_comparison_and_through_tables(A, n, m, k, bf16):
    """Values on the thresholds, next to them, zeros of both signs and denormals; coefficients apart, equal, and one that is zero."""
    for alpha in ([1.0, 0.5, 0.25, 0.125], [0.5, 0.5, 0.5, 0.5], [0.75, 0.0, 0.25, 0.125]):
        alpha = np.array(alpha[:k], np.float32)
        _, _, tau = orc.mbq_levels(alpha)
        near = np.concatenate([tau, np.nextafter(tau, np.float32(9)), np.nextafter(tau, np.float32(-9)),
                               np.array([0.0, -0.0, 1e-45, -1e-45], np.float32)]).astype(np.float32)
        x = si.make_shape("relu_normal", (n, m), 9700 + k)
        x.reshape(-1)[: 4 * near.size] = np.tile(near, 4)[: x.size]  # (short tensors: as many as there is room for)
        run_case(A, x, k, n, m, alpha_prev=alpha, in_bf16=bf16, out_bf16=bf16, tag="levels")
