"""The binding's calls on real device tensors: what the native path takes and what it hands back to the checks
written in Python gives the same results and the same refusals."""
import pytest

import synthetic_inputs as si
from oracle import accept_oracle as orc

from gpu_util import dev_bytes, torch_mod

pytestmark = pytest.mark.gpu

N, M, K = 4, 1024, 5


@pytest.fixture(scope="module")
def A():
    torch = torch_mod()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2311_05827_amd as pkg
    return pkg


@pytest.mark.parametrize("kind", ["plain", "parameter", "subclass", "requires_grad", "other_stream"])
def test_every_tensor_the_binding_takes(A, kind):
    torch = torch_mod()

    class Tagged(torch.Tensor):
        pass

    x = si.make_shape("grad", (N, M), 5)
    xd = torch.from_numpy(x.reshape(-1)).cuda()
    if kind == "parameter":
        xd = torch.nn.Parameter(xd)
    if kind == "subclass":
        xd = xd.as_subclass(Tagged)
    if kind == "requires_grad":
        xd.requires_grad_(True)
    d = A.make_desc(A.UNIFORM, K, N, M)
    stream = torch.cuda.Stream() if kind == "other_stream" else torch.cuda.current_stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        if kind == "other_stream":  # x is replaced on that stream just before: a call on another one would miss it
            xd = torch.zeros_like(xd)
            xd.copy_(torch.from_numpy(x.reshape(-1)).cuda(), non_blocking=True)
        header, payload = A.accept_compress(d, xd)
        out = A.accept_decompress(d, header, payload)
    torch.cuda.synchronize()
    oh, op = orc.uniform_compress(x, K, N, M)
    assert dev_bytes(header) == oh and dev_bytes(payload) == op.tobytes()
    assert out.dtype == torch.float32 and dev_bytes(out) == orc.uniform_decompress(oh, op, K, N, M).tobytes()


@pytest.mark.parametrize("scheme", ["UNIFORM", "MBQ"])
def test_every_tensor_the_binding_refuses(A, scheme):
    torch = torch_mod()
    d = A.make_desc(getattr(A, scheme), 4, N, M)
    x = torch.zeros(N * M, device="cuda")
    alpha = torch.ones(4, device="cuda")
    header, payload, ws = A.alloc_outputs(d, "cuda")
    good = dict(x=x, alpha_prev=alpha, header=header, payload=payload, workspace=ws)
    bad = [("x", x.cpu()), ("x", x[:-1]), ("x", x.view(2, -1).t()), ("x", x.to(torch.bfloat16)),
           ("header", header[:-1]), ("payload", payload[:-1]), ("workspace", ws[:-1]), ("header", header.cpu())]
    if scheme == "MBQ":
        bad += [("alpha_prev", alpha[:3]), ("alpha_prev", None), ("alpha_prev", alpha.double())]
    for name, t in bad:
        with pytest.raises((A.AcceptError, TypeError)):
            A.accept_compress(d, **dict(good, **{name: t}))
    A.accept_compress(d, **good)
    with pytest.raises(A.AcceptError):  # misaligned: the library's own check
        A.accept_compress(d, **dict(good, payload=torch.empty(payload.numel() + 4, dtype=torch.uint8, device="cuda")[4:]))
    out = torch.empty(N * M, device="cuda")
    for h, p, o in ((header[:-1], payload, out), (header, payload[:-1], out), (header, payload, out[:-1]),
                    (header, payload, out.to(torch.bfloat16)), (header, payload, out.cpu())):
        with pytest.raises(A.AcceptError):
            A.accept_decompress(d, h, p, out=o)
    A.accept_decompress(d, header, payload, out=out)
    torch.cuda.synchronize()


def test_other_objects_than_a_descriptor_are_refused(A):
    """64 bytes that happen to describe the call are not a descriptor; a subclass of it is."""
    import ctypes
    torch = torch_mod()

    class Words(ctypes.Structure):
        _fields_ = [("words", ctypes.c_int64 * 8)]

    class Mine(A.Desc):
        pass

    x = torch.from_numpy(si.make_shape("grad", (N, M), 6).reshape(-1)).cuda()
    out = torch.empty(N * M, device="cuda")
    for scheme in (A.UNIFORM, A.MBQ):
        d = A.make_desc(scheme, 4, N, M)
        alpha = torch.ones(4, device="cuda")
        header, payload, ws = A.alloc_outputs(d, "cuda")
        want = [dev_bytes(t) for t in A.accept_compress(d, x, alpha_prev=alpha, header=header, payload=payload, workspace=ws)]
        values = dev_bytes(A.accept_decompress(d, header, payload, out=out))
        header.zero_()
        payload.zero_()
        for other in (bytes(d), bytearray(bytes(d)), memoryview(bytes(d)), Words.from_buffer_copy(bytes(d))):
            with pytest.raises((AttributeError, TypeError, ctypes.ArgumentError)):
                A.accept_compress(other, x, alpha_prev=alpha, header=header, payload=payload, workspace=ws)
            with pytest.raises((AttributeError, TypeError, ctypes.ArgumentError)):
                A.accept_decompress(other, header, payload, out=out)
            if scheme == A.MBQ:
                with pytest.raises((AttributeError, TypeError, ctypes.ArgumentError)):
                    A.accept_mbq_compress_first(other, x, header=header, payload=payload, workspace=ws)
        torch.cuda.synchronize()
        assert not header.any() and not payload.any()
        mine = Mine.from_buffer_copy(bytes(d))
        got = [dev_bytes(t) for t in A.accept_compress(mine, x, alpha_prev=alpha, header=header, payload=payload, workspace=ws)]
        assert got == want and dev_bytes(A.accept_decompress(mine, header, payload, out=out)) == values


def test_decompress_makes_its_output(A):
    """Without `out`, the tensor comes from the native call, on the payload's device and of the descriptor's type; what is wrong is
    refused as with one."""
    torch = torch_mod()
    for code, dtype in ((A.F32, torch.float32), (A.BF16, torch.bfloat16)):
        x = torch.randn(24 * 333, device="cuda").to(dtype)
        d = A.make_desc(A.UNIFORM, 6, 24, 333, in_dtype=code, out_dtype=code)
        header, payload = A.accept_compress(d, x)
        want = A.accept_decompress(d, header, payload, out=torch.empty_like(x))
        got = A.accept_decompress(d, header, payload)
        assert got.dtype is dtype and got.device == payload.device and not got.requires_grad
        assert torch.equal(got.view(torch.uint8), want.view(torch.uint8))
        with pytest.raises(A.AcceptError):
            A.accept_decompress(d, header, payload[:-1].clone())
        with pytest.raises(A.AcceptError):
            A.accept_decompress(A.make_desc(A.UNIFORM, 1, 24, 333), header, payload)
