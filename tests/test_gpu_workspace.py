"""What the library keeps in a workspace between calls (its first 16 KiB): numbers of exchanges and mailboxes."""
import numpy as np
import pytest

import synthetic_inputs as si
from oracle import accept_oracle as orc

from gpu_util import dev_bytes, first_mismatch, torch_mod

pytestmark = pytest.mark.gpu

ROUND = 256 * 512 * 32                  # 256 workgroups of 512 groups of 32 elements
FIRST, WORDS = 8192, 8192 + 3 * 2048    # mailboxes; a workgroup's number of exchanges so far: 256 words


@pytest.fixture(scope="module")
def A():
    torch = torch_mod()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2311_05827_amd as pkg
    return pkg


def words(ws):
    return ws[WORDS:WORDS + 1024].view(torch_mod().int32)


class Uniform:
    """A scheme U call of a kernel that exchanges maxima: on one workspace, checked against the oracle."""

    def __init__(self, A, N, k, seed, channels=0, n=1):
        torch = torch_mod()
        self.A, self.d = A, A.make_desc(A.UNIFORM, k, n, N // n, channels=channels)
        x = si.make_shape("grad", (1, N), seed)
        x[0, N - 1 - N // 5] = 0.5
        self.x = torch.from_numpy(x.reshape(-1)).cuda()
        self.want = orc.uniform_compress(x, k, n, N // n, channels)
        self.header, self.payload, _ = A.alloc_outputs(self.d, "cuda")

    def call(self, ws):
        self.A.accept_compress(self.d, self.x, header=self.header, payload=self.payload, workspace=ws)

    def check(self, what=None):
        assert dev_bytes(self.header) == self.want[0], what
        assert first_mismatch(dev_bytes(self.payload), self.want[1].tobytes()) is None, what


class First:
    """A first batch in one kernel, k - 1 exchanges of sums; its result does not depend on who adds up."""

    def __init__(self, A, n, m, k, seed):
        torch = torch_mod()
        self.A, self.d = A, A.make_desc(A.MBQ, k, n, m)
        x = si.make_shape("relu_lognormal", (n, m), seed)
        self.x = torch.from_numpy(x.reshape(-1)).cuda()
        self.header, self.payload, ws = A.alloc_outputs(self.d, "cuda")
        self.call(ws)
        torch.cuda.synchronize()
        oh = np.frombuffer(orc.mbq_compress_first(x, k, n, m)[0], dtype="<f4")
        gh = np.frombuffer(dev_bytes(self.header), dtype="<f4")
        assert np.all(np.abs(gh.astype(np.float64) - oh) <= 1e-6 * np.abs(oh[:k]).sum())
        op = orc.mbq_pack(orc.mbq_residue_signs(x, gh[:k]), k, n, m)
        self.want = dev_bytes(self.header), op.tobytes()

    def call(self, ws):
        self.A.accept_mbq_compress_first(self.d, self.x, header=self.header, payload=self.payload, workspace=ws)

    def check(self, what=None):
        assert (dev_bytes(self.header), dev_bytes(self.payload)) == self.want, what


def test_calls_that_overlapped_spoil_no_later_call(A):
    """Calls that share a workspace must not overlap; where some did (in bounds and ending all the same), their own
    results may be wrong, but later calls' are not, nor do the workgroups' numbers disagree for good."""
    torch = torch_mod()
    on = [[Uniform(A, ROUND, 8, 1), Uniform(A, 600000, 4, 2)], [Uniform(A, 3 * ROUND // 4, 5, 3), First(A, 64, 4096, 4, 4)]]
    ws = A.alloc_outputs(on[1][1].d, "cuda")[2]
    streams = [torch.cuda.Stream() for _ in on]
    torch.cuda.synchronize()
    for _ in range(30):
        for s, calls in zip(streams, on):
            with torch.cuda.stream(s):
                for c in calls:
                    c.call(ws)
    torch.cuda.synchronize()
    assert len(set(words(ws).tolist())) == 1
    for c in on[0] + on[1]:
        c.header.zero_()
        c.payload.zero_()
        c.call(ws)
        torch.cuda.synchronize()
        c.check()


def test_solving_calls_that_overlapped_spoil_no_later_call(A):
    """The same for encoders and first batches whose last workgroup solves, of 1 to 64 workgroups."""
    torch = torch_mod()
    on = [[First(A, n, m, 3, 20 + n) for n, m in ((8, 2000), (64, 16384), (40, 4096))] for _ in range(2)]
    alpha = torch.tensor([1.0, 0.5, 0.25], device="cuda")
    ws = A.alloc_outputs(on[0][0].d, "cuda")[2]
    later = []
    for c in on[0]:
        header, payload = A.accept_compress(c.d, c.x, alpha_prev=alpha)
        torch.cuda.synchronize()
        later.append((dev_bytes(header), dev_bytes(payload)))
    streams = [torch.cuda.Stream() for _ in on]
    for _ in range(30):
        for s, calls in zip(streams, on):
            with torch.cuda.stream(s):
                for c in calls:
                    c.call(ws)
                    A.accept_compress(c.d, c.x, alpha_prev=alpha, header=c.header, payload=c.payload, workspace=ws)
    torch.cuda.synchronize()
    assert ws[:FIRST].view(torch.int32).view(32, 64)[:, 0].tolist() == [0] * 32   # work counters
    assert int(ws[8:12].view(torch.int32)[0]) % 64 == 0
    for c, want in zip(on[0], later):
        c.header.zero_()
        c.payload.zero_()
        c.call(ws)
        torch.cuda.synchronize()
        c.check()
        header, payload = A.accept_compress(c.d, c.x, alpha_prev=alpha, workspace=ws)
        torch.cuda.synchronize()
        assert (dev_bytes(header), dev_bytes(payload)) == want


def test_numbers_of_exchanges_wrap(A):
    """The number has 32 bits.  Boxes of workgroups that only a call before the wrap had, or none at all (0), are not
    taken for the wrapped call's; on the way there, at multiples of 2^30, every box is renumbered."""
    torch = torch_mod()
    small, large = Uniform(A, 2 * 512 * 32, 8, 11), Uniform(A, ROUND, 8, 12)     # 2 and 256 workgroups
    channels, first = Uniform(A, 64 * 6 * 3136, 6, 13, channels=6, n=64), First(A, 64, 4096, 4, 14)
    ws = A.alloc_outputs(first.d, "cuda")[2]
    boxes = [ws[FIRST:WORDS].view(torch.int64)]
    boxes += [ws[64:FIRST].view(torch.int64).as_strided((32, 24), (32, 1))]       # between the counters

    def number(t):
        return (t >> 32) & 0xFFFFFFFF

    for quarter in range(1, 5):  # the first call of a turn goes past the multiple; the one that has number 0 is a large one
        words(ws).fill_((quarter << 30) - 1 - ((1 << 32) if quarter > 2 else 0))
        for c in (large, channels, first, small) if quarter == 4 else (small, first) if quarter == 2 else (small,):
            c.header.zero_()
            c.payload.zero_()
            c.call(ws)
            torch.cuda.synchronize()
            c.check(quarter)
        now = int(words(ws)[0]) & 0xFFFFFFFF
        assert now < 8 if quarter == 4 else now >= quarter << 30
        for b in boxes:
            assert int(((now - number(b)) & 0xFFFFFFFF).max()) <= 8, quarter
