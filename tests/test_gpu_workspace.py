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

    def call(self, ws, polls=64):
        self.A.accept_compress_polls(self.d, self.x, self.header, self.payload, ws, polls)

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

    def call(self, ws, polls=64):
        self.A.accept_compress_polls(self.d, self.x, self.header, self.payload, ws, polls)

    def check(self, what=None):
        assert (dev_bytes(self.header), dev_bytes(self.payload)) == self.want, what


class Encode:
    """A batch that is not the first; encoders of few workgroups count these, all draw from work counters."""

    def __init__(self, A, n, m, k, seed):
        torch = torch_mod()
        self.A, self.d = A, A.make_desc(A.MBQ, k, n, m, t=5)
        x = si.make_shape("relu_lognormal", (n, m), seed)
        self.x = torch.from_numpy(x.reshape(-1)).cuda()
        self.alpha = torch.tensor([1.0, 0.5, 0.25, 0.125][:k], device="cuda")
        self.header, self.payload, ws = A.alloc_outputs(self.d, "cuda")
        self.call(ws)
        torch.cuda.synchronize()
        self.planes = orc.mbq_pack(orc.mbq_assign(x, self.alpha.cpu().numpy()), k, n, m).tobytes()
        self.coefficients = np.frombuffer(dev_bytes(self.header), dtype="<f4").astype(np.float64)

    def call(self, ws, polls=64):
        self.A.accept_compress(self.d, self.x, alpha_prev=self.alpha, header=self.header, payload=self.payload, workspace=ws)

    def check(self, what=None):
        got = np.frombuffer(dev_bytes(self.header), dtype="<f4").astype(np.float64)
        # which wavefront takes which part decides how the float64 sums are grouped
        assert np.all(np.abs(got - self.coefficients) <= 1e-6 * np.abs(self.coefficients[:-1]).sum()), what
        assert first_mismatch(dev_bytes(self.payload), self.planes) is None, what


def test_all_kinds_of_calls_on_one_workspace(A):
    """Every kernel that exchanges or counts something, with many and few workgroups, one after the other in any order;
    some look in vain and make up for the others."""
    torch = torch_mod()
    rng = np.random.default_rng(31)
    calls = [Uniform(A, 2 * 512 * 32 + 5, 3, 30), Uniform(A, ROUND, 8, 31), Uniform(A, 40 * 512 * 32, 4, 32),
             Uniform(A, 3 * ROUND + 16384 + 3, 8, 33), Uniform(A, 9 * ROUND + 9, 4, 34),
             Uniform(A, 64 * 6 * 3136, 6, 35, channels=6, n=64), Uniform(A, 3 * 7 * 1568, 5, 36, channels=7, n=3),
             Uniform(A, 2 * 2 * 2000000, 8, 37, channels=2, n=2),
             First(A, 64, 16384, 4, 38), First(A, 128, 160, 2, 39), First(A, 40, 6000, 3, 40),
             Encode(A, 4, 65536, 2, 41), Encode(A, 64, 100000, 4, 42)]
    ws = torch.zeros(max(A.accept_workspace_size(c.d) for c in calls), dtype=torch.uint8, device="cuda")
    order = np.concatenate([rng.permutation(len(calls)) for _ in range(6)])
    for step, i in enumerate(order):
        c, polls = calls[i], int(rng.choice([64, 64, 0, 1, 3]))
        c.header.zero_()
        c.payload.zero_()
        c.call(ws, polls)
        torch.cuda.synchronize()
        c.check((step, int(i), polls))
        assert len(set(words(ws).tolist())) == 1, (step, int(i))


@pytest.mark.parametrize("kind", ["whole", "whole, many", "first", "encode"])
def test_small_calls_on_two_streams_and_in_a_graph(A, kind):
    """Calls of two streams, each with its own workspace, run side by side; a captured call is replayed between eager ones."""
    torch = torch_mod()
    make = {"whole": lambda i: Uniform(A, (3 + i) * 512 * 32 + 7, 5, 50 + i), "whole, many": lambda i: Uniform(A, ROUND - i * 9999, 8, 52 + i),
            "first": lambda i: First(A, 64, 16384 - 4 * i, 4, 54 + i), "encode": lambda i: Encode(A, 8, 60000 + 8 * i, 3, 56 + i)}[kind]
    on = [make(0), make(1)]
    spaces = [A.alloc_outputs(c.d, "cuda")[2] for c in on]
    streams = [torch.cuda.Stream() for _ in on]
    torch.cuda.synchronize()
    for turn in range(8):
        for _ in range(12):
            for c, ws, s in zip(on, spaces, streams):
                with torch.cuda.stream(s):
                    c.call(ws, 64 if turn % 2 == 0 else 2)
        torch.cuda.synchronize()
        for c in on:
            c.check((kind, turn))
            c.header.zero_()
            c.payload.zero_()
        torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        on[0].call(spaces[0])
    for turn in range(4):
        on[0].header.zero_()
        on[0].payload.zero_()
        g.replay()
        torch.cuda.synchronize()
        on[0].check((kind, "replay", turn))
        on[1].call(spaces[0])  # another call on the same workspace
        torch.cuda.synchronize()
        on[1].check((kind, "between", turn))


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
