"""Workloads of the boundary compressor: the calls a pipeline stage makes for one tensor.

A stage sends features forward (scheme M: sign bits against k coefficients; 2, 3 or 4 bits as
training goes on) and gradients backward (scheme U: 8 bits, then 4, stochastic rounding by
default; any width 2..8, one range per tensor or per channel), and receives both.  Sizes run from
the paper's smallest boundary tensor (20,480 values and below) to a ResNet-50 stage output at
batch 64 (51.4 M values), in float32 and bfloat16, with aligned and ragged shapes.

ops
  feature_send     accept_compress, scheme M, with the previous batch's coefficients
  feature_first    accept_mbq_compress_first: batch 0 of an epoch
  feature_receive  accept_decompress, scheme M
  feature_trip     feature_send, then feature_receive of what it sent
  grad_send        accept_compress, scheme U
  grad_receive     accept_decompress, scheme U
  grad_trip        grad_send, then grad_receive of what it sent
  batch            boundary.boundary(): forward and backward of one batch through autograd

Buffers and workspaces are made once, as a training loop or a server keeps them.
"""
import math

import numpy as np
import torch

import paper_2311_05827_amd as A

DEVICE = "cuda"


# ---------------------------------------------------------------------------------- the cases
def _case(name, op, n, m, bits, values, dtype="f32", channels=0, rounding="nearest"):
    return {"name": name, "op": op, "n": n, "m": m, "bits": bits, "channels": channels, "dtype": dtype,
            "rounding": rounding, "values": values}


def listed():
    return [
        # One batch over the paper's smallest MobileNetV2 boundary (batch 128, 80 KB) through the
        # training glue, both directions: launches and host time are all there is.
        _case("batch_smallest", "batch", 128, 160, 2, "relu"),
        # A CNN activation of 262,144 values at batch 4 (fewer rows than a plane byte holds).
        _case("feature_small", "feature_trip", 4, 65536, 2, "relu"),
        # First batch of an epoch at a VGG-16 stage (32x128x56x56), middle bit width.
        _case("feature_vgg_first", "feature_first", 32, 401408, 3, "relu_lognormal"),
        # Steady state of training at a ResNet-50 stage boundary (64x256x56x56), float32.
        _case("feature_resnet_send", "feature_send", 64, 802816, 4, "relu_lognormal"),
        _case("feature_resnet_receive", "feature_receive", 64, 802816, 4, "relu_lognormal"),
        # The same boundary under mixed precision.
        _case("feature_resnet_send_bf16", "feature_send", 64, 802816, 4, "relu_lognormal", dtype="bf16"),
        # A last, incomplete batch of hidden states with an odd width: no row is aligned.
        _case("feature_ragged", "feature_trip", 15, 509 * 767, 3, "student_t"),
        # Gradients of the ResNet-50 boundary, early training (8 bits), reproducible streams.
        _case("grad_resnet_send", "grad_send", 64, 802816, 8, "grad"),
        _case("grad_resnet_receive", "grad_receive", 64, 802816, 8, "grad"),
        # The same after the learning rate changed: 4 bits, the paper's stochastic rounding.
        _case("grad_resnet_send_stochastic", "grad_send", 64, 802816, 4, "grad", rounding="stochastic"),
        # Mixed-precision activation with one range per channel.
        _case("channels_resnet_bf16", "grad_trip", 64, 802816, 6, "relu_lognormal", dtype="bf16", channels=256),
        # Transformer hidden states, a width whose codes straddle bytes and words.
        _case("hidden_straddling", "grad_trip", 16, 509 * 768, 5, "student_t"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["feature_send", "feature_send", "feature_receive", "feature_receive", "feature_trip",
                     "feature_first", "grad_send", "grad_send", "grad_receive", "grad_receive", "grad_trip", "batch"])
    dtype = "f32" if op in ("batch", "feature_trip") else rng.choice(["f32", "f32", "bf16"])
    feature = op.startswith("feature") or op == "batch"
    bits = 2 if op == "batch" else rng.choice([2, 3, 4]) if feature else rng.choice([2, 3, 4, 4, 5, 6, 7, 8, 8])
    values = rng.choice(["relu", "relu_lognormal", "student_t"] if feature else ["grad", "grad", "grad_outliers", "student_t"])
    rounding = "nearest" if feature else rng.choice(["nearest", "nearest", "stochastic"])
    # round trips, first batches and whole batches move the data several times: smaller tensors
    largest = {"feature_first": 12845056, "feature_trip": 12845056, "grad_trip": 25690112, "batch": 6254592}.get(op, 51380224)
    if op == "grad_send" and rounding == "stochastic":
        largest = 25690112
    channels = 0
    geometry = rng.choice(["rows", "rows", "odd", "channels", "channels_last"] if not feature else ["rows", "rows", "odd"])
    if geometry == "odd":            # rows that no 16-byte vector divides
        total = _log_uniform(rng, 6400, min(largest, 6254592))
        n = _log_uniform(rng, 1, 130)
        m = max(3, total // n) | 1
    elif geometry == "channels":     # n x C x h x w, one range per channel
        total = _log_uniform(rng, 65536, min(largest, 25690112))
        hw = rng.choice([49, 64, 196, 256, 784, 1024, 3136, 12544])
        if hw == 49:
            total = min(total, 6422528)
        n = max(1, min(_log_uniform(rng, 1, 130), total // (2 * hw)))
        channels = max(2, total // (n * hw))
        m = channels * hw
    elif geometry == "channels_last":
        total = _log_uniform(rng, 65536, min(largest, 25690112))
        channels = 8 * _log_uniform(rng, 4, 256)
        n, m = max(1, total // channels), channels
    else:
        total = _log_uniform(rng, 6400, largest)
        n = _log_uniform(rng, 1, 130)
        if rng.random() < 0.6:
            n = min(128, (n + 7) // 8 * 8)
        m = max(8, total // n // 8 * 8)
    c = _case("", op, n, m, bits, values, dtype, channels, rounding)
    del c["name"]
    return c


# ----------------------------------------------------------------------- inputs, from the seed
def _values(kind, count, gen):
    z = torch.randn(count, device=DEVICE, generator=gen)
    if kind == "relu":
        return z.clamp_(min=0)
    if kind == "relu_lognormal":
        keep = torch.rand(count, device=DEVICE, generator=gen) >= 0.6
        return torch.exp(z - 1.0) * keep
    if kind == "grad":
        return z * 1e-3
    if kind == "grad_outliers":
        out = torch.rand(count, device=DEVICE, generator=gen) < 1e-3
        return torch.where(out, z * 1e-1, z * 1e-3)
    if kind == "student_t":
        chi = torch.zeros(count, device=DEVICE)
        for _ in range(3):
            chi += torch.randn(count, device=DEVICE, generator=gen) ** 2
        return z / torch.sqrt(chi / 3.0)
    raise ValueError(kind)


def _input(case, seed):
    """The tensor, flat; per channel with a gain of its own for every channel."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    x = _values(case["values"], case["n"] * case["m"], gen)
    if case["channels"] > 1:
        gain = torch.exp(0.5 * torch.randn(case["channels"], device=DEVICE, generator=gen))
        x = (x.view(case["n"], case["channels"], -1) * gain[None, :, None]).reshape(-1)
    return x.to(torch.bfloat16) if case["dtype"] == "bf16" else x


def _coefficients(x, bits):
    """Coefficients of a batch like x, as the previous batch leaves them (residue method)."""
    rho = x[: 1 << 22].double()
    alpha = []
    for _ in range(bits):
        a = float(rho.abs().mean())
        alpha.append(round(a * (1 << 20)) / (1 << 20))
        rho = rho - torch.where(rho >= 0, alpha[-1], -alpha[-1])
    return torch.tensor(alpha, dtype=torch.float32, device=DEVICE)


def _rounding_seed(seed):
    return 1000003 * (int(seed) % (1 << 20)) + 17


def _desc(case, seed):
    code = A.BF16 if case["dtype"] == "bf16" else A.F32
    if case["op"].startswith("feature"):
        return A.make_desc(A.MBQ, case["bits"], case["n"], case["m"], in_dtype=code, out_dtype=code, t=20)
    return A.make_desc(A.UNIFORM, case["bits"], case["n"], case["m"], channels=case["channels"], in_dtype=code,
                       out_dtype=code, seed=_rounding_seed(seed),
                       rounding=A.ROUND_STOCHASTIC if case["rounding"] == "stochastic" else A.ROUND_NEAREST_EVEN)


def prepare(case, seed):
    x = _input(case, seed)
    op, n, m = case["op"], case["n"], case["m"]
    if op == "batch":
        gen = torch.Generator(device=DEVICE)
        gen.manual_seed(int(seed) + 1)
        return {"op": op, "x": x.view(n, m).requires_grad_(True), "grad": _values("grad", n * m, gen).view(n, m),
                "forward": A.boundary.ForwardCompressor(n, m),
                "backward": A.boundary.BackwardCompressor(n, m, seed=_rounding_seed(seed))}
    desc = _desc(case, seed)
    header, payload, workspace = A.alloc_outputs(desc, DEVICE)
    state = {"op": op, "desc": desc, "header": header, "payload": payload}
    if op.endswith(("send", "trip", "first")):
        state.update(x=x, workspace=workspace)
        if op in ("feature_send", "feature_trip"):
            state["alpha"] = _coefficients(x, case["bits"])
    if op.endswith(("receive", "trip")):
        state["out"] = torch.empty(n * m, dtype=x.dtype, device=DEVICE)
    if op == "feature_receive":   # what the sender's call left in the two buffers
        alpha = _coefficients(x, case["bits"])
        state["header"] = torch.cat([alpha, alpha[-1:] * 0.125]).view(torch.uint8)
        payload.copy_(_pack_planes(_patterns(x, alpha), n, m, case["bits"]))
    if op == "grad_receive":
        s, r = _scales(x, case)
        state["header"] = s.view(torch.uint8)
        payload.copy_(_pack_stream(_codes(x, r, case, seed), case["bits"]))
    return state


# -------------------------------------------------------------------------------- one pass
def run(s):
    op = s["op"]
    if op == "batch":
        s["forward"].start_epoch()
        y = A.boundary.boundary(s["x"], s["forward"], s["backward"])
        (g,) = torch.autograd.grad(y, s["x"], s["grad"])
        return {"y": y.detach(), "grad": g}
    d, got = s["desc"], {}
    if op == "feature_first":
        A.accept_mbq_compress_first(d, s["x"], header=s["header"], payload=s["payload"], workspace=s["workspace"])
    elif "x" in s:
        A.accept_compress(d, s["x"], alpha_prev=s.get("alpha"), header=s["header"], payload=s["payload"],
                          workspace=s["workspace"])
    if "x" in s:
        got.update(header=s["header"].view(torch.float32), payload=s["payload"])
    if "out" in s:
        got["values"] = A.accept_decompress(d, s["header"], s["payload"], out=s["out"])
    return got


def _sizes(case):
    """(bytes of the tensor, of header and payload)."""
    n, m, k = case["n"], case["m"], case["bits"]
    tensor = n * m * (2 if case["dtype"] == "bf16" else 4)
    if case["op"].startswith("feature"):
        return tensor, 4 * (k + 1) + (n + 7) // 8 * m * k
    return tensor, 4 * max(1, case["channels"]) + (n * m * k + 7) // 8


def work(case):
    """Every input read once, every output written once; a multiply and a rounding per value and
    scheme U call, a multiply-add per bit and value for scheme M's sums."""
    tensor, packed = _sizes(case)
    count = case["n"] * case["m"]
    if case["op"] == "batch":   # features in and out, gradients in and out
        return {"bytes": 4 * tensor, "flops": (2 * case["bits"] + 4) * count}
    tensors = 2 if case["op"].endswith("trip") else 1
    return {"bytes": tensors * tensor + packed, "flops": tensors * count * (2 * case["bits"] if case["op"].startswith("feature") else 2)}


def tolerance(case):
    """Scheme U and every payload: the same bits.  Scheme M's header is a least-squares solution of
    64-bit sums rounded to float32 once: a sum in another order moves it by one unit in the last
    place at most (6e-8), and the values decoded from it by as much."""
    if case["op"] in ("feature_send", "feature_first", "feature_trip", "batch"):
        return {"rel": 2.5e-7, "max": 1e-6, "differ": 0.0}
    return "exact"


# ------------------------------------------- the definition, in plain torch (64-bit where it rounds)
def _levels(alpha):
    """(patterns in the order of their levels, thresholds): float32 by definition."""
    alpha = alpha.cpu().numpy().astype(np.float32)
    k = alpha.size
    level = np.zeros(1 << k, dtype=np.float32)
    for j in range(k):
        level = (level + np.where((np.arange(1 << k) >> j) & 1, alpha[j], -alpha[j]).astype(np.float32)).astype(np.float32)
    order = np.lexsort((np.arange(1 << k), level))
    level = level[order]
    return order, (np.float32(0.5) * (level[:-1] + level[1:])).astype(np.float32)


def _patterns(x, alpha):
    order, tau = _levels(alpha)
    x = x.float()
    at = torch.zeros(x.numel(), dtype=torch.uint8, device=x.device)
    for t in tau:
        at += x > float(t)
    return torch.from_numpy(order.astype(np.uint8)).to(x.device)[at.long()]


def _signs_first(x, bits):
    """Residue method: (coefficients rounded to float32, patterns)."""
    rho = x.double()
    alpha, pattern = [], torch.zeros(x.numel(), dtype=torch.uint8, device=x.device)
    for j in range(bits):
        a = float(np.float32(float(rho.abs().mean())))
        up = rho >= 0
        pattern |= up.to(torch.uint8) << j
        rho = rho - torch.where(up, a, -a)
        alpha.append(a)
    return torch.tensor(alpha, dtype=torch.float64, device=x.device), pattern


def _solve(x, pattern, alpha, t):
    """alpha_t in 64 bits: least squares, then the moving average."""
    k, count = alpha.numel(), x.numel()
    x = x.double()
    g, h = torch.zeros(k, k, dtype=torch.float64), torch.zeros(k, dtype=torch.float64)
    for p in range(k):
        bp = (pattern >> p) & 1
        h[p] = 2 * float(x[bp.bool()].sum()) - float(x.sum())
        for q in range(k):
            g[p, q] = count - 2 * int((bp ^ ((pattern >> q) & 1)).sum())
    prev = alpha.cpu().double()
    beta = min(0.9, (1 + t) / (10 + t))
    return (beta * prev + (1 - beta) * torch.linalg.solve(g, h)).to(x.device)


def _mean_error(x, pattern, alpha):
    """mean(B alpha - x), with alpha as it is sent: float32."""
    total = -float(x.double().sum())
    for p in range(alpha.numel()):
        total += float(alpha[p].float()) * (2 * int(((pattern >> p) & 1).sum()) - x.numel())
    return total / x.numel()


def _decoded(pattern, alpha, error):
    k = alpha.numel()
    bit = (torch.arange(1 << k, device=pattern.device)[:, None] >> torch.arange(k, device=pattern.device)) & 1
    return ((2 * bit - 1).double() @ alpha.double() - error)[pattern.long()]


def _pack_planes(pattern, n, m, bits):
    groups = (n + 7) // 8
    rows = torch.zeros(groups * 8, m, dtype=torch.uint8, device=pattern.device)
    rows[:n] = pattern.view(n, m)
    rows = rows.view(groups, 8, m)
    out = torch.zeros(groups, m, bits, dtype=torch.uint8, device=pattern.device)
    for p in range(bits):
        for i in range(8):
            out[:, :, p] |= ((rows[:, i] >> p) & 1) << (7 - i)
    return out.view(-1)


def _per_value(v, case):
    if v.numel() == 1:
        return v
    return v[None, :, None].expand(case["n"], v.numel(), case["m"] // v.numel()).reshape(-1)


def _scales(x, case):
    """Scale and reciprocal of every range group, float32 by definition."""
    c = x.float().abs().view(case["n"], max(1, case["channels"]), -1).amax(dim=(0, 2))
    top = float((1 << (case["bits"] - 1)) - 1)
    return c / top, torch.where(c > 0, torch.full_like(c, top) / c, torch.zeros_like(c))


def _uniform(seed, count):
    """Top 24 bits of splitmix64's output function at seed + (i + 1) * golden ratio."""
    def shift(z, b):
        return (z >> b) & ((1 << (64 - b)) - 1)

    def signed(v):
        return v - (1 << 64) if v >> 63 else v
    z = torch.arange(1, count + 1, dtype=torch.int64, device=DEVICE) * signed(0x9E3779B97F4A7C15) + int(seed)
    z = (z ^ shift(z, 30)) * signed(0xBF58476D1CE4E5B9)
    z = (z ^ shift(z, 27)) * signed(0x94D049BB133111EB)
    return shift(z ^ shift(z, 31), 40).float() * 2.0 ** -24


def _codes(x, r, case, seed, rounding_seed=None):
    v = x.float() * _per_value(r, case)
    if case["rounding"] == "nearest":
        return torch.round(v).to(torch.int16)
    low = torch.floor(v)
    u = _uniform(_rounding_seed(seed) if rounding_seed is None else rounding_seed, x.numel())
    half = 1 << (case["bits"] - 1)
    return (low + (u < v - low)).clamp_(-half, half - 1).to(torch.int16)


def _pack_stream(q, bits):
    """Codes as a dense stream, most significant bit first, in eights: 8 codes are `bits` bytes."""
    u = (q if bits == 8 else q + (1 << (bits - 1))).long() & ((1 << bits) - 1)
    count = u.numel()
    u = torch.nn.functional.pad(u, (0, -count % 8)).view(-1, 8)
    word = torch.zeros(u.shape[0], dtype=torch.int64, device=u.device)
    for i in range(8):
        word |= u[:, i] << (bits * (7 - i))
    out = torch.stack([(word >> (8 * (bits - 1 - b))) & 0xFF for b in range(bits)], dim=1).to(torch.uint8)
    return out.view(-1)[: (count * bits + 7) // 8]


def exact(case, seed):
    x, op, n, m, bits = _input(case, seed), case["op"], case["n"], case["m"], case["bits"]
    if op == "batch":
        alpha, pattern = _signs_first(x, bits)
        y = _decoded(pattern, alpha, _mean_error(x, pattern, alpha))
        gen = torch.Generator(device=DEVICE)
        gen.manual_seed(int(seed) + 1)
        g = _values("grad", n * m, gen)
        back = dict(case, bits=8, rounding="stochastic")
        s, r = _scales(g, back)
        return {"y": y.view(n, m), "grad": (_codes(g, r, back, seed).double() * s.double()).view(n, m)}
    if op.startswith("feature"):
        if op == "feature_first":
            alpha, pattern = _signs_first(x, bits)
        else:
            alpha = _coefficients(x, bits)
            pattern = _patterns(x, alpha)
        if op == "feature_receive":
            return {"values": _decoded(pattern, alpha, float(alpha[-1]) * 0.125)}
        if op != "feature_first":
            alpha = _solve(x, pattern, alpha, 20)
        error = _mean_error(x, pattern, alpha)
        got = {"header": torch.cat([alpha, torch.tensor([error], dtype=torch.float64, device=DEVICE)]), "payload": None}
        if op == "feature_trip":
            got["values"] = _decoded(pattern, alpha, error)
        return got
    s, r = _scales(x, case)
    got = {}
    if op != "grad_receive":
        top = float((1 << (bits - 1)) - 1)
        c = x.double().abs().view(n, max(1, case["channels"]), -1).amax(dim=(0, 2))
        got.update(header=c / top, payload=None)
    if op != "grad_send":
        got["values"] = _codes(x, r, case, seed).double() * _per_value(s.double(), case)
    return got
