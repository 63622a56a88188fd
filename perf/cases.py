"""The work that a user of the codec has it do, as measurable cases.

Six kinds of pass, each through the public binding (`paper_1811_03617_amd.gvq`):

  step     one compressed aggregation of a training iteration (Eqs. 2-4): every worker's gradient is
           compressed, the compressed vectors are summed, the sum is decompressed;
  ring     what ONE node does in Algorithm 1: its gradient compressed segment by segment, each segment after
           the first added to the partial sum that came in, then every segment of the result decompressed;
  refresh  the basis refresh over pooled slices, its status, and the new basis as the host keeps it for a
           checkpoint or for the other nodes;
  sample   the same with the paper's own sampling: the first slice of every block only (Section 3);
  monitor  Eq. 6, the local compression loss a node watches to decide when to refresh;
  pack     a model's layers flattened into the gradient vector and unflattened out of it (Fig. 2a).

Slices follow the planted model of the repository's workloads: scale * (A z + sigma * eps) plus a small mean, one A
per basis.  The codec cases run on a restored basis (orthonormal, spanning the planted directions), as a program that
resumes from a checkpoint has it.
"""
import math

import torch

from paper_1811_03617_amd import gvq

DEV = "cuda:0"

# (filters, depth, height, width) of the layers behind the vgg16 workload's 138,357,544 numbers: thirteen 3 x 3
# convolutions and three fully connected layers, each with its bias
_VGG16 = ",".join(
    [f"{f}x{d}x3x3,{f}x1x1x1" for d, f in (
        (3, 64), (64, 64), (64, 128), (128, 128), (128, 256), (256, 256), (256, 256), (256, 512), (512, 512),
        (512, 512), (512, 512), (512, 512), (512, 512))]
    + ["4096x25088x1x1,4096x1x1x1,4096x4096x1x1,4096x1x1x1,1000x4096x1x1,1000x1x1x1"])


def _codec(name, kind, M, d, k, N, dtype="f32", block=0, scales=0, sigma=0.05, L=0):
    c = {"kind": kind, "M": M, "d": d, "k": k, "N": N, "dtype": dtype, "block": block, "scales": scales,
         "sigma": sigma, "L": L}
    return dict(c, name=name) if name else c


def listed():
    return [
        # A small network's gradient: everything stays in the caches, six launches of a few microseconds.
        _codec("step_tiny", "step", 460_800, 16, 4, 4),
        # An ordinary network, short slices, layers of very different magnitude, ragged tail.
        _codec("step_resnet50", "step", 25_557_032, 32, 8, 8, scales=64, sigma=0.1),
        # The headline workload.
        _codec("step_vgg16", "step", 138_357_544, 128, 32, 16),
        # bf16 storage, one basis per 1M-element block: 139 bases in one launch.
        _codec("step_vgg16_bf16", "step", 138_357_544, 128, 16, 16, dtype="bf16", block=1_000_000),
        # The paper's example slice size at its average compression of 8.
        _codec("step_conv768", "step", 138_357_544, 768, 96, 8),
        # Slice length and comps that are no powers of two (100 elements, 25 comps), fewer workers.
        _codec("step_ragged", "step", 61_100_840, 100, 25, 4, sigma=0.1),
        # One node of a ring of eight: small launches, fused adds, results decompressed as they arrive.
        _codec("ring_alexnet", "ring", 61_100_840, 64, 16, 8, sigma=0.1),
        # The refresh of the headline workload, over every slice of 32 gradients.
        _codec("refresh_vgg16", "refresh", 138_357_544, 128, 32, 16, L=32),
        # The refresh at the paper's slice size: a 768 x 768 covariance and its eigenvectors.
        _codec("refresh_conv768", "refresh", 138_357_544, 768, 96, 8, L=8),
        # The paper's own sampling: L_t = 100 gradients, one compressor per 1M elements from its first slice.
        _codec("sample_resnet50", "sample", 25_557_032, 768, 96, 8, block=1_000_000, sigma=0.1, L=100),
        # The monitor on the headline workload.
        _codec("monitor_vgg16", "monitor", 138_357_544, 128, 32, 16),
        # The packing of a whole network, from 64-element biases to a layer of 103 M numbers.
        {"name": "pack_vgg16", "kind": "pack", "layers": _VGG16, "dtype": "f32"},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _draw_slice(rng, d_most):
    """Slice length and comps: the powers of two and multiples of filters x depth that networks give, and any other;
    3 to 10 times compression, at most 128 comps."""
    d = rng.choice([16, 32, 64, 128, 256, 512, 768, 1024]) if rng.random() < 0.5 else _log_int(rng, 12, 1024)
    while d > d_most:
        d //= 2
    return d, max(1, min(128, round(d / rng.choice([3, 4, 4, 6, 8, 8, 10]))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "ring", "refresh", "sample", "monitor", "pack"])
    dtype = "bf16" if rng.random() < 0.3 else "f32"
    if kind == "pack":
        # a plain convolutional network: widths that double, 1 x 1 to 5 x 5 filters, a fully connected head
        f, depth, layers = rng.choice([16, 24, 32, 48, 64, 96]), 3, []
        for i in range(rng.randint(2, 10)):
            r = rng.choice([1, 3, 3, 3, 5])
            layers += [f"{f}x{depth}x{r}x{r}", f"{f}x1x1x1"]
            depth, f = f, min(512, f * rng.choice([1, 1, 2]))
        layers += [f"{_log_int(rng, 10, 4096)}x{depth * rng.choice([1, 4, 49])}x1x1"]
        return {"kind": "pack", "layers": ",".join(layers), "dtype": dtype}
    block = rng.choice([500_000, 1_000_000, 2_000_000]) if rng.random() < 0.3 else 0
    scales = 64 if rng.random() < 0.25 else 0
    sigma = rng.choice([0.05, 0.1])
    if kind == "refresh":
        d, k = _draw_slice(rng, 768)
        L = rng.randint(4, 32)
        M = _log_int(rng, 300_000, 800_000_000 // L)  # 32 gradients of up to 25 M elements, 6 of the largest
        M = min(M, 138_357_544)
        return _codec(None, kind, M, d, k, rng.choice([2, 4, 8, 16]), dtype, block if d <= 256 else 0, scales, sigma, L)
    if kind == "sample":
        d, k = _draw_slice(rng, 768)
        d = max(d, 64)
        L = rng.randint(12, 100)
        k = max(1, min(k, L - 2, d // 3))  # only L - 1 columns are determined by L samples
        return _codec(None, kind, _log_int(rng, 1_000_000, 25_557_032), d, k, rng.choice([2, 4, 8, 16]), dtype,
                      1_000_000, 0, sigma, L)
    d, k = _draw_slice(rng, 1024)
    N = rng.randint(2, 16)
    M = _log_int(rng, 300_000, min(138_357_544, 1_000_000_000 // N))
    return _codec(None, kind, M, d, k, N, dtype, block, scales, sigma)


# ---- inputs ---------------------------------------------------------------------------------------------------

def _dims(case):
    """(slices, slices per basis, bases)"""
    S = -(-case["M"] // case["d"])
    per = -(-case["block"] // case["d"]) if case["block"] else S
    return S, min(per, S), -(-S // min(per, S))


class _Model:
    """The planted model of a case: one mixing matrix and one small mean per basis."""

    def __init__(self, case, seed):
        self.case = case
        self.S, self.per, self.B = _dims(case)
        d, k = case["d"], case["k"]
        self.rank = max(1, min(24, (3 * k) // 4))
        self.gen = torch.Generator(device=DEV).manual_seed(seed * 7919 + 13)
        self.A = torch.randn(self.B, self.rank, d, generator=self.gen, device=DEV)
        self.mean = 0.05 * torch.randn(self.B, d, generator=self.gen, device=DEV)
        self.scale = None
        if case["scales"]:
            e = torch.rand(case["scales"], generator=self.gen, device=DEV) * 3.0 - 4.0
            at = torch.arange(self.S, device=DEV) // (-(-self.S // case["scales"]))
            self.scale = torch.pow(10.0, e)[at]

    def gradient(self, n_summed):
        """One gradient as stored: the sum of n_summed workers' draws (mean n_summed / N of the whole)."""
        c, d, root = self.case, self.case["d"], math.sqrt(n_summed)
        out = torch.empty(c["M"], dtype=torch.bfloat16 if c["dtype"] == "bf16" else torch.float32, device=DEV)
        chunk = max(1, (1 << 25) // d)
        for b0 in range(0, self.B, max(1, chunk // self.per)):
            b1 = min(self.B, b0 + max(1, chunk // self.per))
            for r0 in range(0, self.per, chunk):       # a single long basis is drawn in pieces
                r1 = min(self.per, r0 + chunk)
                s0 = b0 * self.per + r0
                z = torch.randn(b1 - b0, r1 - r0, self.rank, generator=self.gen, device=DEV)
                x = torch.randn(b1 - b0, r1 - r0, d, generator=self.gen, device=DEV)
                x = torch.bmm(z, self.A[b0:b1]).add_(x, alpha=c["sigma"]).mul_(root)
                x = x.add_(self.mean[b0:b1, None, :], alpha=n_summed / c["N"]).view(-1, d)
                if self.scale is not None:
                    x = x[: self.S - s0] * self.scale[s0:s0 + x.shape[0], None]
                e0 = s0 * d
                e1 = min(c["M"], e0 + x.shape[0] * d)
                out[e0:e1] = x.reshape(-1)[: e1 - e0]
        return out

    def restore(self, basis):
        """Orthonormal columns that span the planted directions (and random ones past the rank)."""
        k, d = self.case["k"], self.case["d"]
        more = torch.randn(self.B, max(0, k - self.rank), d, generator=self.gen, device=DEV)
        both = torch.cat([self.A, more], 1)[:, :k].transpose(1, 2).cpu().double()
        U = torch.linalg.qr(both)[0].float().contiguous().numpy()
        mean = self.mean if self.scale is None else self.mean * self.scale.mean()
        basis.import_(U, mean.cpu().numpy())


def _offsets(case):
    S, per, B = _dims(case)
    return None if not case["block"] else [min(S, b * per) for b in range(B + 1)]


def prepare(case, seed):
    f32 = dict(dtype=torch.float32, device=DEV)
    if case["kind"] == "pack":
        gen = torch.Generator(device=DEV).manual_seed(seed * 7919 + 29)
        dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        shapes = [tuple(int(v) for v in s.split("x")) for s in case["layers"].split(",")]
        layers = [torch.randn(*s, generator=gen, device=DEV).to(dt) for s in shapes]
        total = sum(t.numel() for t in layers)
        flat, at, parts = torch.empty(total, dtype=dt, device=DEV), 0, []
        for t in layers:
            parts.append(flat[at:at + t.numel()])
            at += t.numel()
        return {"kind": "pack", "dtype": gvq.BF16 if case["dtype"] == "bf16" else gvq.F32, "shapes": shapes,
                "layers": layers, "flat": flat, "parts": parts, "back": [torch.empty_like(t) for t in layers]}
    S, _, B = _dims(case)
    model = _Model(case, seed)
    basis = gvq.Basis(case["M"], case["d"], case["k"], _offsets(case), case["dtype"])
    st = {"kind": case["kind"], "N": case["N"], "basis": basis, "S": S}
    if case["kind"] in ("refresh", "sample"):
        st["grads"] = [model.gradient(case["N"]) for _ in range(case["L"])]
        return st
    model.restore(basis)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    if case["kind"] == "monitor":
        return dict(st, grad=model.gradient(1), loss=torch.empty(B, dtype=torch.float64, device=DEV))
    st["out"] = torch.empty(case["M"], dtype=dt, device=DEV)
    if case["kind"] == "ring":
        # the segments in the order this node meets them, the first node's place in the ring
        n = case["N"]
        cuts = [S * i // n for i in range(n + 1)]
        st["segments"] = [(cuts[i], cuts[i + 1] - cuts[i]) for i in reversed(range(n))]
        st["inbox"] = torch.randn(S * case["k"], generator=model.gen, **f32)
        return dict(st, grad=model.gradient(1), outbox=torch.empty(S * case["k"], **f32))
    return dict(st, grads=[model.gradient(1) for _ in range(case["N"])],
                comps=[torch.empty(S * case["k"], **f32) for _ in range(case["N"])],
                total=torch.empty(S * case["k"], **f32))


# ---- one pass -------------------------------------------------------------------------------------------------

def run(st):
    kind = st["kind"]
    if kind == "pack":
        for x, part, s in zip(st["layers"], st["parts"], st["shapes"]):
            gvq.gvq_flatten_conv(x, part, *s, st["dtype"])
        for x, part, s in zip(st["back"], st["parts"], st["shapes"]):
            gvq.gvq_unflatten_conv(part, x, *s, st["dtype"])
        return [st["flat"]] + st["back"]
    b, n = st["basis"], st["N"]
    if kind == "step":
        for g, c in zip(st["grads"], st["comps"]):
            b.compress(g, n, c)
        b.aggregate(st["comps"], st["total"])
        b.decompress(st["total"], st["out"])
        return [st["total"], st["out"]]
    if kind == "ring":
        for i, (first, count) in enumerate(st["segments"]):
            b.compress_segment(st["grad"], n, first, count, st["inbox"] if i else None, st["outbox"])
        for first, count in st["segments"]:
            b.decompress_segment(st["outbox"], first, count, st["out"])
        return [st["outbox"], st["out"]]
    if kind == "monitor":
        b.local_loss(st["grad"], n, st["loss"])
        return st["loss"]
    b.fit(st["grads"], first_slice_only=kind == "sample")
    b.fit_status()
    return list(b.export())


# ---- what a pass cannot do without, and how close results are ---------------------------------------------------

def work(case):
    es = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "pack":
        n = sum(math.prod(int(v) for v in s.split("x")) for s in case["layers"].split(","))
        return {"bytes": 4 * n * es, "flops": 0}
    S, _, B = _dims(case)
    M, d, k, N, L = (case[x] for x in ("M", "d", "k", "N", "L"))
    if case["kind"] == "step":
        return {"bytes": (N + 1) * M * es + 4 * S * k * (2 * N + 2), "flops": 2 * S * d * k * (N + 1) + N * S * k}
    if case["kind"] == "ring":
        return {"bytes": 2 * M * es + 4 * S * k * 3, "flops": 4 * S * d * k + S * k}
    if case["kind"] == "monitor":
        return {"bytes": M * es + 8 * B, "flops": 4 * S * d * k + 3 * M}
    basis = B * (4 * d * k + 4 * d + 8 * d)
    samples = L * (M // d) if case["kind"] == "refresh" else L * B
    # moments (one triangle), and about 9 d^3 for eigenvalues and eigenvectors; from L < d samples the
    # L x L problem has the same ones
    n = d if case["kind"] == "refresh" else min(L, d)
    return {"bytes": samples * d * es + basis, "flops": samples * d * (n + 1) + 9 * B * n ** 3}


def tolerance(case):
    """About four times what the same work in float64 shows (2-norm, then largest, difference)."""
    if case["kind"] == "pack":
        return "exact"
    if case["kind"] in ("refresh", "sample"):
        # float64 moments and eigenvectors, rounded to fp32; neighbouring noise eigenvalues 1e-9 of the largest
        # apart let an eigenvector of another solver turn by up to 1e-6 (4.6e-7 measured, largest 1e-5)
        return {"rel": 2e-6, "max": 4e-5}
    if case["kind"] == "monitor":
        return {"rel": 4e-7, "max": 1e-6}  # 8.4e-8: fp32 residuals, summed in float64
    if case["dtype"] == "bf16":
        # results are rounded to bf16: 1.7e-3, and one step of a bf16 number where a sum lies near a tie
        return {"rel": 5e-3, "max": 1.6e-2}
    d, k = case["d"], case["k"]
    if 2 * d * k < 40 * (d + k) or (d in (16, 32, 64, 128) and k <= 32):
        return {"rel": 1e-6, "max": 1e-5}  # exact products, fp32 sums: 2.3e-7, 2.5e-6
    return {"rel": 2e-5, "max": 3e-4}      # the documented two-term bf16 products: 5e-6, 8e-5
