"""Finalize with one read of v (large layouts): the edges of its geometry against the oracle, large blocks against
64 bits, and the blocks that it hands on to the passes.  Needs an MI355X."""
import numpy as np
import pytest

from oracle.runner import OracleRunner, assert_stats_close, oracle_params
from test_gpu_parity import env  # noqa: F401

pytestmark = pytest.mark.gpu

# Columns around a lane's four, a load's 64, 128 and 256, two and three of these, a workgroup of 8 wavefronts (6,144) and of 16 (12,288; more go
# through the passes); rows around a load's and a batch's; blocks around the largest that one workgroup takes (65,536) and where the sample grows.
EDGES = [(2, 4), (3, 5), (5, 4), (16, 64), (33, 63), (65, 65), (130, 127), (17, 128), (1030, 67), (64, 1024), (64, 1025), (300, 255), (257, 256), (259, 257),
         (129, 511), (128, 513), (100, 767), (100, 769), (41, 2305), (23, 4097), (12, 6143), (11, 6144), (10, 6145), (6, 11008), (7, 12287), (3, 12288),
         (9, 12289), (2, 30000), (5000, 3), (900, 2048), (3, 0), (4, 0), (5, 0), (8191, 0), (65535, 0), (65536, 0), (65537, 0), (524289, 0), (4194305, 0)]
FILLER = (16384, 8192)


def _layout(pad):
    out, at = [], 0
    for r, c in EDGES + 3 * [FILLER]:                        # 3 * 2^27 coordinates next to the blocks that do not take part
        at = -(-at // pad) * pad
        n = r * c if c else r
        out.append((at, n, r if c else 0, c)); at += n
    return out, at


@pytest.mark.parametrize("grad,theta,pad", [("f32", "f32", 1), ("bf16", "bf16", 1), ("bf16", "f32", 64), ("f32", "bf16", 64), ("f32", None, 1)])
def test_edges_of_the_geometry(env, grad, theta, pad):  # noqa: F811
    torch, binding = env["torch"], env["binding"]
    blocks, numel = _layout(pad)
    params = binding.default_profile_params(grad_dtype=1 if grad == "bf16" else 0)
    prof = binding.Profiler(blocks, params)
    only = list(range(len(EDGES)))

    class Named:                                             # what OracleRunner asks of a block
        def __init__(self, b): self.offset, self.numel, self.rows, self.cols = b
    orc = OracleRunner([Named(b) for b in blocks], only, **oracle_params(params))
    gen = torch.Generator(device="cuda:0").manual_seed(17)
    dtype = {"f32": torch.float32, "bf16": torch.bfloat16}
    scale = torch.randn(numel, device="cuda:0", generator=gen).mul_(0.7).exp_()
    for _ in range(2):
        g = torch.randn(numel, device="cuda:0", generator=gen).mul_(scale).mul_(1e-2).to(dtype[grad])
        prof.step(g)
        orc.step_from_device(g)
    th = None if theta is None else (0.02 * torch.randn(numel, device="cuda:0", generator=gen)).to(dtype[theta])
    stats, _ = prof.finalize(theta=th)
    again, _ = prof.finalize(theta=th)
    assert bytes(stats) == bytes(again)
    want, _ = orc.finalize([], shapes=[b[2:] for b in blocks], theta=th)
    for i in only:
        assert_stats_close(stats[i], want[i], f"block {i} {EDGES[i]}")
    # the large block, against 64 bits: sums of 1.3e8 fp64 terms
    o, n, r, c = blocks[-1]
    v = prof.state(len(blocks) - 1)[1].double().view(r, c)
    row, col = v.mean(1), v.mean(0)
    F = ((v - row[:, None] * col[None, :] / row.mean()).pow(2).sum().sqrt() / v.pow(2).sum().sqrt()).item()
    assert abs(stats[len(blocks) - 1].F - F) <= 1e-6 * F
    if th is not None:
        p, t = 1.0 / (v.view(-1).sqrt() + 1e-12), th[o:o + n].double()
        C = (((p / p.mean() - 1.0) * t).pow(2).sum().sqrt() / t.pow(2).sum().sqrt()).item()
        assert abs(stats[len(blocks) - 1].C - C) <= 1e-6 * C
    order = v.view(-1).sort().values
    for got, q in ((stats[len(blocks) - 1].q10, 0.1), (stats[len(blocks) - 1].q90, 0.9)):
        at = q * (n - 1); lo = int(at)
        w = order[lo].item() + (at - lo) * (order[lo + 1].item() - order[lo].item())
        assert abs(got - w) <= 1e-12 * w


@pytest.mark.parametrize("kind", ["zeros", "constant", "two values", "nan", "inf", "rank one", "rows apart"])
def test_blocks_that_the_sample_does_not_settle(env, kind):  # noqa: F811
    """A block of 1.5 M coordinates, as a matrix and as a vector, next to ordinary ones: untouched coordinates around and well above a tenth,
    equal keys in an interval, values without order, v of rank one, rows of very different size.  The quantiles are those of v itself; F and C are what
    a layout below the line, which goes through the passes, has."""
    torch, binding = env["torch"], env["binding"]
    r, c = 1500, 1000
    blocks = [(0, r * c, r, c), (r * c, r * c), (2 * r * c, *[FILLER[0] * FILLER[1], *FILLER])]
    numel = 2 * r * c + FILLER[0] * FILLER[1]
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    g = torch.randn(numel, device="cuda:0", generator=gen).mul_(1e-2)
    for k in range(2):
        b = g[k * r * c:(k + 1) * r * c]
        hit = torch.rand(r * c, device="cuda:0", generator=gen)
        if kind == "zeros": b[hit < (0.3, 0.1)[k]] = 0.0
        if kind == "constant": b.fill_(0.125)
        if kind == "two values": b.fill_(0.125); b[hit < 0.5] = 0.25
        if kind == "nan": b[12345] = float("nan")
        if kind == "inf": b[12345] = float("inf")
        if kind == "rank one": b.copy_((torch.arange(r, device="cuda:0")[:, None] % 7 + 1.0).mul(torch.arange(c, device="cuda:0")[None, :] % 5 + 1.0).mul(0.25).reshape(-1))
        if kind == "rows apart": b.view(r, c).mul_(torch.randn(r, 1, device="cuda:0", generator=gen).mul_(3.0).exp_())
    theta = 0.02 * torch.randn(numel, device="cuda:0", generator=gen)
    got = binding.Profiler(blocks)
    ref = binding.Profiler(blocks[:2])                        # 3 M coordinates: the passes
    got.step(g); ref.step(g[:2 * r * c])
    a, b = got.finalize(theta=theta)[0], ref.finalize(theta=theta[:2 * r * c])[0]
    for i in range(2):
        assert_stats_close(a[i], b[i], f"{kind} {i}")
        if kind == "rank one":
            assert (a[0].F <= 1e-6) and abs(a[i].C - b[i].C) <= 1e-6 * b[i].C
        for f in ("q10", "q90"):
            assert np.array_equal([getattr(a[i], f)], [getattr(b[i], f)], equal_nan=True)
    assert bytes(a) == bytes(got.finalize(theta=theta)[0])


def _sampled(numel, pieces, piece):
    """First of the four coordinates that k_bracket reads as a block's `piece`-th piece."""
    z = (piece + 1) * 0x9E3779B9 & 0xffffffff
    z ^= z >> 16; z = z * 0x85EBCA6B & 0xffffffff; z ^= z >> 13; z = z * 0xC2B2AE35 & 0xffffffff; z ^= z >> 16
    share = numel // pieces
    return min(piece * share + (z * share >> 32), numel - 4) & ~3


@pytest.mark.parametrize("theta", ["f32", "bf16"])
@pytest.mark.parametrize("dead", [1, 4, 200])
def test_distortion_where_a_rare_p_is_large(env, dead, theta):  # noqa: F811
    """Coordinates with v = 0 and theta = 0 (a pruned or padded weight), at a block's start, where a block of several workgroups samples v, and
    over a whole row: p is 1e12 there and 1e2 elsewhere, so that the typical p of a sample that hits one says nothing about p-bar.  C against 64 bits:
    (p/p-bar - 1)^2 theta^2 and theta^2 are summed from fp32 terms of at most three roundings, which are independent; 1e-6 is eight of them."""
    torch, binding = env["torch"], env["binding"]
    shapes = [(65536, 0), (16384, 0), (4096, 0), (256, 256), (64, 64), (3, 1365), (65537, 0), (1500, 1000), (1500000, 0), FILLER]
    blocks, at = [], 0
    for r, c in shapes:
        n = r * c if c else r
        blocks.append((at, n, r if c else 0, c)); at += n
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    g = torch.rand(at, device="cuda:0", generator=gen).add_(0.5).mul_(0.3)
    th = (0.02 * torch.randn(at, device="cuda:0", generator=gen)).to({"f32": torch.float32, "bf16": torch.bfloat16}[theta])
    for o, n, r, c in blocks:
        pieces = 1024 * (16 if n >= 1 << 27 else 2)
        for first, count in [(0, c if dead == 200 and c else dead)] + ([(_sampled(n, pieces, 5), min(dead, 4))] if n > 65536 else []):
            g[o + first:o + first + count] = 0.0; th[o + first:o + first + count] = 0.0
    prof = binding.Profiler(blocks)
    prof.step(g)
    stats = prof.finalize(theta=th)[0]
    for i, (o, n, _, _) in enumerate(blocks):
        p, t = 1.0 / (prof.state(i)[1].double().sqrt() + 1e-12), th[o:o + n].double()
        C = (((p / p.mean() - 1.0) * t).pow(2).sum().sqrt() / t.pow(2).sum().sqrt()).item()
        assert abs(stats[i].C - C) <= 1e-6 * C, f"{shapes[i]}: {stats[i].C} {C}"


def _lines(prof, blocks, stats):
    """Every block's line of 32 words.  The records follow the states in the workspace (found by the sum of v of the last block, the fourth of its 32
    numbers), then 16 KB of histogram a block, then these."""
    torch, last = prof._torch, len(blocks) - 1
    tail = prof.state(last)[2]
    first = -(-(tail.data_ptr() + tail.numel() * tail.element_size() - prof.workspace.data_ptr()) // 256) * 256
    words = prof.workspace[first:first + (prof.workspace.numel() - first) // 8 * 8].view(torch.float64)
    at = [8 * (int(i) - 3 - 32 * last) for i in (words == stats[last].v_l1).nonzero().flatten()]
    at = [first + i for i in at if i >= 0 and i % 256 == 0]
    assert len(at) == 1
    hist = -(-(at[0] + 256 * len(blocks)) // 256) * 256
    return prof.workspace[hist + 16384 * len(blocks):hist + (16384 + 128) * len(blocks)].view(torch.int32).view(-1, 32)


def _marked(prof, blocks, stats):
    """The blocks that the one pass has handed on to the passes."""
    return _lines(prof, blocks, stats)[:, 2].nonzero().flatten().tolist()


def _quantiles(v):
    v = v.reshape(-1).sort().values
    out = []
    for q in (0.1, 0.9):
        at = q * (v.numel() - 1); lo = int(at)
        a, b = v[lo].item(), v[min(lo + 1, v.numel() - 1)].item()
        out.append(a + (at - lo) * (b - a))
    return out


@pytest.mark.parametrize("kind", ["zero", "constant", "zeros 95", "zeros 90", "clipped", "bf16", "half rounded", "bf16 rows"])
def test_equal_keys_take_one_read(env, kind):  # noqa: F811
    """After one step: dead blocks, mostly untouched ones, gradients clipped by value, constant ones, and bf16 gradients of large blocks
    (42,000 of 16.8 M have the same v at the upper quantile), also next to others between them, and of rows of which most are untouched.  Quantiles are those of the sorted v, and no block goes through the passes."""
    torch, binding = env["torch"], env["binding"]
    shapes = [(1500, 1000), (1500000, 0), (4096, 4096), FILLER]
    blocks, at = [], 0
    for r, c in shapes:
        n = r * c if c else r
        blocks.append((at, n, r if c else 0, c)); at += n
    gen = torch.Generator(device="cuda:0").manual_seed(8)
    g = torch.randn(at, device="cuda:0", generator=gen).mul_(1e-2)
    for o, n, r, c in blocks[:3]:
        b = g[o:o + n]
        if kind == "zero": b.zero_()
        if kind == "constant": b.fill_(0.125)
        if kind.startswith("zeros"): b[torch.rand(n, device="cuda:0", generator=gen) < 0.01 * int(kind[6:])] = 0.0
        if kind == "clipped": b.clamp_(-0.012, 0.012)
        if kind == "half rounded": b.copy_(torch.where(torch.rand(n, device="cuda:0", generator=gen) < 0.5, b.to(torch.bfloat16).float(), b))
        if kind == "bf16 rows" and c: b.view(r, c)[torch.rand(r, device="cuda:0", generator=gen) < 0.8] = 0.0
    prof = binding.Profiler(blocks, binding.default_profile_params(grad_dtype=1 if kind.startswith("bf16") else 0))
    prof.step(g.to(torch.bfloat16) if kind.startswith("bf16") else g)
    if kind == "bf16 rows": prof.step(g.flip(0).to(torch.bfloat16))
    for _ in range(2):
        stats = prof.finalize()[0]
        assert _marked(prof, blocks, stats) == []
        for i in range(len(blocks)):
            want = _quantiles(prof.state(i)[1])
            for got, w in zip((stats[i].q10, stats[i].q90), want):
                assert abs(got - w) <= 1e-12 * w, f"{shapes[i]}: {got} {w}"


@pytest.mark.parametrize("kind", ["nine neighbours", "rows", "equal in a row"])
def test_neighbours_that_are_alike_take_one_read(env, kind):  # noqa: F811
    """240 blocks of 1 M and one of 16.8 M whose neighbouring coordinates share their scale, or their value: the sample's ranks vary more than those of
    independent coordinates.  No block's rank is outside its interval, no list too short."""
    torch, binding = env["torch"], env["binding"]
    blocks = [(i << 20, 1 << 20, 1024, 1024) for i in range(240)] + [(240 << 20, 1 << 24, 4096, 4096)]
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    g = torch.randn(256 << 20, device="cuda:0", generator=gen).mul_(1e-2)
    for o, n, r, c in blocks:
        b = g[o:o + n]
        if kind == "nine neighbours": b[:n // 9 * 9].view(-1, 9).mul_(torch.randn(n // 9, 1, device="cuda:0", generator=gen).mul_(2.0).exp_())
        if kind == "rows": b.view(r, c).mul_(torch.randn(r, 1, device="cuda:0", generator=gen).mul_(2.0).exp_())
        if kind == "equal in a row": b.view(r, c).copy_(torch.randn(r, 1, device="cuda:0", generator=gen).expand(r, c))
    prof = binding.Profiler(blocks)
    prof.step(g)
    stats = prof.finalize()[0]
    assert _marked(prof, blocks, stats) == []
    for i in range(0, len(blocks), 16):
        for got, w in zip((stats[i].q10, stats[i].q90), _quantiles(prof.state(i)[1])):
            assert abs(got - w) <= 1e-12 * w, f"{i}: {got} {w}"


@pytest.mark.parametrize("share", [0.15, 0.2, 0.3, 0.35, 0.45])
def test_mean_of_p_over_long_runs_of_one_value(env, share):  # noqa: F811
    """v is 1/4 over a block's first part and 1 over the rest, so that a lane adds one value of p / p0 - 1 again and again; theta is one at every 1,021st
    coordinate, which leaves the other sums of C exact.  What is rounded are the two values, by at most 2^-25, and their squares, by 2^-24: C is within
    2^-24 of 64 bits for these, and p-bar adds 2^-25 (p/p-bar) / |p/p-bar - 1|, at most 2^-24 * 1.5 for these shares; 1.5e-7 is 2^-24 * 2.5.
    (Sums of 256 fp32 terms: up to 8.8e-7.)"""
    torch, binding = env["torch"], env["binding"]
    shapes = [(1 << 22, 0), (2048, 2048), (65536, 0), FILLER]
    blocks, at = [], 0
    for r, c in shapes:
        n = r * c if c else r
        blocks.append((at, n, r if c else 0, c)); at += n
    g, th = torch.full((at,), 2.0, device="cuda:0"), torch.zeros(at, device="cuda:0")
    for o, n, _, _ in blocks:
        g[o:o + int(share * n)] = 1.0
        th[o + 7:o + n:1021] = 1.0
    prof = binding.Profiler(blocks, binding.default_profile_params(beta_v=0.75))
    prof.step(g)
    stats = prof.finalize(theta=th)[0]
    for i, (o, n, _, _) in enumerate(blocks):
        p, t = 1.0 / (prof.state(i)[1].double().sqrt() + 1e-12), th[o:o + n].double()
        C = (((p / p.mean() - 1.0) * t).pow(2).sum().sqrt() / t.pow(2).sum().sqrt()).item()
        assert abs(stats[i].C - C) <= 1.5e-7 * C, f"{shapes[i]}: {stats[i].C} {C}"


@pytest.mark.parametrize("seed", [5, 7])
def test_row_totals_and_mu_have_no_error_of_their_own(env, seed):  # noqa: F811
    """Equal rows of whole numbers below 2^15: v, the sums over 256 columns in fp32 and the column means are exact, so that of r_i, c_j and mu only r_i is
    rounded, to fp32, and F is that relative error: 2^-24 at most, and 2 % for the cancellation in fp64 (F^2 of 2^-48, terms of 1, 2^-53 each).  (Sums of
    whole rows in fp32 gave 1.18 and 1.31 times 2^-24 here.)"""
    torch, binding = env["torch"], env["binding"]
    blocks, at = [], 0
    for r, c in [(700, 12288), (700, 11008), (1400, 6144), (1400, 4608), (2000, 4096), (4000, 2000), FILLER]:
        blocks.append((at, r * c, r, c)); at += r * c
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    g = torch.empty(at, device="cuda:0")
    for o, n, r, c in blocks:
        g[o:o + n].view(r, c).copy_(2.0 * torch.randint(100, 182, (1, c), device="cuda:0", generator=gen).float().expand(r, c))
    prof = binding.Profiler(blocks, binding.default_profile_params(beta_v=0.75))
    prof.step(g)
    stats = prof.finalize()[0]
    for i, b in enumerate(blocks):
        assert stats[i].F <= 1.02 * 2.0 ** -24, f"{b[2:]}: {stats[i].F * 2.0 ** 24}"


def _packed(shapes):
    out, at = [], 0
    for r, c in shapes:
        n = r * c if c else r
        out.append((at, n, r if c else 0, c)); at += n
    return out, at


@pytest.mark.parametrize("layout", ["edges", "special values"])
def test_layouts_of_these_tests_take_one_read(env, layout):  # noqa: F811
    """Blocks of several workgroups have intervals (words 8 to 11) if they take part."""
    torch, binding = env["torch"], env["binding"]
    blocks, numel = _layout(1) if layout == "edges" else _packed([(1500, 1000), (1500000, 0), FILLER])
    prof = binding.Profiler(blocks)
    prof.step(torch.randn(numel, device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(2)))
    lines = _lines(prof, blocks, prof.finalize()[0])[:, 9].cpu()
    for i, (_, n, r, c) in enumerate(blocks):
        several = n > 65536 or (r and c > 6144)
        assert (int(lines[i]) != 0) == (several and not (r and c > 12288)), blocks[i]


SPECIAL = ["zeros", "constant", "two values", "nan", "inf", "rank one", "dead start"]


@pytest.mark.parametrize("kind", SPECIAL)
@pytest.mark.parametrize("all_take_part", [True, False])
def test_special_values_next_to_each_other(env, kind, all_take_part):  # noqa: F811
    """Blocks of one workgroup (up to 65,536 coordinates) and of several, of untouched, equal and non-finite values.  Where a block of two columns is in
    the layout, which cannot take part, the passes follow the one pass at once instead of after a look at the marks.  Against the passes alone, which a
    layout of these blocks only goes through."""
    torch, binding = env["torch"], env["binding"]
    shapes = [(65536, 0), (256, 256), (5, 0), (33, 63), (16, 64), (4, 0), (65537, 0), (700, 500)] + ([] if all_take_part else [(40000, 2)])
    blocks, small = _packed(shapes)
    whole, numel = _packed(shapes + ([FILLER] if all_take_part else 3 * [FILLER]))
    gen = torch.Generator(device="cuda:0").manual_seed(6)
    g = torch.randn(numel, device="cuda:0", generator=gen).mul_(1e-2)
    theta = 0.02 * torch.randn(numel, device="cuda:0", generator=gen)
    for o, n, r, c in blocks:
        b, hit = g[o:o + n], torch.rand(n, device="cuda:0", generator=gen)
        if kind == "zeros": b[hit < 0.3] = 0.0
        if kind == "constant": b.fill_(0.125)
        if kind == "two values": b.fill_(0.125); b[hit < 0.5] = 0.25
        if kind == "nan": b[n // 2] = float("nan")
        if kind == "inf": b[n // 2] = float("inf")
        if kind == "rank one" and c: b.copy_((torch.arange(r, device="cuda:0")[:, None] % 7 + 1.0).mul(torch.arange(c, device="cuda:0")[None, :] % 5 + 1.0).mul(0.25).reshape(-1))
        if kind == "dead start": b[:c or n // 8] = 0.0; theta[o:o + (c or n // 8)] = 0.0
    one, ref = binding.Profiler(whole), binding.Profiler(blocks)
    one.step(g); ref.step(g[:small])
    a, b = one.finalize(theta=theta)[0], ref.finalize(theta=theta[:small])[0]
    if kind in ("nan", "inf"):
        assert _marked(one, whole, a) == [i for i in range(len(shapes)) if (shapes[i][1] > 2 or (kind == "nan" and not shapes[i][1]))]
    elif kind not in ("two values", "rank one"):             # few values, of which an interval's fill the lists
        assert _marked(one, whole, a) == []
    for i in range(len(shapes)):
        assert_stats_close(a[i], b[i], f"{kind} {shapes[i]}")
        assert np.array_equal([a[i].q10, a[i].q90], [b[i].q10, b[i].q90], equal_nan=True)
    assert bytes(a) == bytes(one.finalize(theta=theta)[0])


@pytest.mark.parametrize("theta", ["f32", "bf16", None])
def test_without_F_and_with_a_given_one_on_another_stream(env, theta):  # noqa: F811
    """compute_F=False and F_raw are kernels of their own: every other statistic is the same to the bit.  Geometries of 8 and of 16 wavefronts, vectors,
    blocks of one workgroup and of several.  The calls are made on a stream of their own."""
    torch, binding = env["torch"], env["binding"]
    shapes = [(4096, 2048), (2000, 11008), (3000, 5000), (256, 256), (900000, 0), (50000, 0), FILLER]
    blocks, numel = _packed(shapes)
    gen = torch.Generator(device="cuda:0").manual_seed(12)
    g = torch.randn(numel, device="cuda:0", generator=gen).mul_(1e-2)
    th = None if theta is None else (0.02 * torch.randn(numel, device="cuda:0", generator=gen)).to({"f32": torch.float32, "bf16": torch.bfloat16}[theta])
    prof = binding.Profiler(blocks)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        prof.step(g)
        full, none, given = (prof.finalize(theta=th, **kw)[0] for kw in ({}, dict(compute_F=False), dict(F_raw=[0.25] * len(blocks))))
    assert _marked(prof, blocks, full) == []
    for i in range(len(blocks)):
        assert none[i].F == 0.0 and given[i].F == 0.25
        for f, _ in full[i]._fields_:
            if f in ("F", "s_F"):
                continue
            # without F a matrix of one workgroup has another order of its sums of C
            same = abs(getattr(none[i], f) - getattr(full[i], f)) <= 2e-7 * abs(getattr(full[i], f))
            assert same and getattr(none[i], f) == getattr(given[i], f), f"{shapes[i]} {f}"
        v = prof.state(i)[1]
        for got, w in zip((none[i].q10, none[i].q90), _quantiles(v)):
            assert abs(got - w) <= 1e-12 * w


def test_records_by_copy(env):  # noqa: F811
    """4,097 blocks have their records copied, the halves of the layout write theirs to pinned memory; the first and the last block go through the passes.
    Tasks are of one size in all three: the same bits."""
    torch, binding = env["torch"], env["binding"]
    blocks, numel = _packed(4097 * [(627, 628)])
    gen = torch.Generator(device="cuda:0").manual_seed(13)
    g = torch.empty(numel, dtype=torch.bfloat16, device="cuda:0")
    for at in range(0, numel, 1 << 28):
        part = g[at:at + (1 << 28)]
        part.copy_(torch.randn(part.numel(), device="cuda:0", generator=gen).mul_(1e-2))
    g[:1000] = float("inf"); g[-1000:] = float("nan")

    def stats(part):
        prof = binding.Profiler(part, binding.default_profile_params(grad_dtype=1))
        prof.step(g)
        return bytes(prof.finalize()[0])
    assert stats(blocks[:2048]) + stats(blocks[2048:]) == stats(blocks)


def test_one_read_without_theta_and_the_passes_with_it(env):  # noqa: F811
    """Blocks of 1,152 columns, of which a quarter of a workgroup's lanes has none, are read once without theta and go through the passes with it: by turns
    on one handle, each with the same bits every time; quantiles are the same, F of either is within the bound of the oracle's comparison."""
    torch, binding = env["torch"], env["binding"]
    blocks, numel = _packed(316 * [(1152, 1152)])
    gen = torch.Generator(device="cuda:0").manual_seed(21)
    prof = binding.Profiler(blocks, binding.default_profile_params(grad_dtype=1))
    prof.step(torch.randn(numel, device="cuda:0", generator=gen).mul_(1e-2).to(torch.bfloat16))
    theta = (0.02 * torch.randn(numel, device="cuda:0", generator=gen)).to(torch.bfloat16)
    first = [prof.finalize(theta=t)[0] for t in (theta, None)]
    for _ in range(2):
        for t, want in zip((theta, None), first):
            assert bytes(prof.finalize(theta=t)[0]) == bytes(want)
    for a, b in zip(*first):
        assert (a.q10, a.q90) == (b.q10, b.q90) and abs(a.F - b.F) <= 1e-6 * b.F and a.C > 0.0 and b.C == 0.0
    for i in (0, 315):
        for got, w in zip((first[0][i].q10, first[0][i].q90), _quantiles(prof.state(i)[1])):
            assert abs(got - w) <= 1e-12 * w
