"""Which path a size takes must not show: launch shapes of the step by layout size, records by pinned memory or by copy, rounds of a matrix
that ends with the parameter buffer.  Needs an MI355X."""
import numpy as np
import pytest

from oracle.runner import assert_stats_close
from synth import workloads as W
from test_gpu_parity import env, run_both  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(16, 65), (32, 63), (48, 67), (64, 127), (160, 129), (16, 1027), (256, 257), (512, 61)])
def test_last_rounds_of_a_matrix_that_ends_with_the_parameters(env, rows, cols):
    """All rows present and some columns missing: the last round takes the path whose loads end with the parameters.  The values; where the
    loads end is checked on the host, in test_host_profile.py."""
    torch = env["torch"]
    for dtype, theta in (("f32", torch.float32), ("bf16", torch.bfloat16)):
        w = W.Workload("end", [W._vec("v", 5), W._mat("m", 300, 70), W._mat("last", rows, cols)], 2, dtype, "cycle", **W.K6)
        W.layout(w, 1); W.draw_stream_params(w, 4)
        w.buffer_numel = max(b.offset + b.numel for b in w.blocks)
        run_both(env, w, 2, seed=5, theta_dtype=theta)


def _layout(kind, total):
    if kind == "matrices":
        shapes = [(4096, 2048), (2049, 4099), (1, 0)]
    elif kind == "vectors":
        shapes = [(total // 2 + 1, 0), (300, 70), (1023, 0)]
    else:      # partial rows (of large fp32 layouts, one per 256 coordinates and up to 7 more) around 3,072, where the second
               # launch begins, and last parts of up to 2,040
        shapes = [(3064, 256), (3072, 256), (3073, 256), (4088, 256), (4095, 256), (5112, 256), (5119, 256), (6144, 256), (1, 0),
                  (8192, 4096)]
    out, at, k = [], 0, 0
    while at < total:
        r, c = shapes[k % len(shapes)]; k += 1
        n = r * c if c else r
        out.append((at, n, r if c else 0, c)); at += n
    return out, at


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("kind,total", [
    ("vectors", 1_000_003), ("matrices", 1 << 23), ("matrices", 1 << 24), ("matrices", (1 << 25) + 1), ("vectors", (1 << 25) + 1),
    ("matrices", 45_000_001), ("vectors", 60_000_001), ("matrices", (1 << 26) + 1), ("vectors", (1 << 26) + 1), ("edges", (1 << 26) + 1)])
def test_default_step_shape_of_every_size_against_an_explicit_one(env, dtype, kind, total):
    """States to the bit, statistics up to the order of the partial sums, across a finalize whose lists may stand where the step's rows do."""
    torch, binding = env["torch"], env["binding"]
    blocks, numel = _layout(kind, total)
    code = 1 if dtype == "bf16" else 0
    own = dict(groups_per_wave=1, waves_per_workgroup=4, chunk_groups=8, resident_workgroups=5)
    profs = [binding.Profiler(blocks, binding.default_profile_params(grad_dtype=code, **kw)) for kw in ({}, own)]
    gen = torch.Generator(device="cuda:0").manual_seed(total % 1000)
    theta = 0.02 * torch.randn(numel, device="cuda:0", generator=gen)
    for t in range(4):
        grad = (torch.randn(numel, device="cuda:0", generator=gen) * 10.0 ** (t % 2 - 2)).to(torch.bfloat16 if code else torch.float32)
        for p in profs:
            p.step(grad)
        if t == 0:
            continue
        (a, _), (b, _) = (p.finalize(theta=theta) for p in profs)
        for i in range(len(blocks)):
            assert_stats_close(a[i], b[i], f"step {t}, block {i} {blocks[i]}")
    for i in range(len(blocks)):
        for x, y in zip(*(p.state(i) for p in profs)):
            assert torch.equal(x, y)


def test_records_of_handles_side_by_side_and_of_many_blocks(env):
    """4,097 blocks have their records copied, the halves of the layout write theirs to pinned memory; the first two handles live at a time, the
    next two take the buffers that they give back.  Blocks of one workgroup do not depend on the layout around them: the same bits."""
    torch, binding = env["torch"], env["binding"]
    blocks, at = [], 0
    for i in range(4097):
        r, c = (3 + i % 7, 2 + i % 11) if i % 3 == 0 else (0, 0)
        n = r * c if r else 1 + i % 300
        blocks.append((at, n, r, c)); at += n
    gen = torch.Generator(device="cuda:0").manual_seed(9)
    grads = [torch.randn(at, device="cuda:0", generator=gen) for _ in range(3)]
    theta = 0.02 * torch.randn(at, device="cuda:0", generator=gen)

    def stats(profs):
        for g in grads:
            for p in profs:
                p.step(g)
        out = [p.finalize(theta=theta)[0] for p in profs]
        for p in profs:
            p.close()
        return [bytes(s) for s in out]

    whole = stats([binding.Profiler(blocks)])[0]
    halves = (blocks[:2000], blocks[2000:])
    for _ in range(2):
        assert b"".join(stats([binding.Profiler(h) for h in halves])) == whole
