"""GPU: the tile variants of the grouped GEMM. A launch of few tiles runs small
ones; the variant must not change a bit of any model's result, at the edges of
either tile size and with a fused softmax-CE wider than the small tile."""
import numpy as np
import pytest

from paper_2408_01331_amd import workloads as W
from _parity import run_gpu

pytestmark = pytest.mark.gpu


def _mlp(widths, classes):
    layers = []
    for w in widths:
        layers += [("linear", w), ("relu",)]
    return {"layers": layers + [("linear", classes)], "num_classes": classes}


# (batch, classes, widths): tile edges +- 1, one row, a k-block remainder, classes
# of one small tile, of more than one (fused over the large width) and of more
# than a large one (separate softmax-CE pass)
CASES = [(1, 10, [8]), (31, 33, [33]), (32, 32, [65, 31]), (33, 64, [64, 127]), (65, 65, [129, 63]),
         (127, 100, [72, 40]), (129, 130, [128, 257])]


@pytest.mark.parametrize("precision", ["f32", "bf16"])
@pytest.mark.parametrize("batch,classes,widths", CASES)
def test_alone_equals_in_a_large_launch(precision, batch, classes, widths):
    """The model alone (small tiles) against the same model beside enough others
    that every one of its launches takes large tiles: losses, parameters and
    gradients."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    spec = _mlp(widths, classes)
    # one hidden level more than the model, and over 256 large tiles at each
    big = [_mlp([136] * (len(widths) + 1), classes) for _ in range(260)]
    specs = [spec] + big

    def wl(sp):
        return W.Workload("t", len(sp), batch, (104,), precision, sp, 0.05, 2, 9)

    alone = run_gpu(wl([spec]), 2)
    merged = run_gpu(wl(specs), 2, models=[0])
    assert np.array_equal(alone[0][:, 0].view(np.uint32), merged[0][:, 0].view(np.uint32))
    for a, b in zip(alone[1][0] + alone[2][0], merged[1][0] + merged[2][0]):
        assert np.array_equal(np.asarray(a, np.float32).view(np.uint32), np.asarray(b, np.float32).view(np.uint32))
    if precision == "bf16":
        return
    # and against the oracle (one step's loss)
    import oracle
    x, y = W.make_batch(wl([spec]), 0)
    lo, _, _ = oracle.step(spec, W.init_params(spec, (104,), 9, 0), x, y, 0.05, precision)
    assert abs(alone[0][0, 0] - lo) <= 1e-5 * abs(lo)


def test_scratch_step_beyond_the_array():
    """40 fp32 MLPs at batch 1024: within the scratch step's limit, which counts
    chunks of 1024 rows (none here), but their chunks of 256 rows need 40 MiB of
    partials. The step runs, in the arena, and equals un_step bit for bit."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_01331_amd import unifiednn as U
    n = 40
    wl = W.Workload("t", n, 1024, (64,), "f32", [_mlp([256, 256], 10)] * n, 0.05, 1, 9)
    x, y = W.make_batch(wl, 0)
    out = []
    for step in (U.un_step, U.un_step_scratch):
        with U.Hybrid(wl.specs, wl.batch, wl.in_shape, "f32", seeds=list(range(n))) as h:
            h.load_batch(x, y)
            losses = step(h.ctx, 0.05, n)
            out.append((losses, h.get_params(0), h.get_params(n - 1)))
    for a, b in zip(*out):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
