"""GPU: the tile variants of the grouped GEMM. A launch of few tiles runs small
ones; the variant must not change a bit of any model's result, at the edges of
either tile size and with a fused softmax-CE wider than the small tile."""
import numpy as np
import pytest

from paper_2408_01331_amd import workloads as W
from _parity import compare_step, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _need_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _mlp(widths, classes):
    layers = []
    for w in widths:
        layers += [("linear", w), ("relu",)]
    return {"layers": layers + [("linear", classes)], "num_classes": classes}


# (batch, classes, widths): tile edges +- 1, one row, a k-block remainder, classes
# of one small tile, of more than one (fused over the large width) and of more
# than a large one (separate softmax-CE pass); widths of whole small tiles, whose
# bias gradient is summed on its own, with a k remainder and split over k
CASES = [(1, 10, [8]), (31, 33, [33]), (32, 32, [65, 31]), (33, 64, [64, 127]), (65, 65, [129, 63]),
         (127, 100, [72, 40]), (129, 130, [128, 257]), (200, 10, [128, 64]), (700, 10, [128, 64])]


def models(batch, classes, widths, precision, alone):
    """The case's model, alone or as the first beside 350 others with one hidden
    level more, enough that every launch that it takes part in has large tiles
    (test_host_runtime checks the variants)."""
    specs = [_mlp(widths, classes)]
    if not alone:
        specs += [_mlp([136] * (len(widths) + 1), classes) for _ in range(350)]
    return W.Workload("t", len(specs), batch, (104,), precision, specs, 0.05, 2, 9)


def _same(a, b):
    assert np.array_equal(np.asarray(a, np.float32).view(np.uint32), np.asarray(b, np.float32).view(np.uint32))


@pytest.mark.parametrize("precision", ["f32", "bf16"])
@pytest.mark.parametrize("batch,classes,widths", CASES)
def test_alone_equals_in_a_large_launch(precision, batch, classes, widths):
    """The model alone (small tiles) against the same model beside enough others
    that every one of its launches takes large tiles: losses, parameters and
    gradients, bit for bit; and alone against the oracle."""
    _need_gpu()
    case = (batch, classes, widths, precision)
    alone = run_gpu(models(*case, True), 2)
    merged = run_gpu(models(*case, False), 2, models=[0])
    _same(alone[0][:, 0], merged[0][:, 0])
    for a, b in zip(alone[1][0] + alone[2][0], merged[1][0] + merged[2][0]):
        _same(a, b)
    orc, spread = run_oracle(models(*case, True), 1, [0], spread=True)
    print(compare_step(models(*case, True), run_gpu(models(*case, True), 1), orc, [0], spread=spread))


@pytest.mark.parametrize("precision", ["f32", "bf16"])
@pytest.mark.parametrize("kind", ["sgd", "momentum", "adam"])
@pytest.mark.parametrize("batch,classes,widths", [(33, 64, [64, 127]), (129, 130, [128, 257]), (700, 10, [128, 64])])
def test_optimizer_epilogues_agree(precision, kind, batch, classes, widths):
    """The same with a rate per model, under SGD beside SGD models, and under
    momentum and Adam beside models of all three kinds in turn, so that a large
    launch's first-layer weight gradient mixes them over its rows: parameters and
    optimizer state."""
    _need_gpu()
    from paper_2408_01331_amd.unifiednn import Hybrid, flatten_params
    out = []
    for alone in (True, False):
        wl = models(batch, classes, widths, precision, alone)
        with Hybrid(wl.specs, wl.batch, wl.in_shape, wl.precision) as h:
            for i in range(wl.n_models):
                h.set_params(i, flatten_params(W.init_params(wl.specs[i], wl.in_shape, wl.seed, i, wl.init)))
                if kind != "sgd":
                    h.set_optimizer(i, kind if i == 0 else ("sgd", "momentum", "adam")[i % 3], momentum=0.9)
            rates = 1e-3 * (1 + np.arange(wl.n_models) % 5).astype(np.float32)
            for step in range(3):
                h.load_batch(*W.make_batch(wl, step))
                h.step(rates)
            out.append((h.get_params(0), h.get_opt_state(0)[0]))
    for a, b in zip(*out):
        _same(a, b)


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
