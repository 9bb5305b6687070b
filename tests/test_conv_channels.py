"""Channel counts that are no whole 16-byte vectors: stored padded with zero
channels, which must never show - in parameters, gradients, optimizer state,
losses - and never become non-zero."""
import numpy as np
import pytest

from paper_2408_01331_amd import workloads as W
from _parity import compare_run, compare_step, fro_err, run_gpu, run_oracle, tensor_err

L, C, R, POOL, FLAT, RB, RE = (lambda n: ("linear", n)), (lambda *a: ("conv",) + a), ("relu",), ("pool",), \
    ("flatten",), ("res_begin",), ("res_end",)


def _specs():
    return [
        # one channel, then three, unpooled and without a ReLU, odd maps
        {"layers": [C(1, 3, 1), R, POOL, C(3, 3, 0), C(8, 3, 1), R, FLAT, L(10)], "num_classes": 10},
        # a residual block of padded channels
        {"layers": [C(6, 3, 1), R, POOL, RB, C(6, 3, 1), R, C(6, 3, 1), RE, R, C(7, 3, 1), R, POOL, C(8, 1, 0), R, FLAT,
                    L(10)], "num_classes": 10},
        # LeNet-like: 5x5 without padding
        {"layers": [C(9, 5, 0), R, POOL, C(16, 5, 0), R, POOL, FLAT, L(20), R, L(10)], "num_classes": 10},
    ]


def _wl(precision, specs=None, steps=2):
    specs = _specs() if specs is None else specs
    return W.Workload("channels", len(specs), 13, (3, 28, 28), precision, specs, 0.02, steps, 4, init="torch")


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["f32", "bf16"])
def test_against_the_oracle_and_alone(precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = _wl(precision)
    m = list(range(wl.n_models))
    orc, spread = run_oracle(wl, 1, m, spread=True)
    print(compare_step(wl, run_gpu(wl, 1), orc, m, spread=spread))
    merged = run_gpu(wl, 2)
    orc, spread = run_oracle(wl, 2, m, spread=True)
    print(compare_run(wl, merged, orc, m, spread=spread))
    for i in m:
        solo = run_gpu(_wl(precision, [wl.specs[i]]), 2, theta={0: W.init_params(wl.specs[i], wl.in_shape, 4, i, "torch")})
        for a, b in zip([merged[0][:, i]] + merged[1][i] + merged[2][i], [solo[0][:, 0]] + solo[1][0] + solo[2][0]):
            assert np.array_equal(np.asarray(a, np.float32).view(np.uint32), np.asarray(b, np.float32).view(np.uint32))


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["f32", "bf16"])
@pytest.mark.parametrize("side,batch", [(5, 40), (9, 3), (18, 7), (22, 5), (24, 9), (40, 2), (66, 2)])
def test_row_tiles_that_rows_do_not_fill(precision, side, batch):
    """Maps whose rows or images do not fill a tile, pooled with and without a
    dropped last row and column, and maps wider than half a tile."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    specs = [{"layers": [C(c, 3, 1), R, POOL, C(40, 3, 1), R, C(8, 3, p), R] + ([POOL] if side > 9 else []) + [FLAT, L(10)],
              "num_classes": 10} for c, p in ((16, 1), (72, 0))]
    wl = W.Workload("rows", 2, batch, (3, side, side), precision, specs, 0.02, 1, 6, init="torch")
    if side == 5:  # the second model's last map would be empty
        wl.specs, wl.n_models = specs[:1], 1
    m = list(range(wl.n_models))
    orc, spread = run_oracle(wl, 1, m, spread=True)
    print(compare_step(wl, run_gpu(wl, 1), orc, m, spread=spread))


def tiles(precision, k, c1, c2):
    """k equal models of three convs."""
    spec = {"layers": [C(c1, 3, 1), R, POOL, C(c2, 3, 1), R, C(16, 3, 1), R, POOL, FLAT, L(10)], "num_classes": 10}
    return W.Workload("tiles", k, 16, (3, 24, 24), precision, [spec] * k, 0.02, 2, 4, init="torch")


TILES = [("f32", 40), ("bf16", 120)], [(8, 24), (33, 72)]


@pytest.mark.gpu
@pytest.mark.parametrize("precision,n", TILES[0])
@pytest.mark.parametrize("c1,c2", TILES[1])
def test_small_and_large_conv_tiles_agree(precision, n, c1, c2):
    """A model alone (small conv tiles) against the same model beside so many
    others that every conv launch takes the large ones: bit for bit."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    solo = run_gpu(tiles(precision, 1, c1, c2), 2)
    merged = run_gpu(tiles(precision, n, c1, c2), 2, models=[0])
    for a, b in zip([merged[0][:, 0]] + merged[1][0] + merged[2][0], [solo[0][:, 0]] + solo[1][0] + solo[2][0]):
        assert np.array_equal(np.asarray(a, np.float32).view(np.uint32), np.asarray(b, np.float32).view(np.uint32))


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["momentum", "adam"])
def test_parameters_and_state_round_trip(kind):
    """What set_params / set_opt_state put in, get_* gives back, and a run
    continued in a fresh context equals the run it left."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2408_01331_amd.unifiednn import Hybrid
    wl = _wl("f32")

    def fresh():
        h = Hybrid(wl.specs, wl.batch, wl.in_shape, "f32", seeds=[7, 8, 9])
        for i in range(h.n):
            h.set_optimizer(i, kind, momentum=0.9)
        h.load_batch(*W.make_batch(wl, 0))
        return h

    with fresh() as a, fresh() as b:
        a.step(1e-3)
        for i in range(a.n):
            b.set_params(i, a.get_params(i))
            b.set_opt_state(i, *a.get_opt_state(i))
            assert np.array_equal(a.get_params(i), b.get_params(i))
            assert np.array_equal(a.get_opt_state(i)[0], b.get_opt_state(i)[0])
        la, lb = a.step(1e-3), b.step(1e-3)
        assert np.array_equal(la, lb)
        for i in range(a.n):
            assert np.array_equal(a.get_params(i), b.get_params(i))


def unpadded(precision):
    """A model whose rows of a padded channel count would pass 2^24 elements: it
    runs with its own channels (1, 3, 1), element by element in every pass."""
    spec = {"layers": [C(3, 3, 1), R, C(1, 3, 1), R, POOL, C(1, 1, 0), FLAT, L(10)], "num_classes": 10}
    return W.Workload("unpadded", 1, 1, (1, 2, 1 << (21 if precision == "bf16" else 22)), precision, [spec], 0.02, 1, 4,
                      init="torch")


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["f32", "bf16"])
def test_channels_that_are_not_padded(precision):
    """The element-wise passes against the oracle. Some of the 2^22 ReLU and pool
    decisions per channel lie within rounding of a tie; one that goes the other
    way changes a gradient by one of 2^22 pixels' contributions, 2^-11 of its
    norm where they are independent, so ten of them 1.6e-3 (bf16: the operands'
    rounding, 2^-8, is more)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    wl = unpadded(precision)
    tol, grad_tol = {"f32": (1e-4, 1e-2), "bf16": (2e-2, 2e-2)}[precision]
    losses, params, grads = run_gpu(wl, 1)
    lo, po, go, _ = run_oracle(wl, 1, [0])[0]
    assert abs(losses[0, 0] - lo[0]) <= tol * abs(lo[0])
    for t, (a, b, ga, gb) in enumerate(zip(params[0], po, grads[0], go)):
        assert tensor_err(a, b) <= tol, t
        assert fro_err(ga, gb) <= grad_tol, (t, fro_err(ga, gb))


def test_planner_takes_channels_it_cannot_pad():
    """One-channel bf16 maps of 128 x 1024 x 1024 pass 2^31 bytes only when padded
    to 8 channels: the model is accepted and keeps its one channel, while at
    batch 64 it is padded."""
    from paper_2408_01331_amd.unifiednn import un_plan_bytes
    spec = {"layers": [C(1, 1, 256), POOL, C(8, 1, 0), POOL, FLAT, L(10)], "num_classes": 10}
    half, full = (un_plan_bytes([spec], b, (8, 512, 512), "bf16")[0] for b in (64, 128))
    # activation and gradient of the pooled one-channel map: 8 channels at batch 64, one at 128
    assert full < 2 * half - 2 * 64 * 512 * 512 * 2 * 6


def test_planner_takes_an_input_it_cannot_pad():
    """A one-channel bf16 input of 2^18 x 28 x 28 passes 2^31 bytes only when
    padded to 8 channels (3.3 GB, of which the kernels would read the first
    2^31 bytes): the group keeps its one channel, and no copy is made."""
    from paper_2408_01331_amd.unifiednn import un_plan_bytes
    spec = {"layers": [C(4, 5, 0), R, POOL, C(8, 3, 1), R, POOL, FLAT, L(10)], "num_classes": 10}
    n = 1 << 18
    small, full = (un_plan_bytes([spec], b, (1, 28, 28), "bf16")[0] for b in (n // 4, n))
    pix = 28 * 28
    # per sample: the staged fp32 batch, and the input in bf16: one channel, or 8
    assert full < 4 * small - n * pix * 2 * 6


def narrow_tails():
    """Last convs of 1 and 2 channels (pooled and not, a first conv and a second)
    in front of Linear layers so wide that the padded inputs would cost more than
    the vector loaders save; and one whose skip keeps it padded."""
    return [{"layers": sp + [FLAT, L(n), R, L(10)], "num_classes": 10} for sp, n in (
        ([C(1, 3, 1), R], 1024),
        ([C(8, 3, 1), R, POOL, C(1, 3, 1), R], 2560),
        ([C(2, 5, 0), R, POOL], 10240),
        ([C(1, 3, 1), R, RB, C(1, 3, 1), RE, R], 1024))]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["f32", "bf16"])
def test_narrow_conv_before_a_wide_linear(precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for k, sp in enumerate(narrow_tails()):
        wl = W.Workload("tail", 1, 8, (3, 32, 32), precision, [sp], 0.02, 1, 4, init="torch")
        orc, spread = run_oracle(wl, 1, [0], spread=True)
        print(k, compare_step(wl, run_gpu(wl, 1), orc, [0], spread=spread), flush=True)
