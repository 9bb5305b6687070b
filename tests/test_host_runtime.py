"""CPU tests of the runtime around the kernels, on the host HIP stub."""
import pytest

import _host_hip as H


def test_a_failed_create_gives_everything_back(tmp_path):
    """A context whose creation fails after its memory is allocated gives back
    the arena and its slot of the pinned losses."""
    res = H.run("""
spec = {"layers": [("conv", 4, 3, 1), ("relu",), ("pool",), ("flatten",), ("linear", 3)], "num_classes": 3}
a = U.un_create([spec], 4, (3, 8, 8), "bf16")
failed = 0
for nth in (0, 1):  # the arena's clearing, the padded input's
    stub.stub_fail_memset(nth)
    try:
        U.un_create([spec], 4, (3, 8, 8), "bf16")
    except U.UnError as e:
        failed += e.status == U.UN_ERR_DEVICE and "stub error" in str(e)
stub.stub_fail_memset(-1)
U.un_destroy(a)
result = [failed, stub.stub_device(), stub.stub_pinned()]
""", tmp_path)
    assert res == [2, 0, 0]


@pytest.mark.parametrize("precision", ["f32", "bf16"])
def test_tokens_of_a_one_pixel_map(precision, tmp_path):
    """A 1x1 map read as tokens: the token layer's width and row stride are a
    token's, not the sample's (24 channels as 3 tokens of 8 features)."""
    res = H.run("""
spec = {"layers": [("conv", 24, 4, 0), ("relu",), ("flatten",), ("unflatten", 3), ("linear", 16), ("flatten",),
                   ("linear", 5)], "num_classes": 5}
h = U.Hybrid([spec], 6, (2, 4, 4), %r)
h.load_batch(np.zeros((6, 2, 4, 4), np.float32), np.zeros(6, np.int32))
launches()
h.step(0.1)
g = [l for l in launches() if "gemm_kernel" in l[0]]
p = [gemm_of(l) for l in g]
result = [(q.M, q.N, q.K, q.lda, q.ldb, q.ldc) for q in p]
""" % precision, tmp_path)
    # forward token layer and logits; backward by level: logits' data gradient,
    # token layer's data gradient, token layer's weight gradient
    assert res[0][:4] == [18, 16, 8, 8]
    assert res[1][:4] == [6, 5, 48, 48]
    assert res[3][:3] == [18, 8, 16] and res[3][5] == 8
    assert res[4][:3] == [16, 9, 18] and res[4][3:5] == [16, 8]


@pytest.mark.parametrize("precision", ["f32", "bf16"])
def test_unpadded_channels_take_the_element_wise_passes(precision, tmp_path):
    """test_conv_channels' model that cannot be padded runs what it is there for."""
    res = H.run("""
import test_conv_channels as T
wl = T.unpadded(%r)
h = U.Hybrid(wl.specs, wl.batch, wl.in_shape, wl.precision)
h.load_batch(*W.make_batch(wl, 0))
launches()
h.step(0.1)
result = [l[0] for l in launches() if "conv" in l[0]]
""" % precision, tmp_path)
    want = ["conv_fwd_kernel"] * 3 + ["conv_dgrad_kernel"] * 2 + ["conv_wgrad_kernel"]
    assert len(res) == len(want) and all(w in r for w, r in zip(want, res)), res


def test_scratch_limit_counts_the_models_own_channels(tmp_path):
    """un_step_scratch's limit counts a Linear layer's own inputs behind a conv
    whose 9 channels are stored as 16: its weight gradient's 2 splits of 1500 x
    2305 fit the 32 MiB array, of 1500 x 4097 they would not. The step runs; its
    padded partials outgrow the array, so in the context's own workspace. One of
    1500 x 4096 channels of its own is refused."""
    res = H.run("""
def status(channels):
    spec = {"layers": [("conv", channels, 1, 0), ("relu",), ("flatten",), ("linear", 1500), ("relu",), ("linear", 4)],
            "num_classes": 4}
    h = U.Hybrid([spec], 1088, (8, 16, 16), "bf16")
    h.load_batch(np.zeros((1088, 8, 16, 16), np.float32), np.zeros(1088, np.int32))
    try:
        U.un_step_scratch(h.ctx, 0.1, 1)
    except U.UnError as e:
        return e.status
    return 0


result = [status(9), status(16)]
""", tmp_path)
    assert res == [0, 7]


@pytest.mark.parametrize("precision", ["f32", "bf16"])
def test_narrow_conv_before_a_wide_linear_keeps_its_channels(precision, tmp_path):
    """Its one channel is not stored as 4 (bf16: 8), which would widen the Linear
    layer as much: the logits' and the wide layer's K in the forward pass, and the
    bytes of the plan."""
    res = H.run("""
import test_conv_channels as T
result = []
for sp in T.narrow_tails():
    h = U.Hybrid([sp], 8, (3, 32, 32), %r)
    h.load_batch(np.zeros((8, 3, 32, 32), np.float32), np.zeros(8, np.int32))
    launches()
    h.step(0.1)
    log = launches()
    wide = gemm_of([l for l in log if "gemm_kernel" in l[0]][0])
    result.append([wide.K, sum("conv_wgrad_kernel" in l[0] for l in log)])
    h.close()
""" % precision, tmp_path)
    vec = 8 if precision == "bf16" else 4
    assert res == [[1024, 1], [256, 1], [2 * 14 * 14, 1], [vec * 1024, 0]]


MLPS = """
def variants(width, n, batch, classes=10):
    layers = [x for w in [width] * 2 for x in (("linear", w), ("relu",))] + [("linear", classes)]
    h = U.Hybrid([{"layers": layers, "num_classes": classes}] * n, batch, (1024,), "bf16")
    h.load_batch(np.zeros((batch, 1024), np.float32), np.zeros(batch, np.int32))
    launches()
    h.step(0.1)
    log = launches()
    h.close()
    return log
"""


def test_small_tiles_only_where_large_ones_leave_half_the_chip_idle(tmp_path):
    """Forward launches of more than 512 small tiles take large ones (two bf16
    layers of width w, n models, a batch: 4096, 1, 1024 has 1024 of them; 2048, 1, 960
    at most 495), backward launches of more than 800 with weight gradients
    counted half."""
    res = H.run(MLPS + "result = [variants(4096, 1, 1024), variants(2048, 1, 960)]", tmp_path)
    wide, narrow = [H.gemm_variants(log) for log in res]
    # forward: two hidden layers, then the logits; backward: the logits' data
    # gradient, the second layer's with the logits' weight gradient, and the rest
    assert [v for b, v in wide if not b] == [0, 0, 1] and [v for b, v in wide if b] == [0, 0, 0]
    assert [v for b, v in narrow if not b] == [1, 1, 1] and [v for b, v in narrow if b] == [1, 1, 0]


def test_weight_gradients_that_one_chunk_holds_are_not_split(tmp_path):
    """bf16 blocks of more than 4 small tiles at batch 768 (12 k-blocks, one chunk
    of 16) take no partials and no reduction launch; longer batches split."""
    res = H.run(MLPS + """
result = [sum("reduce_kernel" in l[0] for l in variants(*a)) for a in ((256, 8, 768, 130), (256, 8, 2048, 130))]
""", tmp_path)
    assert res == [0, 1]


def test_small_conv_tiles_only_for_short_or_badly_filled_launches(tmp_path):
    """bf16 halo launches: 32 x 32 maps of 64 channels at batch 64 (256 tiles' area)
    take small tiles and at batch 128 large ones; 24 channels on 24 x 24, whose
    large tiles are mostly padding, small ones."""
    res = H.run("""
def convs(o, side, n, batch):
    spec = {"layers": [("conv", o, 3, 1), ("relu",), ("conv", o, 3, 1), ("relu",), ("pool",), ("flatten",), ("linear", 10)],
            "num_classes": 10}
    h = U.Hybrid([spec] * n, batch, (3, side, side), "bf16")
    h.load_batch(np.zeros((batch, 3, side, side), np.float32), np.zeros(batch, np.int32))
    launches()
    h.step(0.1)
    out = ["small" if "conv_halo_small" in l[0] else "large" for l in launches() if "conv_halo" in l[0]]
    h.close()
    return out


result = [convs(64, 32, 1, 64), convs(64, 32, 1, 128), convs(24, 24, 8, 64)]
""", tmp_path)
    assert res == [["small"] * 3, ["large"] * 3, ["small"] * 3]


def test_tile_variants_that_the_gpu_tests_compare(tmp_path):
    """test_gpu_gemm_tiles and test_conv_channels compare a model alone with one
    beside others: alone every launch takes small (or wide) tiles, beside the
    others every launch that the model takes part in large ones."""
    res = H.run("""
import test_conv_channels as TC
import test_gpu_gemm_tiles as T


def log(wl):
    h = U.Hybrid(wl.specs, wl.batch, wl.in_shape, wl.precision)
    h.load_batch(*W.make_batch(wl, 0))
    launches()
    h.step(0.1)
    out = launches()
    h.close()
    return out


result = [[[log(T.models(*c, p, alone)) for alone in (True, False)] for c in T.CASES] for p in ("f32", "bf16")]
conv = [[["small" in l[0] for l in log(TC.tiles(p, k, *c)) if "conv_halo" in l[0]] for k in (1, n)]
        for p, n in TC.TILES[0] for c in TC.TILES[1]]
result = [result, conv]
""", tmp_path)
    res, conv = res
    for alone, merged in conv:
        # (two rows of 24 pixels, which a pooled pass needs, are no small fp32 tile of 32 x 32)
        assert len(alone) == len(merged) == 5 and all(alone[1:]) and not any(merged)
    import test_gpu_gemm_tiles as T
    wide = 0
    for by_case in res:
        for (batch, classes, widths), (alone, merged) in zip(T.CASES, by_case):
            a, m = H.gemm_variants(alone), H.gemm_variants(merged)
            assert all(v != 0 for _, v in a), (batch, classes, widths)
            wide += sum(v == 2 for _, v in a)
            # forward: the model's levels; backward: all but the others' deepest
            assert all(v == 0 for _, v in [x for x in m if not x[0]][:len(widths) + 1]), (batch, classes, widths)
            assert all(v == 0 for _, v in [x for x in m if x[0]]), (batch, classes, widths)
    assert wide > 0
