"""CPU tests of the runtime around the kernels, on the host HIP stub."""
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
