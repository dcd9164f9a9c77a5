"""What fv_launch_shape reports is what launches take: one quote per thread at
any configured quotes_per_thread (the ragged kernel: one or two by the batch's
size), the workgroup size as configured."""
import ctypes

import pytest

from paper_2604_27210_amd import _native as N


def _shape(fn, *args):
    b, q = ctypes.c_int(), ctypes.c_int()
    assert fn(*args, ctypes.byref(b), ctypes.byref(q)) == N.FV_OK
    return b.value, q.value


@pytest.mark.parametrize("kernel", sorted(N.KERNELS, key=N.KERNELS.get))
def test_reported_shape(kernel):
    lib, k = N.load(), N.KERNELS[kernel]
    saved = _shape(lib.fv_get_launch, k)
    try:
        assert lib.fv_set_launch(k, 256, 8) == N.FV_OK
        assert _shape(lib.fv_get_launch, k) == (256, 8)  # kept and given back
        most = 2 if kernel == "chains" else 1
        assert _shape(lib.fv_launch_shape, k, 0, 1 << 30) == (256, most)
        assert _shape(lib.fv_launch_shape, k, 0, 1000) == (64, 1)
        # as refused as before, though no launch has that many queue entries
        refused = kernel in ("iv_halley", "iv_halley_f32")
        assert (lib.fv_set_launch(k, 512, 16) == N.FV_E_INVALID_ARG) == refused
    finally:
        assert lib.fv_set_launch(k, *saved) == N.FV_OK


@pytest.mark.gpu
def test_tuned_size_of_a_file_with_quotes_per_thread(tmp_path):
    """A tuning file of an earlier build: its sizes are taken, its
    quotes_per_thread is kept in the file alone; the autotuner finds a size."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_27210_amd as fv
    path = tmp_path / "t.json"
    try:
        fv.reset_tuning()
        b, q = fv.autotune("iv_halley", "bs", 1 << 15)
        assert b in (64, 128, 256, 512) and q == 1
        fv.save_tuning(str(path))
        text = path.read_text()
        assert '"qpt": 1,' in text
        path.write_text(text.replace('"block": %d, "qpt": 1' % b, '"block": 128, "qpt": 4'))
        fv.load_tuning(str(path))
        assert fv.launch_shape("iv_halley", "bs", 1 << 15) == (128, 1)
        fv.save_tuning(str(path))
        assert '"block": 128, "qpt": 4' in path.read_text()
    finally:
        fv.reset_tuning()
