"""The U-Net's launch shapes against each other: a layer's result does not depend on the shape it is
launched in, bit for bit, as long as its products accumulate in the same order (include/ssn.h)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _net(levels, base, n, H, W, seed=11):
    import paper_2603_24370_amd as ss
    from paper_2603_24370_amd import learned
    net = ss.Net(levels, base, 2, 4, n, H, W)
    net.set_weights(learned.init_weights(seed, levels, base))
    return net


def _images(n, H, W, seed=5):
    rng = np.random.default_rng(seed)
    return (rng.normal(size=(n, H, W, 2)).astype(np.float32), rng.normal(size=(n, H, W, 4)).astype(np.float32))


def _grads_at(net, n):
    import paper_2603_24370_amd as ss  # noqa: F401
    return [net.read_tensor(3, k, n) for k in range(4 * net.levels - 2)]


# widths of 1 to 4 tiles of 32 pixels, channel blocks that end part-way (48) and half-filled chunks (16, 48)
@pytest.mark.parametrize("levels,base,H,W", [(2, 64, 64, 128), (2, 48, 64, 96), (3, 16, 64, 64), (2, 16, 32, 64)])
def test_rows_per_wave_do_not_change_the_result(levels, base, H, W, monkeypatch):
    """Chunked layers: a batch (several rows per wave) and its images one at a time (one row per wave)."""
    monkeypatch.setenv("SSN_CONV_SHAPE", "3")
    n = 8
    net = _net(levels, base, n, H, W)
    x, t = _images(n, H, W)
    whole = net.forward(x).cpu().numpy().copy()
    net.backward(t)
    scale = np.float32(n)  # the loss is a mean over the batch: its gradient scales by a power of two
    gz = _grads_at(net, n)
    for k in (0, n - 1):
        one = net.forward(x[k:k + 1]).cpu().numpy()
        assert np.array_equal(one[0], whole[k]), k
        net.backward(t[k:k + 1])
        for layer, g in enumerate(_grads_at(net, 1)):
            assert np.array_equal(g[0], scale * gz[layer][k]), (k, layer)
    net.close()


# every layer of these accumulates tap by tap: 32- and 96-pixel rows, 16 to 384 input channels
@pytest.mark.parametrize("levels,base,H,W", [(3, 32, 128, 128), (2, 16, 32, 96), (3, 48, 64, 64), (3, 64, 64, 64)])
def test_streamed_weights_equal_direct_operands(levels, base, H, W, monkeypatch):
    x, t = _images(1, H, W)
    got = {}
    for shape in ("0", "2"):
        monkeypatch.setenv("SSN_CONV_SHAPE", shape)
        net = _net(levels, base, 1, H, W)
        out = net.forward(x).cpu().numpy()
        net.backward(t)
        got[shape] = [out, net.get_grads()] + _grads_at(net, 1)
        net.close()
    for a, b in zip(got["0"], got["2"]):
        assert np.array_equal(a, b)
