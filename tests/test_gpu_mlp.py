"""GPU parity of the control-variate network kernels against the oracle:
forward pass (four outputs), gradients of the multiplier loss (per-tensor
relative Frobenius error < 1e-3 on the same bf16 operands, with per-sample
multipliers and with the first output alone) and Adam, at batch sizes that
span several 64-sample workgroups and a ragged tail."""
import numpy as np
import pytest
import torch

from gpu_util import announce
from oracle import mlp as omlp
from paper_1501_01405_amd import inputs, mrip

pytestmark = pytest.mark.gpu

NAMES = [n for n, _ in omlp.SHAPES]


def _theta(seed):
    t = inputs.he_uniform_init(seed).astype(np.float64)
    rng = np.random.default_rng(seed + 100)
    d = omlp.unpack(t)
    d = {k: v.copy() for k, v in d.items()}
    for b in ("b1", "b2", "b3"):
        d[b] = rng.normal(0, 0.1, d[b].shape)
    return omlp.pack(d).astype(np.float32)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("n", [1, 63, 64, 200, 1024, 4097])
def test_forward_matches_oracle(gpu, n):
    announce("mlp forward", n)
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, 10)).astype(np.float32)
    theta = _theta(1)
    y = torch.empty((n, mrip.MRIP_MLP_OUT), dtype=torch.float32, device="cuda")
    mrip.mrip_mlp_forward(_dev(theta), _dev(x), n, y, mrip.current_stream())
    torch.cuda.synchronize()
    got = y.cpu().numpy().astype(np.float64)
    ref, _ = omlp.forward(theta, x, bf16=True)
    assert got.shape == ref.shape
    assert np.max(np.abs(got - ref)) <= 2e-3 * max(1.0, np.max(np.abs(ref)))


@pytest.mark.parametrize("n,mult", [(64, True), (777, True), (1024, False), (4096, True),
                                    (1000, False)])
def test_gradient_matches_oracle(gpu, n, mult):
    announce("mlp grad", n, mult)
    rng = np.random.default_rng(7 + n)
    x = rng.normal(size=(n, 10)).astype(np.float32)
    yt = rng.normal(size=n).astype(np.float32)
    z = rng.normal(size=(n, 4)).astype(np.float32) if mult else None
    theta = _theta(2)
    grad = torch.empty(mrip.MRIP_MLP_PARAMS, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    mrip.mrip_mlp_grad(_dev(theta), _dev(x), None if z is None else _dev(z), _dev(yt), n, grad,
                       loss, mrip.current_stream())
    torch.cuda.synchronize()
    g = grad.cpu().numpy().astype(np.float64)
    ref, ref_loss = omlp.backward(theta, x, yt, bf16=True, z=z)
    gd, rd = omlp.unpack(g), omlp.unpack(ref)
    for name in NAMES:
        err = np.linalg.norm(gd[name] - rd[name]) / max(np.linalg.norm(rd[name]), 1e-30)
        assert err < 1e-3, (name, err)
    assert abs(float(loss.cpu()[0]) - ref_loss) <= 1e-4 * ref_loss
    if not mult:  # z = e_0: the other outputs' weights get no gradient
        assert np.all(gd["W3"][1:] == 0.0) and np.all(gd["b3"][1:] == 0.0)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65, 1024, 1025])
def test_gradient_at_the_edges_of_its_tiles(gpu, n):
    # part-filled groups of 16 samples, one and two rows, 16 and 17 partial
    # rows; one bf16 rounding that falls the other way in a layer of 128 units
    # moves a norm by 2^-8 / sqrt(128), 3.5e-4
    announce("mlp grad edges", n)
    rng = np.random.default_rng(70 + n)
    x = rng.normal(size=(n, 10)).astype(np.float32)
    yt = rng.normal(size=n).astype(np.float32)
    z = rng.normal(size=(n, 4)).astype(np.float32)
    theta = _theta(2)
    grad = torch.empty(mrip.MRIP_MLP_PARAMS, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    mrip.mrip_mlp_grad(_dev(theta), _dev(x), _dev(z), _dev(yt), n, grad, loss,
                       mrip.current_stream())
    ref, ref_loss = omlp.backward(theta, x, yt, bf16=True, z=z)
    gd, rd = omlp.unpack(grad.cpu().numpy().astype(np.float64)), omlp.unpack(ref)
    for name in NAMES:
        err = np.linalg.norm(gd[name] - rd[name]) / max(np.linalg.norm(rd[name]), 1e-30)
        assert err < 1e-3, (name, err)
    assert abs(float(loss.cpu()[0]) - ref_loss) <= 1e-4 * ref_loss


@pytest.mark.parametrize("rows", [31, 32, 33, 47, 48, 49, 64, 65])
def test_gradient_over_many_rows(gpu, rows):
    # partial rows around the 32 and 16 that are summed at a time, the last one
    # of a few samples; both entry points sum the same rows in the same order
    announce("mlp grad rows", rows)
    n = 64 * rows - (59 if rows % 2 else 0)
    rng = np.random.default_rng(rows)
    x = rng.normal(size=(n, 10)).astype(np.float32)
    yt = rng.normal(size=n).astype(np.float32)
    z = rng.normal(size=(n, 4)).astype(np.float32)
    theta = _theta(2)
    ref, ref_loss = omlp.backward(theta, x, yt, bf16=True, z=z)
    rd = omlp.unpack(ref)
    args = [_dev(a) for a in (theta, x, z, yt)]
    grads = []
    for call in (mrip.mrip_mlp_grad, mrip.mrip_mlp_grad_noalloc):
        if n > mrip.MRIP_MLP_GRAD_NOALLOC_MAX and call is mrip.mrip_mlp_grad_noalloc:
            continue
        grad = torch.empty(mrip.MRIP_MLP_PARAMS, dtype=torch.float32, device="cuda")
        loss = torch.empty(1, dtype=torch.float32, device="cuda")
        call(*args, n, grad, loss, mrip.current_stream())
        grads.append(grad.cpu().numpy())
        gd = omlp.unpack(grads[-1].astype(np.float64))
        for name in NAMES:  # as at the tiles' edges
            err = np.linalg.norm(gd[name] - rd[name]) / max(np.linalg.norm(rd[name]), 1e-30)
            assert err < 1e-3, (name, err)
        assert abs(float(loss.cpu()[0]) - ref_loss) <= 1e-4 * ref_loss
    assert all(np.array_equal(g, grads[0]) for g in grads)


def test_gradient_of_constant_network_is_bias_only(gpu):
    # W3 = 0: every gradient except dW3 and db3 vanishes; with prediction
    # c = b3 . z, db3_k = 2 mean((c - y) z_k)
    announce("mlp grad constant")
    n = 300
    rng = np.random.default_rng(3)
    x = rng.normal(size=(n, 10)).astype(np.float32)
    yt = rng.normal(size=n).astype(np.float32)
    z = rng.normal(size=(n, 4)).astype(np.float32)
    d = omlp.unpack(_theta(4).astype(np.float64))
    d = {k: v.copy() for k, v in d.items()}
    d["W3"][:] = 0.0
    d["b3"][:] = [0.5, -0.25, 1.0, 0.125]
    theta = omlp.pack(d).astype(np.float32)
    grad = torch.empty(mrip.MRIP_MLP_PARAMS, dtype=torch.float32, device="cuda")
    mrip.mrip_mlp_grad(_dev(theta), _dev(x), _dev(z), _dev(yt), n, grad, None,
                       mrip.current_stream())
    torch.cuda.synchronize()
    gd = omlp.unpack(grad.cpu().numpy().astype(np.float64))
    for name in ("W1", "b1", "W2", "b2"):
        assert np.all(gd[name] == 0.0), name
    z64 = z.astype(np.float64)
    err = z64 @ d["b3"] - yt.astype(np.float64)
    want = 2.0 * (err[:, None] * z64).mean(axis=0)
    assert np.max(np.abs(gd["b3"] - want)) < 1e-5 * max(1.0, np.abs(want).max())


def test_misaligned_output_is_refused(gpu):
    announce("mlp alignment")
    theta = torch.zeros(mrip.MRIP_MLP_PARAMS, dtype=torch.float32, device="cuda")
    x = torch.zeros((4, 10), dtype=torch.float32, device="cuda")
    y = torch.zeros(20, dtype=torch.float32, device="cuda")
    with pytest.raises(mrip.MripError):
        mrip.mrip_mlp_forward(theta, x, 4, y[1:], mrip.current_stream())
    # the weights are read as 16-byte vectors
    t1 = torch.zeros(mrip.MRIP_MLP_PARAMS + 4, dtype=torch.float32, device="cuda")[1:]
    with pytest.raises(mrip.MripError):
        mrip.mrip_mlp_forward(t1, x, 4, y[:16], mrip.current_stream())
    grad = torch.zeros(mrip.MRIP_MLP_PARAMS, dtype=torch.float32, device="cuda")
    yt = torch.zeros(4, dtype=torch.float32, device="cuda")
    with pytest.raises(mrip.MripError):
        mrip.mrip_mlp_grad(t1, x, None, yt, 4, grad, None, mrip.current_stream())
    with pytest.raises(mrip.MripError):
        mrip.mrip_mlp_grad_noalloc(t1, x, None, yt, 4, grad, None, mrip.current_stream())


def test_adam_matches_oracle(gpu):
    announce("adam")
    rng = np.random.default_rng(5)
    p = mrip.MRIP_MLP_PARAMS
    theta = rng.normal(size=p).astype(np.float32)
    m = np.zeros(p, np.float32)
    v = np.zeros(p, np.float32)
    t_d, m_d, v_d = _dev(theta), _dev(m), _dev(v)
    ref_t, ref_m, ref_v = theta.astype(np.float64), m.astype(np.float64), v.astype(np.float64)
    for step in range(1, 6):
        g = rng.normal(size=p).astype(np.float32)
        mrip.mrip_adam_step(t_d, m_d, v_d, _dev(g), p, step, 1e-3, 0.9, 0.999, 1e-8,
                            mrip.current_stream())
        ref_t, ref_m, ref_v = omlp.adam_step(ref_t, ref_m, ref_v, g, step)
    torch.cuda.synchronize()
    assert np.max(np.abs(t_d.cpu().numpy() - ref_t)) < 1e-6
    assert np.max(np.abs(m_d.cpu().numpy() - ref_m)) < 1e-6
