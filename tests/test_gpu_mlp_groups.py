"""The MLP calls over groups of mini-batches large enough to change how the
forward splits d_in (1, 2, 3 or 4 slices, by the number of output tiles) or to
read W1 packed, and
quads with 1-4 mini-batches: every loss against the same batch evaluated by
itself, and sampled ones against the oracle.  And gradients whose workgroups take
one, several or unequal numbers of feature blocks, with every number of unit
groups: sampled mini-batches against the oracle, every loss too."""

import numpy as np
import pytest

import oracle
from oracle.mlp import BF16, Shape
from paper_2211_00889_amd import _lib
from synth import mlp_data
from tests.test_gpu_mlp import _grad_ok

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# A loss is fp32 sums of d_in + hidden bf16 products in two orders: each sum is off
# by at most about sqrt(d_in + hidden) * 2^-24 of its size (1.7e-6 at 896) and the
# loss, 2 to 3, is a difference of logits of that size; eight times that.
TOL_ORDER = 1.5e-5
TOL_BF16 = 1e-2


# (d_in, hidden, batches): tiles = (hidden / 128 rounded up) * quads
@pytest.mark.parametrize("d_in,hidden,batches", [
    (256, 512, 128),   # 128 tiles, 2 slices
    (256, 512, 253),   # 256 tiles, 1 slice, a last quad of one
    (512, 512, 261),   # 264 tiles, 4 slices
    (384, 512, 86),    # 88 tiles, 3 slices of one chunk a half, a last quad of two
    (640, 512, 30),    # 32 tiles, 4 slices of 10 chunks: halves of one and of two
    (896, 512, 125),   # 128 tiles, 2 slices of 14 chunks: halves of three and four
    (1024, 448, 63),   # a half-filled last unit block, a last quad of three
    (1664, 448, 145),  # W1 packed: 148 tiles, 3 slices of 10 steps, uneven halves
    (3072, 64, 260),   # W1 packed: half of the only unit block, 3 slices of 8 steps
])
def test_losses_of_large_groups(d_in, hidden, batches):
    classes, n_samples = 7, 900
    dims = (d_in, hidden, classes)
    A = mlp_data.inputs(3, n_samples, d_in)
    y = mlp_data.teacher_labels(3, A, hidden, classes)
    x0 = mlp_data.student_init(3, d_in, hidden, classes)
    P = _lib.mlp_param_count(*dims)
    prm = torch.zeros(P, dtype=torch.float32, device=DEV)
    prm[:x0.size] = torch.from_numpy(x0.astype(np.float32)).to(DEV)
    data, labels = torch.from_numpy(A).to(DEV), torch.from_numpy(y.astype(np.int32)).to(DEV)
    idx = np.random.default_rng(batches).integers(0, n_samples, size=(batches, 32)).astype(np.int32)
    ws = torch.empty((_lib.mlp_workspace_bytes(*dims, 32 * batches) + 15) // 16 * 4,
                     dtype=torch.float32, device=DEV)
    print(f"[case] losses d_in={d_in} hidden={hidden} batches={batches}", flush=True)
    whole = torch.full((batches,), -1.0, dtype=torch.float32, device=DEV)
    _lib.mlp_loss(prm, dims, data, labels, idx, whole, ws)
    one = torch.full((batches,), -1.0, dtype=torch.float32, device=DEV)
    for k in range(batches):
        _lib.mlp_loss(prm, dims, data, labels, idx[k], one[k:k + 1], ws)
    torch.cuda.synchronize()
    w, o = whole.cpu().numpy(), one.cpu().numpy()
    # Another order may also move a hidden unit over a bf16 rounding boundary: 2^-8 of
    # it at most, which moves that sample's logits by 2^-8 h |W2|, its loss by at most
    # twice that and the mean of 32 by a 32nd; a sample may be in a batch twice
    # (3072x64: three such samples, 1.6e-5 a time)
    W1, b1 = x0[:d_in * hidden].reshape(d_in, hidden), x0[d_in * hidden:(d_in + 1) * hidden]
    W2 = x0[(d_in + 1) * hidden:(d_in + 1) * hidden + hidden * classes]
    flip = 2.0 ** -8 * np.max(A @ W1 + b1) * np.max(np.abs(W2)) * 2 / 32
    assert np.all(np.abs(w - o) <= TOL_ORDER * np.abs(o) + 2 * flip)
    assert np.sum(np.abs(w - o) > TOL_ORDER * np.abs(o)) <= batches // 16  # and rarely
    s = Shape(d_in, hidden, classes, 32)
    for k in (0, batches // 2, batches - 1):
        _, loss = oracle.mlp.grad(x0, A[idx[k]], y[idx[k]], s, BF16)
        assert abs(w[k] - loss) <= TOL_BF16 * abs(loss), k


@pytest.mark.parametrize("d_in,hidden,classes,n,m", [
    (1408, 448, 16, 4, 16),  # 11 feature blocks by threes, a lone last unit group of 7
    (2176, 256, 3, 3, 16),   # 17 blocks by fours, 4 unit groups
    (640, 384, 10, 8, 15),   # 5 blocks in two workgroups, 6 unit groups, two idle waves
    (1024, 64, 5, 16, 20),   # 8 blocks by sixes (the most), one unit group for 8 waves
    (128, 320, 10, 1, 2),    # one block
    (1152, 448, 10, 3, 60),  # W1 packed: three learners, one slice of 9 steps a half
    (3072, 192, 10, 3, 64),  # as long, but the packed W1 would not fit the workspace
])
def test_gradients_of_large_groups(d_in, hidden, classes, n, m):
    n_samples = 700
    dims = (d_in, hidden, classes)
    A = mlp_data.inputs(5, n_samples, d_in)
    y = mlp_data.teacher_labels(5, A, hidden, classes)
    x0 = mlp_data.student_init(5, d_in, hidden, classes)
    rng = np.random.default_rng(d_in + hidden)
    P = _lib.mlp_param_count(*dims)
    X = np.zeros((n, P), np.float32)
    X[:, :x0.size] = x0 + 0.05 * rng.standard_normal((n, x0.size)).astype(np.float32)
    mask = np.ones((n, m), np.uint8)
    mask[n - 1, m // 2] = 0
    idx = rng.integers(0, n_samples, size=(n, m, 32)).astype(np.int32)
    data, labels = torch.from_numpy(A).to(DEV), torch.from_numpy(y.astype(np.int32)).to(DEV)
    G = torch.full((n, m, P), 7.0, dtype=torch.float32, device=DEV)
    losses = torch.full((n * m,), -1.0, dtype=torch.float32, device=DEV)
    ws = torch.empty((_lib.mlp_workspace_bytes(*dims, n * m * 32) + 15) // 16 * 4,
                     dtype=torch.float32, device=DEV)
    print(f"[case] gradients d_in={d_in} hidden={hidden} classes={classes} n={n} m={m}", flush=True)
    _lib.mlp_grad(torch.from_numpy(X).to(DEV), m, dims, data, labels, idx, mask, G, losses, ws)
    torch.cuda.synchronize()
    Lh = losses.cpu().numpy().reshape(n, m)
    s = Shape(d_in, hidden, classes, 32)
    assert (G[n - 1, m // 2] == 7.0).all() and Lh[n - 1, m // 2] == -1.0
    for i, j in {(0, 0), (n // 2, m - 1), (n - 1, 0), (n - 1, m - 1)} - {(n - 1, m // 2)}:
        prm, b = X[i, :s.n_params], idx[i, j]
        g = G[i, j].cpu().numpy()
        assert _grad_ok(g, prm, A[b], y[b], s, dims), (i, j)
        assert (g[s.n_params:] == 0).all()
    for i in range(n):
        for j in range(m):
            if mask[i, j] and (i + j) % 5 == 0:
                _, loss = oracle.mlp.grad(X[i, :s.n_params], A[idx[i, j]], y[idx[i, j]], s, BF16)
                assert abs(Lh[i, j] - loss) <= TOL_BF16 * abs(loss), (i, j)
