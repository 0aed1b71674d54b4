"""The MLP calls over groups of mini-batches large enough to change how the
forward splits d_in (1, 2, 3 or 4 slices, by the number of output tiles) or to
read W1 packed, and quads with 1-4 mini-batches: every loss, bit for bit, against
the same batch evaluated by itself, and sampled ones against the oracle.
Gradients whose workgroups take one, several or unequal numbers of feature blocks,
with every number of unit groups: sampled mini-batches against the oracle, every
loss too.  And gradients of mini-batches in calls of many and in calls of their own,
bit for bit."""

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
TOL_BF16 = 1e-2


# (d_in, hidden, batches): tiles = (hidden / 128 rounded up) * quads; a batch by
# itself takes as many slices as its d_in has parts (2, 3 or 4)
@pytest.mark.parametrize("d_in,hidden,batches", [
    (128, 512, 40),    # two chunks: one part, one slice
    (256, 512, 128),   # 128 tiles, 2 slices
    (256, 512, 253),   # 256 tiles, 1 slice of two parts, a last quad of one
    (512, 512, 261),   # 264 tiles, 1 slice of four parts
    (384, 512, 86),    # 88 tiles, 1 slice of three parts, a last quad of two
    (640, 512, 30),    # 32 tiles, 4 slices of 10 chunks: leaves of one and of two
    (896, 512, 125),   # 128 tiles, 2 slices of 14 chunks: leaves of one and of two
    (1024, 448, 63),   # a half-filled last unit block, a last quad of three
    (1664, 448, 145),  # W1 packed: 148 tiles, uneven leaves
    (3072, 64, 260),   # W1 packed: half of the only unit block
    (3072, 512, 70),   # W1 packed: 72 tiles, 2 slices of two parts
    (1408, 512, 256),  # W1 packed: 256 tiles, 1 slice of four parts, uneven leaves
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
    w = whole.cpu().numpy()
    assert np.array_equal(w, one.cpu().numpy())
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


@pytest.mark.parametrize("d_in,hidden,classes,n,m", [
    (3072, 512, 10, 4, 24),  # 96 tiles, 2 slices; by themselves 4
    (1408, 448, 10, 8, 20),  # 160 tiles; uneven leaves
    (384, 512, 10, 16, 16),  # 256 tiles, 1 slice of three parts; by themselves 3 slices
    (640, 320, 7, 16, 64),   # more than one launch group: the last entries in another
])
def test_a_mini_batchs_results_do_not_depend_on_the_others(d_in, hidden, classes, n, m):
    """Every mini-batch of the call finished, then only a few of them: the same
    gradients and losses bit for bit, however the launch cuts d_in."""
    n_samples, dims = 600, (d_in, hidden, classes)
    A = mlp_data.inputs(6, n_samples, d_in)
    y = mlp_data.teacher_labels(6, A, hidden, classes)
    x0 = mlp_data.student_init(6, d_in, hidden, classes)
    rng = np.random.default_rng(d_in)
    P = _lib.mlp_param_count(*dims)
    X = np.zeros((n, P), np.float32)
    X[:, :x0.size] = x0 + 0.05 * rng.standard_normal((n, x0.size)).astype(np.float32)
    idx = rng.integers(0, n_samples, size=(n, m, 32)).astype(np.int32)
    data, labels = torch.from_numpy(A).to(DEV), torch.from_numpy(y.astype(np.int32)).to(DEV)
    Xd = torch.from_numpy(X).to(DEV)
    ws = torch.empty((_lib.mlp_workspace_bytes(*dims, n * m * 32) + 15) // 16 * 4,
                     dtype=torch.float32, device=DEV)
    print(f"[case] independence d_in={d_in} hidden={hidden} n={n} m={m}", flush=True)

    def grads(mask):
        G = torch.full((n, m, P), 7.0, dtype=torch.float32, device=DEV)
        losses = torch.full((n, m), -1.0, dtype=torch.float32, device=DEV)
        _lib.mlp_grad(Xd, m, dims, data, labels, idx, mask, G, losses.view(-1), ws)
        return G, losses

    G, losses = grads(np.ones((n, m), np.uint8))
    some = np.zeros((n, m), np.uint8)
    some[0, 0] = some[n // 2, m // 3] = some[n - 1, m - 1] = some[n - 1, m - 2] = 1
    for mask in (some, np.eye(1, n * m, n * m - 1, dtype=np.uint8).reshape(n, m)):
        g, l = grads(mask)
        done = torch.from_numpy(mask.astype(bool)).to(DEV)
        assert torch.equal(g[done], G[done]) and torch.equal(l[done], losses[done])
        assert (g[~done] == 7.0).all() and (l[~done] == -1.0).all()
