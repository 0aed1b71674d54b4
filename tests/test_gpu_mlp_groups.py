"""The MLP calls over groups of mini-batches large enough to change how the
forward splits d_in (1, 2, 3 or 4 slices, by the number of output tiles), and
quads with 1-4 mini-batches: every loss against the same batch evaluated by
itself, and sampled ones against the oracle."""

import numpy as np
import pytest

import oracle
from oracle.mlp import BF16, Shape
from paper_2211_00889_amd import _lib
from synth import mlp_data

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
    assert np.max(np.abs(w - o) / np.abs(o)) <= TOL_ORDER
    s = Shape(d_in, hidden, classes, 32)
    for k in (0, batches // 2, batches - 1):
        _, loss = oracle.mlp.grad(x0, A[idx[k]], y[idx[k]], s, BF16)
        assert abs(w[k] - loss) <= TOL_BF16 * abs(loss), k
