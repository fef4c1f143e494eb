"""Training at minibatch sizes that leave remainders: a last workgroup of one sample, a batch of
exactly one workgroup, a last minibatch cut short."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N_PARAMS = 8 * 64 + 64 + 64 * 64 + 64 + 64 * 2 + 2


def samples(m, seed):
    rng = np.random.default_rng(seed)
    X = np.stack([10.0 ** rng.uniform(-4, -2, m), rng.uniform(0.01, 0.99, m), 10.0 ** rng.uniform(3.7, 4.5, m),
                  10.0 ** rng.uniform(-16, -12, m), 10.0 ** rng.uniform(10, 12, m), 10.0 ** rng.uniform(-27, -23, m),
                  rng.uniform(0, 0.5, m), rng.uniform(0, 0.5, m)], 1).astype(np.float32)
    # smooth functions of the inputs, so that more training fits them better
    Y = np.stack([X[:, 1] * (0.6 + 0.3 * X[:, 6]), X[:, 2] * 10.0 ** (0.1 * np.sin(2.0 * np.log10(X[:, 0])))], 1)
    return X, Y.astype(np.float32)


@pytest.mark.parametrize("m,batch", [(1024, 64), (1100, 65), (1500, 100), (2000, 1024), (3000, 129)])
def test_batches_train(arc, m, batch):
    """Deterministic, finite, and better after more epochs, whatever the remainders."""
    import torch

    X, Y = (torch.from_numpy(v).cuda() for v in samples(m, m + batch))
    ctx = arc.Context(0)
    try:
        blobs, reps = [], []
        for epochs in (1, 1, 12):
            net = arc.MLP(ctx)
            reps.append(net.train(X, Y, epochs=epochs, batch=batch, lr=2e-3, seed=5))
            blobs.append(np.frombuffer(net.save()[-4 * N_PARAMS:], np.float32))
            net.close()
    finally:
        ctx.close()
    assert np.array_equal(blobs[0], blobs[1])
    assert np.isfinite(blobs[2]).all()
    assert reps[2]["val_rmse_logt"] < reps[0]["val_rmse_logt"]
