"""GPU training of the launch predictor against the same epochs made of the
single calls (forward, loss, backward, Adam): the fused passes add in the same
order, so parameters, moments and losses agree bit for bit. Batches around the
edges of a workgroup's 16 samples and a wavefront's two, and more workgroups
than a thread of the gradient sum has loads in flight (48)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NP, IN, H, K = 6816, 8, 64, 32


@pytest.mark.parametrize("batch", [1, 3, 4, 5, 16, 17, 31, 48 * 16, 48 * 16 + 1, 4400])
def test_training_equals_single_calls_bitwise(gfx, batch):
    import torch
    rng = np.random.default_rng(batch)
    new = lambda a: torch.from_numpy(np.asarray(a, np.float32)).cuda()
    start = rng.standard_normal(NP) * 0.2
    f, tgt = new(rng.standard_normal((batch, IN))), new(rng.random((batch, K)))
    mask = new(rng.random((batch, K)) < 0.9)
    inv, epochs, lr = 1.0 / (batch * K), 3, 3e-3

    p, m, v, hist = new(start), torch.zeros(NP, device="cuda"), torch.zeros(NP, device="cuda"), torch.zeros(epochs, device="cuda")
    gfx.train_predictor(p, m, v, f, tgt, mask, batch, inv, epochs, lr, hist)

    q, mq, vq, hq = new(start), torch.zeros(NP, device="cuda"), torch.zeros(NP, device="cuda"), torch.zeros(epochs, device="cuda")
    y, g = torch.zeros(batch, K, device="cuda"), torch.zeros(NP, device="cuda")
    z1, z2 = torch.zeros(batch, H, device="cuda"), torch.zeros(batch, H, device="cuda")
    for e in range(epochs):
        gfx.mlp_forward(q, f, batch, y, z1, z2)
        gfx.mlp_loss(y, tgt, mask, batch * K, inv, hq[e:])
        gfx.mlp_backward(q, f, z1, z2, y, tgt, mask, batch, inv, g)
        gfx.adam_step(q, g, mq, vq, NP, lr, 0.9, 0.999, 1e-8, e + 1)
    torch.cuda.synchronize()
    for a, b in ((p, q), (m, mq), (v, vq), (hist, hq)):
        assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.mark.parametrize("batch", [7, 8, 255, 4095, 4096, 4097, 50001])
def test_loss_alone_and_in_training_bitwise(gfx, batch):
    """The loss call sums with four wavefronts per part, training with one:
    the same sum, at counts around a turn (8,192 elements) and a trip of
    sixteen, and close to the sum in 64 bits (each of at most 300 terms in a
    strand and 14 halvings and parts rounds once: 2^-24 * 320 of the sum)."""
    import torch
    rng = np.random.default_rng(batch)
    new = lambda a: torch.from_numpy(np.asarray(a, np.float32)).cuda()
    p, f, tgt = new(rng.standard_normal(NP) * 0.2), new(rng.standard_normal((batch, IN))), new(rng.random((batch, K)))
    mask = new(rng.random((batch, K)) < 0.9)
    inv = 1.0 / (batch * K)
    y, loss = torch.zeros(batch, K, device="cuda"), torch.zeros(2, device="cuda")
    gfx.mlp_forward(p, f, batch, y)
    gfx.mlp_loss(y, tgt, mask, batch * K, inv, loss)
    gfx.train_predictor(p, torch.zeros(NP, device="cuda"), torch.zeros(NP, device="cuda"), f, tgt, mask, batch, inv, 1,
                        1e-3, loss[1:])
    torch.cuda.synchronize()
    assert loss[0] == loss[1]
    d = y.double().cpu().numpy() - tgt.double().cpu().numpy()
    ref = float((mask.double().cpu().numpy() * d * d).sum() * np.float64(np.float32(inv)))
    assert abs(float(loss[0]) - ref) <= 2.0 ** -24 * 320 * ref
