"""The generated noise's bytes against the draws' own: the fused kernel draws in single
precision where that decides a byte, so every byte has to equal the one that the
(double-precision) draws give through Eq. (7).
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(gain_model=1), dict(gain_model=1, k=1.0, theta=1.0), dict(gain_model=1, k=1.5, theta=0.7, scale=0.5),
    dict(gain_model=1, k=64.0, theta=1 / 64.0), dict(gain_model=1, k=1024.0, theta=1 / 1024.0), dict(gain_model=1, k=1025.0, theta=1 / 1025.0), dict(gain_model=1, k=1e6, theta=1e-6),
    dict(gain_model=1, theta=30.0), dict(gain_model=1, theta=float("inf")), dict(gain_model=1, scale=0.0),
    dict(gain_model=2, gain_sd=0.05, mu=0.0, sigma=4.0), dict(gain_model=2, gain_sd=3.0, mu=-20.0, sigma=60.0),
    dict(gain_model=2, gain_sd=4.5, sigma=1e5), dict(gain_model=0), dict(gain_model=0, mu=0.5, sigma=0.0),
    dict(gain_model=0, mu=300.0, sigma=500.0),
])
def test_bytes_are_those_of_the_draws(kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2201_11924_amd.native as nat
    g = torch.Generator(device="cuda").manual_seed(5)
    for W, H, seed in ((1, 1, 0), (257, 3, 1), (1920, 1083, 2), (2048, 2048, 2 ** 41 + 3)):
        img = torch.randint(0, 256, (H, W), generator=g, device="cuda", dtype=torch.uint8)
        out = nat.ir_noise_generate(img, seed=seed, noise_stream=seed % 3, **kw)
        gamma, n = nat.noise_draws(W * H, seed=seed, noise_stream=seed % 3, **kw)
        want = nat.ir_noise(img, gamma.view(H, W), n.view(H, W))
        assert torch.equal(out, want), (W, H, int((out != want).sum()))
