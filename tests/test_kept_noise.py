"""What a fitting step holds between forward and backward: noise spectra up to a bound, then none."""

import os
import threading

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2509_08675_amd", "libhufield.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libhufield.so not built")


@pytest.fixture()
def hf(monkeypatch):
    from paper_2509_08675_amd import hufield
    monkeypatch.setattr(hufield, "_kept_noise", hufield._KeptNoise())
    return hufield


def test_the_bound_counts_tensors_while_they_live(hf, monkeypatch):
    monkeypatch.setattr(hf, "NOISE_KEEP_BYTES", 2500)
    cpu = torch.device("cpu")

    class Keeps(torch.autograd.Function):
        kept = []

        @staticmethod
        def forward(ctx, x):
            noise = torch.zeros(1000, dtype=torch.uint8)
            keep = hf._kept_noise.keep(noise)
            Keeps.kept.append(keep)
            ctx.save_for_backward(noise if keep else None)
            return x * 2

        @staticmethod
        def backward(ctx, g):
            return g * 2

    x = torch.ones(2, requires_grad=True)
    y = [Keeps.apply(x) for _ in range(3)]
    assert Keeps.kept == [True, True, False] and hf._kept_noise.held(cpu) == 2000
    y[0].sum().backward()                            # its saved tensor goes with the backward pass
    assert hf._kept_noise.held(cpu) == 1000
    y[1].sum().backward(retain_graph=True)           # ... or stays for another one
    assert hf._kept_noise.held(cpu) == 1000
    del y
    assert hf._kept_noise.held(cpu) == 0
    Keeps.apply(x)                                   # dropped without a backward pass
    assert Keeps.kept[-1] and hf._kept_noise.held(cpu) == 0


def test_the_bound_holds_with_several_threads(hf, monkeypatch):
    monkeypatch.setattr(hf, "NOISE_KEEP_BYTES", 5000)
    over = []

    def work():
        for _ in range(300):
            t = torch.zeros(1000, dtype=torch.uint8)
            if hf._kept_noise.keep(t) and hf._kept_noise.held(t.device) > 5000:
                over.append(1)
            del t

    threads = [threading.Thread(target=work) for _ in range(8)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not over and hf._kept_noise.held(torch.device("cpu")) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("dims", [(64, 96), (32, 24, 48)])
def test_steps_beyond_the_bound_give_the_same_bits(hf, monkeypatch, dims):
    print("fitting steps beyond the bound", dims, flush=True)
    target = dict(p=4.0, semi=(1.0, 1.5, 2.0), rot=0.0, alpha=4.0, k0=0.25, width=0.05, sigma_f=1.0)
    one = hf.workspace_size(hf.HU_OP_NOISE, dims, 1, (12, 1))

    def grads(bytes_kept):
        monkeypatch.setattr(hf, "NOISE_KEEP_BYTES", bytes_kept)
        theta = torch.tensor([1.5, 1.0, 1.0, 2.0, 0.3, 0.22, 0.06], dtype=torch.float64, device="cuda", requires_grad=True)
        loss = sum(hf.spectrum_loss(theta, dims, s, 12, target, alpha=2.0) for s in (3, 4, 5))
        held = hf._kept_noise.held(loss.device)
        P = hf.FilterSpectrum.apply(theta, dims, 6, (12, 1), 2.0)
        g, = torch.autograd.grad(loss + P.sum(), theta)
        del loss, P
        return g, held

    a, held = grads(1 << 30)
    assert held == 3 * one
    for kept in (one, 0):
        b, held = grads(kept)
        assert held == kept and torch.equal(a, b)
    assert hf._kept_noise.held(a.device) == 0


@pytest.mark.gpu
def test_memory_of_a_loss_over_many_seeds(hf, monkeypatch):
    print("memory of a loss over many seeds", flush=True)
    dims = (64, 64, 64)
    one = hf.workspace_size(hf.HU_OP_NOISE, dims, 1, (16, 1))
    monkeypatch.setattr(hf, "NOISE_KEEP_BYTES", 2 * one)
    target = dict(p=4.0, semi=(1.0, 1.5, 2.0), rot=0.0, alpha=4.0, k0=0.25, width=0.05, sigma_f=1.0)
    theta = torch.tensor([1.5, 1.0, 1.0, 2.0, 0.3, 0.22, 0.06], dtype=torch.float64, device="cuda", requires_grad=True)
    hf.spectrum_loss(theta, dims, 1, 16, target, alpha=2.0).backward()
    m0 = torch.cuda.memory_allocated()
    loss = sum(hf.spectrum_loss(theta, dims, s, 16, target, alpha=2.0) for s in range(20))
    assert torch.cuda.memory_allocated() - m0 < 4 * one
    loss.backward()
    assert torch.isfinite(theta.grad).all()
