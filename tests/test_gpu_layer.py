"""GPU parity of the autograd wrapper (BlockCirculantLinear) against the float64 oracle.

The oracle sees only the layer's parameter (float32 first columns), rounded to the
storage type exactly as the wrapper does, and computes its own packed spectra from
them (oracle rdfft, rounded to the storage type); outputs and gradients must match
``oracle.bca`` on those spectra to the storage type's tolerance.
"""

import numpy as np
import pytest
import torch

from oracle import bca as obca
from oracle import rdfft as ord_
from paper_2511_01385_amd import inputs
from paper_2511_01385_amd.layer import BlockCirculantLinear
from tests._helpers import TORCH_DTYPE, assert_close, to_device, to_host_f64

pytestmark = pytest.mark.gpu


def _oracle_spectra(c: torch.Tensor, dtype: str) -> np.ndarray:
    q, kb, p = c.shape
    c_st = inputs.round_to(c.detach().cpu().double().numpy(), dtype)  # what the wrapper feeds rdfft
    spec = ord_.rdfft_forward(inputs.to_f64(c_st, dtype).reshape(q * kb, p))
    return inputs.to_f64(inputs.round_to(spec, dtype), dtype).reshape(q, kb, p)


LAYER_SHAPES = [(dt, *sh) for dt in ("f32", "bf16") for sh in
                [(256, 256, 64, (3, 5)), (512, 1024, 128, (7,)), (768, 256, 256, (2, 3)), (4096, 4096, 512, (3,)),
                 (16384, 16384, 16384, (2, 2))]]
LAYER_SHAPES += [("f16", 256, 256, 64, (3, 5)), ("f16", 768, 768, 256, (4, 3)), ("f16", 16384, 16384, 16384, (2, 2))]
# blocks beyond 8192 with more input than output blocks (one accumulating forward pass per block)
LAYER_SHAPES += [("f32", 32768, 16384, 16384, (3,)), ("bf16", 32768, 32768, 16384, (2, 2))]


@pytest.mark.parametrize("dtype,d_in,d_out,p,lead", LAYER_SHAPES,
                         ids=[f"{s[0]}_{s[1]}x{s[2]}_p{s[3]}" for s in LAYER_SHAPES])
def test_forward_backward_match_oracle(dtype, d_in, d_out, p, lead):
    torch.manual_seed(d_in + d_out + p)
    layer = BlockCirculantLinear(d_in, d_out, p, dtype=TORCH_DTYPE[dtype])
    x_st = inputs.normal_rows(inputs.seed_for(1, salt=d_in + p), int(np.prod(lead)), d_in, dtype)
    g_st = inputs.normal_rows(inputs.seed_for(1, salt=d_out + p + 1), int(np.prod(lead)), d_out, dtype)
    x = to_device(x_st, dtype).reshape(*lead, d_in).requires_grad_(True)
    g = to_device(g_st, dtype).reshape(*lead, d_out)
    g_copy = g.clone()
    y = layer(x)
    y.backward(g)
    torch.cuda.synchronize()
    assert torch.equal(g, g_copy), "the upstream gradient must be left intact by default"

    spec = _oracle_spectra(layer.c, dtype)
    xf, gf = inputs.to_f64(x_st, dtype), inputs.to_f64(g_st, dtype)
    y_ref = obca.forward_spectral(xf, spec, d_out, p)
    dx_ref, dc_ref = obca.backward_spectral(xf, spec, gf, p)
    staged = 2 if p > 8192 else 0  # long blocks store their intermediate spectra
    # The wrapper makes the parameter's spectra itself and rounds them to the storage type from
    # float32; the oracle rounds its own from float64.  Near a tie the two roundings can pick
    # neighbouring values, and a spectrum that differs in one slot changes whole output rows,
    # like one more rounding of a staged spectrum: y and dx get that allowance (dc does not
    # depend on c).
    c_round = 1 if dtype != "f32" else 0
    assert_close(to_host_f64(y.reshape(-1, d_out)), y_ref, dtype, "y", staged + c_round)
    assert_close(to_host_f64(x.grad.reshape(-1, d_in)), dx_ref, dtype, "dx", staged + c_round)
    assert layer.c.grad.dtype == torch.float32
    # long blocks keep a 16-bit layer's intermediate spectra in its storage type: dc meets
    # that type's bar
    dc_bar = dtype if dtype != "f32" and p > 8192 else "f32"
    assert_close(layer.c.grad.double().cpu().numpy().reshape(-1, p), dc_ref.reshape(-1, p), dc_bar, "dc", staged)


def test_clobber_grad_reuses_the_upstream_gradient():
    """clobber_grad=True works in the upstream gradient itself and gives the same results.

    dx is computed token by token with no reduction across workgroups, so it is compared bit
    for bit.  dc is a float32 sum over tokens whose atomic order differs from run to run, so
    each layer's dc is compared with the oracle at the float32 bar instead of with the other's."""
    d, p, tokens, dtype = 256, 64, 9, "bf16"
    torch.manual_seed(5)
    layer = BlockCirculantLinear(d, d, p, dtype=torch.bfloat16, clobber_grad=True)
    layer2 = BlockCirculantLinear(d, d, p, dtype=torch.bfloat16)
    layer2.c.data.copy_(layer.c.data)
    x_st = inputs.normal_rows(inputs.seed_for(1, salt=91), tokens, d, dtype)
    g_st = inputs.normal_rows(inputs.seed_for(1, salt=92), tokens, d, dtype)
    x = to_device(x_st, dtype).requires_grad_(True)
    x2 = to_device(x_st, dtype).requires_grad_(True)
    g = to_device(g_st, dtype)
    layer(x).backward(g)
    layer2(x2).backward(to_device(g_st, dtype))
    torch.cuda.synchronize()
    assert torch.equal(x.grad, x2.grad)
    assert not torch.equal(g, to_device(g_st, dtype)), "clobber_grad=True must work in the upstream gradient"
    spec = _oracle_spectra(layer.c, dtype)
    dx_ref, dc_ref = obca.backward_spectral(inputs.to_f64(x_st, dtype), spec, inputs.to_f64(g_st, dtype), p)
    assert_close(to_host_f64(x.grad), dx_ref, dtype, "dx", 1)  # spectra rounded from float32 (see above)
    for name, lay in (("clobbered", layer), ("copied", layer2)):
        assert_close(lay.c.grad.double().cpu().numpy().reshape(-1, p), dc_ref.reshape(-1, p), "f32", f"dc {name}")


@pytest.mark.parametrize("d_in,d_out,p,tokens", [(768, 768, 256, 2100), (2048, 2048, 1024, 1100), (2048, 512, 128, 2100),
                                                 (64, 64, 16, 5), (512, 256, 32, 9)])
def test_backward_leaves_the_gradient_bits(d_in, d_out, p, tokens):
    """Token counts at which the library would stage its dC sums in a gradient it may overwrite."""
    layer = BlockCirculantLinear(d_in, d_out, p, dtype=torch.bfloat16)
    x = torch.randn(tokens, d_in, device="cuda").bfloat16().requires_grad_(True)
    g = torch.randn(tokens, d_out, device="cuda").bfloat16()
    kept = g.clone()
    layer(x).backward(g)
    dx, dc = x.grad.clone(), layer.c.grad.clone()
    assert torch.equal(g, kept)
    other = BlockCirculantLinear(d_in, d_out, p, dtype=torch.bfloat16, clobber_grad=True)
    other.c.data.copy_(layer.c.data)
    x.grad = None
    other(x).backward(g)
    assert torch.equal(x.grad, dx)
    # dc: float32 sums in another order
    torch.testing.assert_close(other.c.grad, dc, rtol=0, atol=1e-5 * dc.square().mean().sqrt().item() * tokens**0.5)


def test_backward_takes_any_gradient():
    """Gradients that the library itself refuses: a view that starts off its 16-byte grid, x itself, an
    expanded row."""
    d, p = 256, 64
    layer = BlockCirculantLinear(d, d, p, dtype=torch.float32)
    x = torch.randn(6, d, device="cuda").requires_grad_(True)
    room = torch.randn(6 * d + 1, device="cuda")
    for g in (room[1:].view(6, d), x.detach(), room[:d].expand(6, d)):
        want = torch.autograd.grad(layer(x), (x, layer.c), g.clone().contiguous())
        kept = g.clone()
        got = torch.autograd.grad(layer(x), (x, layer.c), g)
        assert torch.equal(g, kept) and torch.equal(got[0], want[0])
        torch.testing.assert_close(got[1], want[1], rtol=1e-5, atol=1e-4)


def test_training_step_reduces_loss():
    # a few SGD steps toward a fixed circulant target: the gradient points downhill
    torch.manual_seed(0)
    target = BlockCirculantLinear(256, 256, 32, dtype=torch.float32)
    layer = BlockCirculantLinear(256, 256, 32, dtype=torch.float32)
    x = torch.randn(64, 256, device="cuda")
    with torch.no_grad():
        t = target(x)
    losses = []
    for _ in range(5):
        layer.c.grad = None
        loss = ((layer(x) - t) ** 2).mean()
        loss.backward()
        with torch.no_grad():
            layer.c -= 0.5 * layer.c.grad
        losses.append(loss.item())
    assert losses[-1] < 0.5 * losses[0]


def test_memory_harness_row():
    from paper_2511_01385_amd import memory_harness

    r = memory_harness.measure(1024, 16, 256, torch.bfloat16)
    # the layer's extra memory: spectra, y, one gradient-sized work buffer and dc, well
    # under a dense weight
    assert 0 < r["peak_bytes"] < r["dense_weight_bytes"]
