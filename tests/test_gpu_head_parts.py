"""Backward of the head where its sum over the vocabulary is cut into parts, and operands that end inside a tile."""
import pytest

torch = pytest.importorskip("torch")
import armt_synth as S
import paper_2506_05229_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows, vocab", [
    (1, 2047),       # one part
    (65, 2048),      # two parts
    (16, 20011),     # sixteen parts of unequal length, vocabulary not a multiple of 64
    (272, 16640),    # a strip of 16 rows
    (700, 5000),
])
def test_head_backward_parts(dtype, rows, vocab):
    shape = S.get_shape("tiny").replace(d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, d_ff=512, n_mem=16, dtype=dtype)
    act = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(rows + vocab)
    normal = lambda *dims: torch.randn(*dims, device="cuda", generator=gen)
    gain, w = (1 + 0.1 * normal(256)).to(act), (0.05 * normal(vocab, 256)).to(act)
    hidden, d_logits = normal(rows, 256).to(act), normal(rows, vocab) / rows
    ends = P.TokenEnds(shape, torch.zeros(1, 256, dtype=act, device="cuda"), gain, w)
    got = ends.logits_backward(hidden, d_logits)
    leaves = [t.double().requires_grad_() for t in (hidden, gain, w)]
    h, g, wd = leaves
    n = h * torch.rsqrt((h * h).mean(-1, keepdim=True) + shape.rms_eps) * g
    want = torch.autograd.grad(n @ wd.T, leaves, d_logits.double())
    # bf16: d_logits and the normalised rows are rounded once (2^-9 each) in front of the products; fp32: sums of up to
    # 20011 products, whose rounding errors add up like a random walk (2^-24 sqrt(20011) = 8e-6)
    tol = 2.0 ** -8 if dtype == "bf16" else 3e-5
    for a, b in zip(got, want):
        assert (a.double() - b).norm() <= tol * b.norm()
