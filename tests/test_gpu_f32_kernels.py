"""The fp32 grouped GEMM and the delta rule with fewer than 16 memory tokens at the sizes where their tiles, K shares and
vector loads end."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import armt_synth as S
import paper_2506_05229_amd as P
from oracle import armt_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g, M, N, K, shift", [
    (1, 1, 1, 1, 0),
    (2, 16, 32, 16, 0),         # 16-row tile, one chunk of K: three waves without work
    (1, 17, 33, 60, 0),         # one row and column into the next tile, K ends inside a chunk
    (3, 31, 160, 67, 0),        # K not a multiple of 4: element-wise reads
    (2, 72, 128, 512, 0),
    (2, 72, 128, 512, 1),       # rows that start 4 bytes past a 16-byte boundary
    (1, 33, 40, 2116, 0),       # shares of 33 chunks: several batches and a partial one
    (4, 700, 1000, 333, 0),     # many tiles of rows that are not multiples of 16 bytes
])
def test_f32_gemm(g, M, N, K, shift):
    gen = torch.Generator(device="cuda").manual_seed(M * N + K)

    def mat(r, c):
        return torch.randn(r * c + shift, device="cuda", generator=gen)[shift:].view(r, c)

    a, b = [mat(M, K) for _ in range(g)], [mat(N, K) for _ in range(g)]
    out = P.grouped_gemm(a, b, [torch.full((M, N), float("nan"), device="cuda") for _ in range(g)])
    for i in range(g):
        want = a[i].double() @ b[i].double().T
        # K fp32 products and sums: at most (K + 1) 2^-24 of the sum of the products' magnitudes
        bound = (K + 1) * 2.0 ** -24 * (a[i].double().abs() @ b[i].double().abs().T)
        assert ((out[i].double() - want).abs() <= bound + 1e-30).all(), i


@pytest.mark.parametrize("operand", ["a", "b"])
@pytest.mark.parametrize("K", [60, 192, 320, 2116])     # shares of K that end inside a batch of loads, or K inside a chunk
def test_f32_gemm_infinities(K, operand):
    """One infinity in every row of an operand, at positions spread over all of K: results are +-infinity, and never the NaN of
    an infinity that was read past the end of a share of K and multiplied by zero."""
    M, N = 33, 64
    gen = torch.Generator(device="cuda").manual_seed(K)
    a, b = (torch.randn(r, K, device="cuda", generator=gen) for r in (M, N))
    t = b if operand == "b" else a
    rows = torch.arange(t.shape[0], device="cuda")
    t[rows, rows * (K - 1) // (t.shape[0] - 1)] = float("inf")
    out, = P.grouped_gemm([a], [b])
    want = a.double() @ b.double().T
    assert torch.isinf(want).all() and torch.equal(out.double(), want)


@pytest.mark.parametrize("g, M, N, K", [(4, 700, 1000, 333), (9, 520, 512, 130)])
def test_f32_gemm_bits_do_not_depend_on_the_group(g, M, N, K):
    gen = torch.Generator(device="cuda").manual_seed(K)
    a, b = ([torch.randn(r, K, device="cuda", generator=gen) for _ in range(g)] for r in (M, N))
    for i, t in enumerate(P.grouped_gemm(a, b)):
        assert torch.equal(t, P.grouped_gemm([a[i]], [b[i]])[0]), i


def test_f32_orders_same_bits_with_unaligned_rows():
    """Diagonal, sequential and batched execution are the same recurrence bit for bit, also where the rows of a weight (d_ff = 1002)
    are not multiples of 16 bytes and a diagonal holds many more tiles than a cell."""
    shape = S.get_shape("tiny").replace(n_layers=4, d_model=512, n_heads=8, n_kv_heads=4, head_dim=64, d_ff=1002, seg_len=1032,
                                        n_mem=8, d_mem=32, n_tokens=1032 * 4)
    layers, mem_emb = S.make_weights(shape, seed=1)
    model = P.Armt(shape, layers, mem_emb)
    x = model.embed(np.stack([S.make_embeddings(shape, seed=2 + b) for b in range(2)]))
    diagonal = [t.clone() for t in model.forward(x[0].contiguous(), diagonal=True)]
    for other in (model.forward(x[0].contiguous(), diagonal=False), [t[0] for t in model.forward_batched(x, diagonal=True)]):
        for u, v in zip(diagonal, other):
            assert torch.equal(u, v)


@pytest.mark.parametrize("shift_in, shift_out", [(0, 0), (1, 0), (0, 3), (2, 1)])
@pytest.mark.parametrize("dh", [4, 32, 20])
def test_f32_attention_on_buffers_of_any_alignment(dh, shift_in, shift_out):
    """The entry point asks for no alignment of its fp32 buffers: floats in front of them shift them off 16 bytes."""
    H, Hkv, g = 4, 2, 2
    shape = S.get_shape("tiny").replace(n_layers=g, d_model=H * dh, n_heads=H, n_kv_heads=Hkv, head_dim=dh, seg_len=70, n_mem=5)
    T, steps = shape.T, P.ArmtSteps(shape)
    qkv = np.random.default_rng(dh).standard_normal((g, T, (H + 2 * Hkv) * dh)).astype(np.float32)
    src = torch.zeros(shift_in + qkv.size, device="cuda")[shift_in:].view(qkv.shape)
    src.copy_(torch.from_numpy(qkv))
    room = torch.full((shift_out + g * T * H * dh + 1,), 7.0, device="cuda")
    ptr = lambda t: C.c_void_p(t.data_ptr())
    code = steps.lib.armt_segment_attention(C.byref(steps.cfg), g, ptr(src), ptr(room[shift_out:]), ptr(steps.ws), steps.ws.numel(),
                                            C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert code == 0
    got = room[shift_out:-1].view(g, T, H * dh).cpu().numpy()
    assert (room[:shift_out] == 7.0).all() and room[-1] == 7.0
    for i in range(g):
        q, k, v = (t.reshape(T, -1, dh).astype(np.float64) for t in np.split(qkv[i], [H * dh, (H + Hkv) * dh], axis=1))
        want = O.causal_gqa_attention(O.rope(q, shape.rope_theta), O.rope(k, shape.rope_theta), v).reshape(T, H * dh)
        # averages of up to 75 values of order 1 with weights of sums of dh fp32 products
        assert np.abs(got[i] - want).max() <= 2e-5


@pytest.mark.parametrize("n_mem, d_mem", [(1, 32), (5, 32), (15, 64), (16, 32)])
@pytest.mark.parametrize("d_model", [128, 200])
def test_delta_rule_few_tokens(n_mem, d_mem, d_model):
    g = 3
    shape = S.get_shape("tiny").replace(n_layers=g, d_model=d_model, n_heads=4, n_kv_heads=2, head_dim=d_model // 4, n_mem=n_mem,
                                        d_mem=d_mem)
    rng = np.random.default_rng(n_mem)
    w = [{"wm_k": rng.standard_normal((d_mem, d_model)) * 0.05, "wm_v": rng.standard_normal((d_model, d_model)) * 0.1,
          "wm_b": rng.standard_normal((1, d_model)) * 0.1} for _ in range(g)]
    ym = rng.standard_normal((g, n_mem, d_model))
    A, z = rng.standard_normal((g, d_model, shape.phi)) * 0.1, rng.random((g, shape.phi)) + 0.1
    w = [{k: v.astype(np.float32) for k, v in wi.items()} for wi in w]
    ym, A, z = (t.astype(np.float32) for t in (ym, A, z))
    dev = lambda t: torch.as_tensor(t).cuda()
    Ad, zd = dev(A), dev(z)
    P.ArmtSteps(shape).assoc_update(dev(ym), *[[dev(w[i][f]) for i in range(g)] for f in ("wm_k", "wm_v", "wm_b")], Ad, zd)
    for i in range(g):
        wA, wz = O.assoc_update(*(t[i].astype(np.float64) for t in (ym, A, z)), False,
                                {k: v.astype(np.float64) for k, v in w[i].items()}, shape.assoc_eps, shape.dpfp_nu)
        # sums of d_model and Phi fp32 products, squared once by the feature map
        for got, want in ((Ad[i], wA), (zd[i], wz)):
            assert np.linalg.norm(got.cpu().numpy() - want) <= 1e-5 * np.linalg.norm(want)


@pytest.mark.parametrize("n_mem", [5, 16])
@pytest.mark.parametrize("d_model", [1000, 2048])       # 8 cells: 16 and 32 rows per block; one cell: 8
def test_delta_rule_bits_do_not_depend_on_the_group(n_mem, d_model):
    g = 8
    shape = S.get_shape("tiny").replace(n_layers=g, d_model=d_model, n_heads=4, n_kv_heads=2, head_dim=d_model // 4, n_mem=n_mem,
                                        d_mem=64, seg_len=16)
    gen = torch.Generator(device="cuda").manual_seed(n_mem)
    normal = lambda *dims: torch.randn(*dims, device="cuda", generator=gen)
    w = [[0.05 * normal(r, d_model) for _ in range(g)] for r in (64, d_model, 1)]
    ym, A, z = normal(g, n_mem, d_model), 0.1 * normal(g, d_model, shape.phi), normal(g, shape.phi).abs() + 0.1
    steps = P.ArmtSteps(shape)
    together = steps.assoc_update(ym, *w, A.clone(), z.clone())
    for i in range(g):
        alone = steps.assoc_update(ym[i:i + 1].contiguous(), *[t[i:i + 1] for t in w], A[i:i + 1].clone(), z[i:i + 1].clone())
        assert torch.equal(alone[0][0], together[0][i]) and torch.equal(alone[1][0], together[1][i]), i
