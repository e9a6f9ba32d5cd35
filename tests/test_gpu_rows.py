"""The products of a pass of up to 8 rows against float64 products of the same half-precision inputs, at the edges of the
layouts over K, of the work-groups' runs of weight rows and of the row counts that are compiled."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


U = 2.0 ** -24          # half a unit of a float32 next to 1


def _normed(x, gain, eps):
    """The RMSNorm in float64, rounded once to half: what the product multiplies.  Second: how far the kernel's halves may be off.
    Its float32 value carries the roundings of K / 256 groups of four squares, the fold over a wave, root, quotient and two
    products, so that values next to a tie may round the other way, by a unit; all others are the same."""
    xd, K = x.double(), x.shape[1]
    y = (xd / (xd.pow(2).mean(dim=1, keepdim=True) + eps).sqrt() * gain.double()).clamp(-65504, 65504)
    off = (K / 512 + 11) * U
    half = lambda v: v.clamp(-65504, 65504).half().double()
    return half(y), half(y.abs() * (1 + off)) - half(y.abs() * (1 - off))


def _room(A, off, W, K):
    """Error bound of every sum A W^T: inputs that rounded the other way, and the float32 roundings of at most K / 64 additions in
    a lane (two for a pair of products) and ten over lanes and waves.  A reference whose norm is not rounded, or rounded twice, is 4
    to 1,300 times beyond it (K = 4,096 to 8)."""
    W = W.double().abs()
    return (0 if off is None else off @ W.T) + (K / 64 + 10) * U * (A.abs() @ W.T)


# K: below, at and above each layout's end (512, 1536, 2048, 4096, 12288, 20480), with masked lanes and without
@pytest.mark.parametrize("M,N,K", [(1, 344, 128), (8, 300, 8), (5, 257, 512), (1, 2048, 1536), (8, 1536, 1536), (3, 515, 520), (6, 344, 1536),
                                   (7, 1000, 1544), (2, 264, 2048), (4, 700, 3584), (3, 4608, 4096), (2, 5, 3592),
                                   (1, 1536, 8960), (8, 1536, 8960), (5, 72, 12288), (4, 3584, 18944), (3, 40, 20480)])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_rows_product(M, N, K, mode):
    import torch
    from paper_2505_24298_amd import binding
    L = binding.lib()
    g = torch.Generator(device="cuda").manual_seed(M * 7 + N + K)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    W0, W1 = (rand(N, K) * 0.05).half(), (rand(N, K) * 0.05).half()
    gain = (rand(K) * 0.1 + 1).half()
    x = rand(M, K) * 3
    if mode == 1:
        x, gain = x.half(), None
    served = K <= 4096 or mode == 1
    assert L.areal_op_rows_serves(M, N, K, mode) == int(served)
    C = rand(M, N)
    base = C.clone()
    if mode == 2:
        C = C.half()
    if not served:
        with pytest.raises(binding.ArealError):
            binding.op_rows_product(x, gain, 1e-6, [W0, W1][:1 + mode // 2], C, mode)
        return
    binding.op_rows_product(x, gain, 1e-6, [W0, W1] if mode == 2 else [W0], C, mode)
    A, off = (x.double(), None) if mode == 1 else _normed(x, gain, 1e-6)
    ref0, ref1 = A @ W0.double().T, A @ W1.double().T
    room0, room1 = _room(A, off, W0, K), _room(A, off, W1, K)
    if mode == 0:
        want, room = ref0, room0
    elif mode == 1:
        want = base.double() + ref0
        room = room0 + U * want.abs()
    else:
        # |silu'| <= 1.1; the exponential and the quotient within 2^-18, one rounding to half
        silu = ref0 / (1 + torch.exp(-ref0))
        want = silu * ref1
        room = 1.1 * room0 * (ref1.abs() + room1) + silu.abs() * room1 + (2.0 ** -11 + 2.0 ** -18) * want.abs() + 2.0 ** -25
    worst = ((C.double() - want).abs() / room).max().item()
    print(f"mode {mode}, {M} x {N} x {K}: {worst:.3f} of the bound", flush=True)
    assert worst <= 1


@pytest.mark.parametrize("M,parts,K", [(m, (1536, 256, 256), 1536) for m in (1, 2, 3, 4, 8)] +
                         [(m, (8, 16, 5), 264) for m in (1, 5, 6, 7, 8)] + [(8, (128, 64, 64), 128), (2, (3584, 512, 512), 3584)])
def test_rows_product_of_three_segments(M, parts, K):
    """The segments' rows as one matrix: the same bits.  Untouched neighbours of C stay."""
    import torch
    from paper_2505_24298_amd import binding
    g = torch.Generator(device="cuda").manual_seed(M + K)
    W = [(torch.randn((p, K), generator=g, device="cuda") * 0.05).half() for p in parts]
    x, gain = torch.randn((M, K), generator=g, device="cuda"), torch.ones(K, device="cuda").half()
    N = sum(parts)
    buf = torch.full((M + 1, N), 7.0, device="cuda")
    one = torch.empty((M, N), device="cuda")
    binding.op_rows_product(x, gain, 1e-6, W, buf[:M], 0)
    binding.op_rows_product(x, gain, 1e-6, [torch.cat(W)], one, 0)
    assert torch.equal(buf[:M], one) and (buf[M] == 7.0).all()


def test_rows_product_takes_subnormal_halves_and_saturates():
    """Products of subnormal halves count, as on the matrix cores; a normalised value beyond the half range is its largest."""
    import torch
    from paper_2505_24298_amd import binding
    K, N = 1536, 64
    W = torch.full((N, K), 2.0 ** -24, device="cuda").half()             # the smallest subnormal
    x = torch.full((1, K), 1.5, device="cuda").half()
    C = torch.zeros((1, N), device="cuda")
    binding.op_rows_product(x, None, 0.0, [W], C, 1)
    assert np.allclose(C.cpu().numpy(), K * 1.5 * 2.0 ** -24, rtol=1e-6)
    xf = torch.zeros((1, K), device="cuda")
    xf[0, 0] = 100.0                                                     # normalised: sqrt(K) = 39.2
    gain = torch.full((K,), 60000.0, device="cuda").half()
    binding.op_rows_product(xf, gain, 0.0, [torch.ones((N, K), device="cuda").half()], C, 0)
    assert (C == 65504.0).all()


@pytest.mark.parametrize("M,N,K", [(9, 64, 128), (0, 64, 128), (1, 64, 100), (1, 64, 20488), (5, 64, 3584), (5, 64, 12296), (1, 16385, 128)])
def test_rows_product_refuses(M, N, K):
    from paper_2505_24298_amd import binding
    L = binding.lib()
    assert L.areal_op_rows_serves(M, N, K, 1) == 0
    assert L.areal_op_rows_product(None, 16, None, 0.0, 16, None, None, N, N, 16, M, N, K, 1) != 0


@pytest.mark.parametrize("M,N,K", [(1, 151936, 64), (4, 32003, 1536), (8, 163840, 8)])
def test_rows_product_of_many_outputs(M, N, K):
    """The output projection: as many rounds as the sums in LDS hold; one more is refused."""
    import torch
    from paper_2505_24298_amd import binding
    g = torch.Generator(device="cuda").manual_seed(N)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.05).half()
    x, gain = torch.randn((M, K), generator=g, device="cuda"), torch.ones(K, device="cuda").half()
    C = torch.empty((M, N), device="cuda")
    binding.op_rows_product(x, gain, 1e-6, [W], C, 0)
    A, off = _normed(x, gain, 1e-6)
    assert ((C.double() - A @ W.double().T).abs() <= _room(A, off, W, K)).all()
    assert binding.lib().areal_op_rows_serves(M, 163841, K, 0) == 0
