"""Values near the ends of fp32 and values that are not finite: where they may and may not show."""
import numpy as np
import pytest

from paper_2506_05233_amd import libmesa as L

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    L.load()
    yield
    torch.cuda.synchronize()


def _bf16(x):
    """fp32 array rounded to the nearest bf16 (ties to even), as fp32."""
    u = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32)
    return ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(np.float32)


@pytest.mark.parametrize("d", [64, 128])
def test_single_pass_states_round_the_weighted_y(d):
    """The single-pass bf16 chunk states are sums of k_i[R] bf16(w_i y_i[c]) with y the key (H) or the
    value (G), rounded to bf16 once.  With one gated token in a chunk the sum is one product of two
    bf16 numbers, exact in fp32, so every stored bit is known: (w, k, y) whose rounding differs if
    the weight goes to the key instead (about a third of the elements) must show it nowhere."""
    T, n = 65, 3
    rng = np.random.default_rng(d)
    k, v = (_bf16(rng.standard_normal((n, T, d))) for _ in range(2))
    beta = np.zeros((n, T), dtype=np.float32)
    at = [0, 37, 63]
    w = np.array([0.7, 0.3, 0.9], dtype=np.float32)
    for b in range(n):
        beta[b, at[b]] = w[b]

    def dev(x, *shape, dtype=torch.float32):
        return torch.from_numpy(np.ascontiguousarray(x)).cuda().to(dtype).reshape(*shape)

    kt, vt = (dev(x, n, 1, T, d, dtype=torch.bfloat16) for x in (k, v))
    gamma, bt = torch.ones((n, 1, T), device="cuda"), dev(beta, n, 1, T)
    need = L.forward_workspace_bytes(n, 1, T, d, d, 64)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    st = L.load().mesa_forward_states(L._ptr(kt), L._ptr(vt), L._ptr(gamma), L._ptr(bt), n, 1, T, d, d,
                                      L.MESA_DTYPE_BF16, 64, L.MESA_PREC_BF16, None, None, L._ptr(ws), need,
                                      L._stream(ws.device))
    assert st == L.MESA_OK
    torch.cuda.synchronize()
    elems = n * 2 * d * d
    raw = ws.cpu().numpy()[:4 * elems].view(np.uint16).astype(np.uint32) << 16
    frags = raw.view(np.float32).reshape(2, n, 2, d // 16, d // 32, 4, 16, 2, 4)  # part, bh, chunk, t, sb, g, m, half, i
    # fragment (t, sb), lane (g, m): rows 32 sb + 16 half + 4 g + i of column 16 t + m
    got = frags.transpose(0, 1, 2, 4, 7, 5, 8, 3, 6).reshape(2, n, 2, d, d)
    assert not got[:, :, 0].any()
    for b in range(n):
        kb, vb = k[b, at[b]], v[b, at[b]]
        for part, y in ((0, kb), (1, vb)):
            want = _bf16(kb[:, None] * _bf16(w[b] * y)[None, :])
            other = _bf16(_bf16(w[b] * kb)[:, None] * y[None, :])
            assert (want != other).mean() > 0.1
            assert np.array_equal(got[part, b, 1], want), (part, b)


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("dk", [64, 128])
def test_decode_few_pairs_large_curvature(dk, packed):
    """p^T A p near and past the largest fp32 number: the kernel for few pairs follows the one for many
    (states aligned to 4 bytes only take that one).  A = s (u u^T + I / 8) with s a power of two: up to
    overflow every CG quantity scales exactly, the solve ends after two iterations, and the outputs
    (G scaled by s too) are those of s = 1; past it alpha = delta / inf = 0 leaves the Jacobi start,
    finite.  The start is up to 8 times the solution and its roundings grow 8 times in the solve (the
    condition of A): 16 roundings of 2^-24 times 64."""
    u = (1.0 + 0.1 * np.cos(np.arange(dk))) / np.sqrt(dk)
    q = u / np.linalg.norm(u) * 0.8  # |q|^2 in [1/2, 2): solved unscaled
    A = np.outer(u, u) + np.eye(dk) / 8
    r = q - A @ (q / np.diag(A))
    top = 126 - int(np.floor(np.log2(r @ A @ r)))  # 2^top p^T A p in [2^126, 2^127)
    G1 = np.random.default_rng(dk).standard_normal((dk, dk))

    def step(e, aligned):
        s = 2.0 ** e

        def place(x):
            x = torch.from_numpy(x.astype(np.float32)).cuda()
            buf = torch.empty(x.numel() + 4, device="cuda")
            at = 0 if aligned else 1
            view = buf[at:at + x.numel()].view(x.shape)
            view.copy_(x)
            return view
        H = torch.from_numpy((s * np.outer(u, u)).astype(np.float32)).cuda().reshape(1, 1, dk, dk)
        H = (L.pack_state(H) if packed else H).cpu().numpy()
        z = torch.zeros((1, 1, dk), device="cuda")
        one = torch.ones((1, 1), device="cuda")
        out = L.decode_step(place(H), place(s * G1.reshape(1, 1, dk, dk)), torch.from_numpy(q.astype(np.float32)).cuda().reshape(1, 1, dk),
                            z, z.clone(), one, one.clone(), torch.full((1, dk), s / 8, device="cuda"), 6, packed=packed)
        torch.cuda.synchronize()
        return out.double().cpu().numpy()

    for e in (0, top - 2, top, top + 1, top + 4):
        few, many = step(e, True), step(e, False)
        assert np.isfinite(many).all(), e
        assert np.isfinite(few).all(), e
        assert np.linalg.norm(few - many) <= 6e-5 * np.linalg.norm(many), e
        if e <= top + 1:
            want = step(0, False)
            assert np.linalg.norm(few - want) <= 6e-5 * np.linalg.norm(want), e


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("dv", [64, 128])
@pytest.mark.parametrize("tile", [1, 2, 3])
def test_value_of_a_later_sub_chunk_stays_out_of_earlier_tokens(tile, dv, dtype):
    """fp32 products, d_k = 64, chunk 64: an infinity or a NaN among the values of one 16-token
    sub-chunk leaves the outputs of every earlier sub-chunk bit for bit as they were."""
    g = torch.Generator(device="cuda").manual_seed(tile + dv)
    n, t = 2, 64
    q, k, v = (torch.randn((1, n, t, d), generator=g, device="cuda").to(dtype) for d in (64, 64, dv))
    gamma, beta = (torch.rand((1, n, t), generator=g, device="cuda") for _ in range(2))
    lam = torch.rand((n, 64), generator=g, device="cuda") + 0.25
    clean = L.forward(q, k, v, gamma, beta, lam, 8, 64, L.MESA_PREC_F32)
    v = v.clone()
    v[0, 0, 16 * tile + 3, 5] = float("nan")
    v[0, 1, 16 * tile, 7] = float("inf")
    got = L.forward(q, k, v, gamma, beta, lam, 8, 64, L.MESA_PREC_F32)
    torch.cuda.synchronize()
    assert torch.equal(got[:, :, :16 * tile], clean[:, :, :16 * tile])
    assert not torch.isfinite(got[0, 0, 16 * tile + 3, 5])


@pytest.mark.parametrize("dk", [64, 128])
@pytest.mark.parametrize("exponent", [120, 126, 127])
def test_jacobi_start_divides(dk, exponent):
    """n_cg = 0, fp32 products: q* = q / diag(H_t + Lambda) also where 1 / diag is below the smallest
    normal number (the quotient of q scaled to |q| near one keeps 2^-19 there: subnormals of 2^-149
    beside elements of q / 8)."""
    t = 70
    g = torch.Generator(device="cuda").manual_seed(dk + exponent)
    q = torch.randn((1, 1, t, dk), generator=g, device="cuda") * 2.0 ** 12
    k, v = (torch.randn((1, 1, t, dk), generator=g, device="cuda") for _ in range(2))
    gamma, beta = torch.ones((1, 1, t), device="cuda"), torch.zeros((1, 1, t), device="cuda")
    lam = torch.full((1, dk), 2.0 ** exponent, device="cuda")
    got = L.forward(q, k, v, gamma, beta, lam, 0, 64, L.MESA_PREC_F32, want_qstar=True)["qstar"]
    want = q.double() / 2.0 ** exponent
    torch.cuda.synchronize()
    assert float((got.double() - want).norm() / want.norm()) <= (1e-7 if exponent == 120 else 2.0 ** -18)


@pytest.mark.parametrize("dk,dv", [(64, 64), (64, 128), (128, 64)])
@pytest.mark.parametrize("v_exp,a_exp", [(-120, 0), (-112, 0), (-104, 0), (100, 0), (120, 0), (0, 100), (0, 110), (0, 120), (-116, 110)])
def test_fp32_products_scale_by_powers_of_two(dk, dv, v_exp, a_exp):
    """fp32 products: values times 2^a scale the outputs by it, and H + Lambda times 2^b (keys times
    2^(b/2)) by 2^(-b/2), to the rounding that is left where numbers reach below 2^-126 (outputs of
    2^-120 beside steps of 2^-149 and solutions of 2^-120 alike: 1e-7; ten times that allowed)."""
    g = torch.Generator(device="cuda").manual_seed(dk + dv)
    n, t = 3, 150
    q, k = (torch.randn((1, n, t, dk), generator=g, device="cuda") for _ in range(2))
    v = torch.randn((1, n, t, dv), generator=g, device="cuda").clamp(-4, 4)
    q, k = q / q.norm(dim=-1, keepdim=True), k / k.norm(dim=-1, keepdim=True)
    gamma, beta = torch.sigmoid(torch.randn((1, n, t), generator=g, device="cuda") + 4), torch.rand((1, n, t), generator=g, device="cuda")
    lam = torch.rand((n, dk), generator=g, device="cuda") + 0.25

    def run(ve, ae):
        out = L.forward(q, k * 2.0 ** (ae // 2), v * 2.0 ** ve, gamma, beta, lam * 2.0 ** ae, 10, 64, L.MESA_PREC_F32)
        return out.double() / 2.0 ** (ve - ae // 2)

    want, got = run(0, 0), run(v_exp, a_exp)
    torch.cuda.synchronize()
    err = float((got - want).norm() / want.norm())
    # outputs of 2^(v_exp - a_exp / 2) below 2^-126 are multiples of 2^-149
    floor = 2.0 ** (-149 - (v_exp - a_exp // 2)) if v_exp - a_exp // 2 < -120 else 0.0
    assert err <= 1e-6 + 4 * floor, err


@pytest.mark.parametrize("dk,dv", [(64, 64), (64, 128), (128, 64)])
@pytest.mark.parametrize("n_cg", [0, 1])
def test_fp32_products_of_a_tiny_system(dk, dv, n_cg):
    """fp32 products: H + Lambda times 2^-116 (keys times 2^-58) scales the outputs by 2^58, elements of H
    of 2^-124 beside steps of 2^-149.  One iteration at most, whose p^T A p is normal (the queries are
    the keys, weighed by at least a half, so that r_0 is nowhere small): Alg. 1 stops below."""
    g = torch.Generator(device="cuda").manual_seed(dk + dv)
    n, t = 3, 150
    k = torch.randn((1, n, t, dk), generator=g, device="cuda")
    v = torch.randn((1, n, t, dv), generator=g, device="cuda")
    k = k / k.norm(dim=-1, keepdim=True)
    gamma = torch.sigmoid(torch.randn((1, n, t), generator=g, device="cuda") + 4)
    beta = 0.5 + 0.5 * torch.rand((1, n, t), generator=g, device="cuda")
    lam = torch.rand((n, dk), generator=g, device="cuda") + 0.25
    want = L.forward(k, k, v, gamma, beta, lam, n_cg, 64, L.MESA_PREC_F32).double()
    got = L.forward(k, k * 2.0 ** -58, v, gamma, beta, lam * 2.0 ** -116, n_cg, 64, L.MESA_PREC_F32).double() * 2.0 ** -58
    torch.cuda.synchronize()
    err = float((got - want).norm() / want.norm())
    assert err <= 1e-6, err


@pytest.mark.parametrize("dk", [64, 128])
def test_fp32_products_of_the_largest_values(dk):
    """One token with values up to the largest finite number: o = beta v (k . q*), finite, to fp32 rounding."""
    dv = 64
    g = torch.Generator(device="cuda").manual_seed(dk)
    q, k = (torch.randn((1, 1, 1, dk), generator=g, device="cuda") for _ in range(2))
    q, k = q / q.norm(), k / k.norm()
    v = torch.linspace(-1, 1, dv, device="cuda", dtype=torch.float64).mul(3.4028234e38).float().reshape(1, 1, 1, dv)
    beta = torch.full((1, 1, 1), 0.5, device="cuda")
    res = L.forward(q, k, v, torch.ones_like(beta), beta, torch.ones((1, dk), device="cuda"), 4, 64, L.MESA_PREC_F32, want_qstar=True)
    torch.cuda.synchronize()
    want = 0.5 * v.double() * (k.double() * res["qstar"].double()).sum()
    assert float((res["out"].double() - want).norm() / want.norm()) <= 1e-6 / abs(float((k.double() * res["qstar"].double()).sum()))


@pytest.mark.parametrize("dtype,prec", [(torch.float32, L.MESA_PREC_F32), (torch.bfloat16, L.MESA_PREC_BF16X3),
                                        (torch.bfloat16, L.MESA_PREC_BF16)])
@pytest.mark.parametrize("t", [32 * 64, 3 * 64])
@pytest.mark.parametrize("gate", [-0.5, float("nan")])
def test_gates_that_are_not_positive_reset(gate, t, dtype, prec):
    """A gate that is negative or NaN resets the states like a zero gate, bit for bit, in the forward
    and its gradients, whichever form the state pass takes (chunk totals and a scan, or a walk)."""
    g = torch.Generator(device="cuda").manual_seed(t)
    n, d = 2, 64
    q, k, v = (torch.randn((1, n, t, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    gamma = 1.0 - 0.01 * torch.rand((1, n, t), generator=g, device="cuda")
    beta = torch.rand((1, n, t), generator=g, device="cuda")
    lam = torch.rand((n, d), generator=g, device="cuda") + 0.25
    dout = torch.randn((1, n, t, d), generator=g, device="cuda")

    def run(value):
        gm = gamma.clone()
        gm[0, 0, t // 3] = value
        f = L.forward(q, k, v, gm, beta, lam, 6, 64, prec, want_qstar=True)
        b = L.backward(k, v, gm, beta, lam, f["qstar"], dout, 6)
        torch.cuda.synchronize()
        return [f["out"], f["qstar"]] + [b[x] for x in ("dq", "dk", "dv", "dgamma", "dbeta", "dlam")]

    for a, b in zip(run(0.0), run(gate)):
        assert torch.isfinite(a).all() and torch.equal(a, b)
