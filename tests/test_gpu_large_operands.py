"""Operands of 4 GiB and more, past the 32-bit row offsets of the matrix-core
matmuls: the kernels that take them instead, fp32 and bf16, and an fp32 layer
whose QKV weight is that large (its rotary embedding and KV append then run as
a pass of their own).  Compared with float64 on the GPU, on the first, the last
and some rows and columns between.

Tolerances: bf16 results one rounding from an fp32 sum, 1e-2 of the largest
output; fp32 sums of up to 8192 terms 2e-5, the one of 2 million 2e-4 (about
K^0.5 2^-24 per split, with room); the fp32 layer 1e-4 as in the parity tests."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2308_16369_amd import sarathi as S  # noqa: E402

GIB4 = 1 << 32


def _some(n, g):
    """First and last 70 of n, and 60 between."""
    if n <= 200:
        return torch.arange(n, device="cuda")
    between = torch.randint(70, n - 70, (60,), generator=g, device="cuda")
    return torch.cat([torch.arange(70, device="cuda"), between, torch.arange(n - 70, n, device="cuda")])


@pytest.mark.parametrize("dtype,kind,M,N,K,tol", [
    (S.F32, S.LINEAR_PLAIN, 3, 262152, 4096, 2e-5), (S.F32, S.LINEAR_GELU, 65, 131080, 8192, 2e-5),
    (S.F32, S.LINEAR_SWIGLU, 3, 131080, 4096, 2e-5), (S.F32, S.LINEAR_RESID, 131080, 40, 8192, 2e-5),
    (S.F32, S.LINEAR_RESID_F32IN, 3, 512, 2097160, 2e-4),   # split over K
    (S.BF16, S.LINEAR_PLAIN, 3, 262152, 8192, 1e-2), (S.BF16, S.LINEAR_SWIGLU, 70, 131080, 8192, 1e-2),
    (S.BF16, S.LINEAR_RESID, 262152, 40, 8192, 1e-2), (S.BF16, S.LINEAR_RESID_F32IN, 3, 1024, 2097216, 1e-2)])
def test_linear_past_4gib(dtype, kind, M, N, K, tol):
    dt = torch.float32 if dtype == S.F32 else torch.bfloat16
    w_rows = 2 * N if kind == S.LINEAR_SWIGLU else N
    es = 4 if dtype == S.F32 else 2
    assert max(M, w_rows) * K * es >= GIB4
    g = torch.Generator(device="cuda").manual_seed(M + N)
    x = torch.empty(M, K, device="cuda", dtype=dt).normal_(0, 1, generator=g)
    w = torch.empty(w_rows, K, device="cuda", dtype=dt).normal_(0, 0.05, generator=g)
    resid_kind = kind in (S.LINEAR_RESID, S.LINEAR_RESID_F32IN)
    rdt = dt if kind == S.LINEAR_RESID else torch.float32
    resid = torch.empty(M, N, device="cuda", dtype=rdt).normal_(0, 1, generator=g) if resid_kind else None
    odt = torch.float32 if kind == S.LINEAR_RESID else dt
    out = torch.full((M, N), float("nan"), device="cuda", dtype=odt)
    scratch = torch.empty(S.sarathi_linear_scratch_bytes(M, N) if resid_kind else 0, device="cuda", dtype=torch.uint8)
    S.sarathi_linear(dtype, kind, M, N, K, x.data_ptr(), w.data_ptr(), resid.data_ptr() if resid_kind else 0,
                     out.data_ptr(), scratch.data_ptr() if resid_kind else 0, scratch.numel(),
                     torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out).all())
    r, c = _some(M, g), _some(N, g)
    xs = x[r].double()
    z = xs @ w[c].double().t()
    if kind == S.LINEAR_SWIGLU:
        z = torch.nn.functional.silu(z) * (xs @ w[N + c].double().t())
    elif kind == S.LINEAR_GELU:
        z = torch.nn.functional.gelu(z)
    elif resid_kind:
        z += resid[r][:, c].double()
    assert float((out[r][:, c].double() - z).abs().max() / z.abs().max()) <= tol


def test_f32_layer_with_a_qkv_weight_past_4gib():
    H, nh, hd, F, seq, base = 12288, 228, 128, 8, 40, 10000.0
    QD = nh * hd
    assert 3 * QD * H * 4 >= GIB4
    cfg = S.make_cfg(hidden=H, n_heads=nh, head_dim=hd, ffn=F, norm=S.NORM_RMS, act=S.ACT_SWIGLU, rope=1,
                     rope_base=base, eps=1e-6, dtype=S.F32)
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *d, m=0.0, s=0.02: torch.empty(*d, device="cuda").normal_(m, s, generator=g)
    w = {"w_qkv": rnd(3 * QD, H), "w_o": rnd(H, QD), "w_up": rnd(2 * F, H), "w_down": rnd(H, F),
         "norm1_g": rnd(H, m=1.0), "norm2_g": rnd(H, m=1.0)}
    rows = [(1, 30), (1, 31), (1, 32), (0, 7), (2, 39)]     # (slot, position): a chunk of three and two decodes
    x = rnd(len(rows), H, s=1.0)
    kv_t = rnd(1, 3, 2, nh, seq, hd, s=1.0)
    before = kv_t.clone()
    kv = S.sarathi_kv_alloc(cfg, 3, seq, kv_t.data_ptr(), kv_t.numel() * 4)
    batch, keep = S.make_batch(1, 30, 3, [0, 2], [7, 39])
    ws_bytes = S.sarathi_workspace_bytes(cfg, len(rows), 2, seq)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    y = torch.empty_like(x)
    S.sarathi_hybrid_layer_forward(cfg, S.make_weights({k: t.data_ptr() for k, t in w.items()}), kv, 0, batch,
                                   x.data_ptr(), y.data_ptr(), ws.data_ptr(), ws_bytes,
                                   torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()

    d = lambda t: t.double()
    norm = lambda v, gain: v / torch.sqrt((v * v).mean(-1, keepdim=True) + 1e-6) * d(gain)
    a = norm(d(x), w["norm1_g"])
    q, k, v = ((a @ d(w["w_qkv"][i * QD:(i + 1) * QD]).t()).view(-1, nh, hd) for i in range(3))
    pos = torch.tensor([p for _, p in rows], device="cuda", dtype=torch.float64)
    ang = pos[:, None] * base ** (-2.0 * torch.arange(hd // 2, device="cuda", dtype=torch.float64) / hd)
    cs, sn = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    rot = lambda t: torch.cat([t[..., :64] * cs - t[..., 64:] * sn, t[..., :64] * sn + t[..., 64:] * cs], -1)
    q, k = rot(q), rot(k)
    cache = d(before)
    for i, (s, p) in enumerate(rows):
        cache[0, s, 0, :, p], cache[0, s, 1, :, p] = k[i], v[i]
    o = torch.stack([(torch.softmax((q[i][:, None] * cache[0, s, 0, :, :p + 1]).sum(-1) / hd ** 0.5, -1)[..., None]
                      * cache[0, s, 1, :, :p + 1]).sum(1) for i, (s, p) in enumerate(rows)])
    h = d(x) + o.reshape(len(rows), QD) @ d(w["w_o"]).t()
    z = norm(h, w["norm2_g"]) @ d(w["w_up"]).t()
    ref = h + (torch.nn.functional.silu(z[:, :F]) * z[:, F:]) @ d(w["w_down"]).t()
    assert float((d(y) - ref).abs().max() / ref.abs().max()) <= 1e-4
    changed = torch.zeros_like(kv_t, dtype=torch.bool)
    for i, (s, p) in enumerate(rows):
        changed[0, s, :, :, p] = True
        for got, want in ((kv_t[0, s, 0, :, p], k[i]), (kv_t[0, s, 1, :, p], v[i])):
            assert float((d(got) - want).abs().max() / want.abs().max()) <= 1e-4
    assert torch.equal(kv_t[~changed], before[~changed])
