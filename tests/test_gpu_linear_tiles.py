"""Edges of the linear ops' matrix-core kernels through the C-ABI: the large
bf16 tiles (288 x 192, 192 x 256 and 256 x 256) at one to three k-tiles, rows
around the tile height, column counts that are no multiple of four and an output
that is not 16-byte aligned; their tails; the streamed instances of the others;
every fp32 tile at K tails and partial tiles, split and unsplit.

Tolerances: bf16 results are one rounding (2^-9) from an fp32 sum whose terms
the test keeps at |x w| <= ~0.5, so 1e-2 of the largest output; fp32 sums of K
<= 2048 terms are within K^0.5 2^-24 of it per unit, 2e-5 with room."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2308_16369_amd import sarathi as S  # noqa: E402


def _ref(kind, x, w, resid, N):
    z = x.double().cpu() @ w.double().cpu().t()
    if kind == S.LINEAR_SWIGLU:
        return torch.nn.functional.silu(z[:, :N]) * z[:, N:]
    if kind == S.LINEAR_GELU:
        return torch.nn.functional.gelu(z)
    return z + resid.double().cpu() if resid is not None else z


def _inputs(kind, M, N, K, dt, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(M, K, generator=g).to(dt)
    w = (torch.randn(2 * N if kind == S.LINEAR_SWIGLU else N, K, generator=g) * 0.05).to(dt)
    resid = None
    if kind in (S.LINEAR_RESID, S.LINEAR_RESID_F32IN):
        resid = torch.randn(M, N, generator=g).to(dt if kind == S.LINEAR_RESID else torch.float32)
    return x, w, resid


def _err(got, ref):
    return float((got.double().cpu() - ref).abs().max() / ref.abs().max())


KINDS = [S.LINEAR_PLAIN, S.LINEAR_RESID, S.LINEAR_RESID_F32IN, S.LINEAR_SWIGLU, S.LINEAR_GELU]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("mnk", [(1, 4, 64), (255, 260, 128), (257, 515, 192), (193, 129, 448)])
@pytest.mark.parametrize("tile", [(288, 192), (192, 256), (256, 256)])
def test_quad_tile_edges(tile, mnk, shift):
    M, N, K = mnk
    index = [S.sarathi_linear_tile_shape(t) for t in range(S.sarathi_linear_tile_count())].index(tile)
    scratch = torch.empty(S.sarathi_linear_scratch_bytes(M, N), dtype=torch.uint8, device="cuda")
    for kind in KINDS:
        x, w, resid = _inputs(kind, M, N, K, torch.bfloat16, M + N + K + kind)
        xd, wd, rd = x.cuda(), w.cuda(), None if resid is None else resid.cuda()
        odt = torch.float32 if kind == S.LINEAR_RESID else torch.bfloat16
        for n_split in (1, 3) if resid is not None else (1,):
            # one element past the end and before the start stay untouched
            buf = torch.full((M * N + 2 + shift,), 7.0, dtype=odt, device="cuda")
            out = buf[shift:shift + M * N]
            S.sarathi_linear_tiled(kind, M, N, K, xd.data_ptr(), wd.data_ptr(), 0 if rd is None else rd.data_ptr(),
                                   out.data_ptr(), scratch.data_ptr(), scratch.numel(), index, n_split,
                                   torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert _err(out.view(M, N), _ref(kind, x, w, resid, N)) <= 1e-2, (kind, n_split)
            assert bool((buf[:shift] == 7.0).all()) and bool((buf[shift + M * N:] == 7.0).all()), (kind, n_split)


PRODUCER_TILES = [(64, 64), (64, 128), (64, 256), (96, 128), (96, 192), (96, 256), (128, 128), (128, 192), (128, 224),
                  (128, 256), (160, 128), (160, 192), (160, 224), (160, 256)]
STREAMED = 32 << 20   # W of this many bytes and one M-tile: loaded non-temporally, by an instance of its own


@pytest.mark.parametrize("tile", PRODUCER_TILES)
def test_streamed_weights(tile):
    """Every tile with one M-tile over 32 MB of weights, every plain epilogue, unsplit and split."""
    index = [S.sarathi_linear_tile_shape(t) for t in range(S.sarathi_linear_tile_count())].index(tile)
    M, K = tile[0] - 3, 1088
    for kind in KINDS:
        N = 7723 if kind == S.LINEAR_SWIGLU else 15437
        w_rows = 2 * N if kind == S.LINEAR_SWIGLU else N
        assert w_rows * K * 2 >= STREAMED
        g = torch.Generator(device="cuda").manual_seed(M + kind)
        x = torch.empty(M, K, device="cuda").normal_(generator=g).bfloat16()
        w = torch.empty(w_rows, K, device="cuda").normal_(0, 0.05, generator=g).bfloat16()
        z = x.double() @ w.double().t()
        resid = None
        if kind == S.LINEAR_SWIGLU:
            z = torch.nn.functional.silu(z[:, :N]) * z[:, N:]
        elif kind == S.LINEAR_GELU:
            z = torch.nn.functional.gelu(z)
        elif kind in (S.LINEAR_RESID, S.LINEAR_RESID_F32IN):
            resid = torch.empty(M, N, device="cuda").normal_(generator=g)
            resid = resid.bfloat16() if kind == S.LINEAR_RESID else resid
            z += resid.double()
        scratch = torch.empty(S.sarathi_linear_scratch_bytes(M, N), dtype=torch.uint8, device="cuda")
        for n_split in (1, 3) if resid is not None else (1,):
            out = torch.full((M, N), float("nan"), device="cuda",
                             dtype=torch.float32 if kind == S.LINEAR_RESID else torch.bfloat16)
            S.sarathi_linear_tiled(kind, M, N, K, x.data_ptr(), w.data_ptr(), 0 if resid is None else resid.data_ptr(),
                                   out.data_ptr(), scratch.data_ptr(), scratch.numel(), index, n_split,
                                   torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert _err(out, z.cpu()) <= 1e-2, (kind, n_split)


@pytest.mark.parametrize("H,nh,T,tile", [(1536, 29, 5, (64, 64)), (1024, 43, 5, (64, 128)), (512, 129, 5, (64, 256)),
                                         (1024, 43, 70, (96, 128)), (512, 86, 5, (96, 192)), (512, 129, 70, (96, 256)),
                                         (1024, 43, 100, (128, 128)), (512, 86, 100, (128, 192)),
                                         (512, 129, 100, (128, 224)), (1024, 65, 140, (160, 128)),
                                         (512, 86, 140, (160, 192)), (512, 129, 140, (160, 224))])
def test_streamed_weights_rope_layer(H, nh, T, tile):
    """The rotary + KV-append epilogue behind a streamed QKV weight."""
    import numpy as np

    import workloads as wl
    from test_gpu_parity import run_and_check
    assert S.sarathi_linear_plan(S.BF16, S.LINEAR_PLAIN, T, 3 * nh * 128, H, 0)[:2] == tile
    assert T <= tile[0] and 3 * nh * 128 * H * 2 >= STREAMED
    shape = wl.LayerShape(hidden=H, n_heads=nh, head_dim=128, ffn=max(4096, nh * 128), dtype="bf16")
    b = wl.Batch(prefill_slot=0, chunk_offset=17, chunk_len=T - 2, decode_slots=np.array([1, 2], np.int32),
                 decode_ctx=np.array([3, 190], np.int32))
    run_and_check(wl.make_instance(shape, b, max_seq_len=192, n_slots=3, seed=37),
                  f"streamed rope nh={nh} T={T} {tile}")


@pytest.mark.parametrize("mnk", [(33, 65, 40), (97, 129, 104), (161, 1100, 72), (8, 33, 2048), (1030, 260, 136)])
def test_f32_tile_edges(mnk):
    M, N, K = mnk
    scratch = torch.empty(S.sarathi_linear_scratch_bytes(M, N), dtype=torch.uint8, device="cuda")
    for kind in KINDS:
        x, w, resid = _inputs(kind, M, N, K, torch.float32, M + N + K + kind)
        # the last row's and the last weight row's tails end the buffers: what lies behind them is not read as data
        xd = torch.cat([x.flatten(), torch.full((64,), float("nan"))]).cuda()
        wd = torch.cat([w.flatten(), torch.full((64,), float("nan"))]).cuda()
        rd = None if resid is None else resid.cuda()
        out = torch.empty(M, N, dtype=torch.float32, device="cuda")
        for scratch_bytes in (scratch.numel(), 0):
            S.sarathi_linear(S.F32, kind, M, N, K, xd.data_ptr(), wd.data_ptr(), 0 if rd is None else rd.data_ptr(),
                             out.data_ptr(), scratch.data_ptr() if scratch_bytes else 0, scratch_bytes,
                             torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            assert _err(out, _ref(kind, x, w, resid, N)) <= 2e-5, (kind, scratch_bytes)


# (M, N, K, fp32 tile the planner picks): every fp32 tile with a partial M-tile, a partial panel and a short last
# k-tile (K % 32 = 8), two k-tiles (fewer than the ring's stages) and nine (more)
F32_PLAIN = [(5, 33, 40, (32, 32)), (5, 33, 264, (32, 32)), (5, 8201, 40, (32, 64)), (5, 8201, 264, (32, 64)),
             (33, 8201, 40, (64, 64)), (33, 8201, 264, (64, 64)), (65, 8201, 40, (96, 64)), (65, 8201, 264, (96, 64)),
             (97, 8201, 40, (160, 64)), (129, 12001, 264, (160, 64)), (161, 12001, 40, (96, 128)),
             (161, 12001, 264, (96, 128)), (321, 8201, 40, (160, 128)), (290, 15001, 264, (160, 128))]
F32_SWIGLU = [(5, 33, 40, (32, 32)), (5, 33, 264, (32, 32)), (5, 4101, 40, (32, 64)), (5, 4101, 264, (32, 64)),
              (33, 4101, 40, (64, 64)), (33, 4101, 264, (64, 64)), (65, 4101, 40, (96, 64)), (65, 4101, 264, (96, 64)),
              (97, 4101, 40, (160, 64)), (129, 6150, 264, (160, 64)), (65, 8201, 40, (96, 128)),
              (65, 8201, 264, (96, 128)), (129, 8201, 40, (160, 128)), (129, 8201, 264, (160, 128))]
# split over K, the last split short
F32_SPLIT = [(5, 33, 2056, (32, 32)), (5, 2062, 2056, (32, 64)), (33, 2062, 2056, (64, 64)), (65, 2062, 2056, (96, 64)),
             (129, 2062, 2056, (160, 64)), (65, 6150, 2056, (96, 128)), (129, 6150, 2056, (160, 128))]


@pytest.mark.parametrize("kind,split,M,N,K,tile", [
    (kind, split, *case)
    for kinds, split, cases in (([k for k in KINDS if k != S.LINEAR_SWIGLU], False, F32_PLAIN),
                                ([S.LINEAR_SWIGLU], False, F32_SWIGLU),
                                ([S.LINEAR_RESID, S.LINEAR_RESID_F32IN], True, F32_SPLIT))
    for kind in kinds for case in cases])
def test_f32_every_tile(kind, split, M, N, K, tile):
    scratch = torch.empty(S.sarathi_linear_scratch_bytes(M, N) if split else 0, dtype=torch.uint8, device="cuda")
    plan = S.sarathi_linear_plan(S.F32, kind, M, N, K, scratch.numel())
    assert plan[:2] == tile and (plan[2] > 1) == split
    x, w, resid = _inputs(kind, M, N, K, torch.float32, M + N + K + kind)
    xd = torch.cat([x.flatten(), torch.full((64,), float("nan"))]).cuda()
    wd = torch.cat([w.flatten(), torch.full((64,), float("nan"))]).cuda()
    rd = None if resid is None else resid.cuda()
    buf = torch.full((M * N + 64,), 7.0, dtype=torch.float32, device="cuda")
    out = buf[:M * N]
    S.sarathi_linear(S.F32, kind, M, N, K, xd.data_ptr(), wd.data_ptr(), 0 if rd is None else rd.data_ptr(),
                     out.data_ptr(), scratch.data_ptr() if split else 0, scratch.numel(),
                     torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert _err(out.view(M, N), _ref(kind, x, w, resid, N)) <= 2e-5
    assert bool((buf[M * N:] == 7.0).all())


# (hidden, heads, head_dim, rows, preproj tile): the rotary + KV-append epilogue on every fp32 tile, hidden no
# multiple of 32
@pytest.mark.parametrize("H,nh,hd,T,tile", [(264, 1, 64, 5, (32, 32)), (264, 43, 64, 5, (32, 64)),
                                            (264, 43, 64, 33, (64, 64)), (264, 43, 64, 65, (96, 64)),
                                            (264, 57, 64, 129, (160, 64)), (264, 57, 64, 161, (96, 128)),
                                            (264, 57, 128, 129, (160, 128))])
def test_f32_rope_every_tile(H, nh, hd, T, tile):
    import numpy as np

    import workloads as wl
    from test_gpu_parity import run_and_check
    assert S.sarathi_linear_plan(S.F32, S.LINEAR_PLAIN, T, 3 * nh * hd, H, 0)[:2] == tile
    shape = wl.LayerShape(hidden=H, n_heads=nh, head_dim=hd, ffn=1024, dtype="f32")
    b = wl.Batch(prefill_slot=0, chunk_offset=17, chunk_len=T - 2, decode_slots=np.array([1, 2], np.int32),
                 decode_ctx=np.array([3, 190], np.int32))
    run_and_check(wl.make_instance(shape, b, max_seq_len=192, n_slots=3, seed=31), f"f32 rope nh={nh} T={T} {tile}")


@pytest.mark.parametrize("kind,M,N,K", [(S.LINEAR_SWIGLU, 1021, 13824, 1024), (S.LINEAR_SWIGLU, 544, 17920, 1024),
                                        (S.LINEAR_SWIGLU, 1021, 13826, 1024), (S.LINEAR_PLAIN, 1021, 27648, 512),
                                        (S.LINEAR_GELU, 1000, 27660, 512), (S.LINEAR_RESID, 1021, 27648, 512),
                                        (S.LINEAR_RESID, 544, 35842, 512), (S.LINEAR_RESID_F32IN, 1000, 27661, 512),
                                        (S.LINEAR_RESID_F32IN, 544, 35840, 512)])
def test_quad_tail(kind, M, N, K):
    """Shapes whose 256-wide tiles fill one round and a part of the next: the columns left go to 192-wide tiles
    (a last tile that N cuts, N no multiple of 8 or of 4), with every epilogue but the rotary one (below); the
    residual kinds without scratch, so unsplit."""
    assert S.sarathi_linear_plan(S.BF16, kind, M, N, K, 0)[1] == 256
    tail_cols, tail_bn = S.sarathi_linear_plan_tail(S.BF16, kind, M, N, K, 0)
    assert 0 < tail_cols < N and tail_bn == 192
    g = torch.Generator(device="cuda").manual_seed(M + N)
    x = torch.empty(M, K, device="cuda").normal_(generator=g).bfloat16()
    w = torch.empty(2 * N if kind == S.LINEAR_SWIGLU else N, K, device="cuda").normal_(0, 0.05, generator=g).bfloat16()
    resid = None
    if kind in (S.LINEAR_RESID, S.LINEAR_RESID_F32IN):
        resid = torch.empty(M, N, device="cuda").normal_(generator=g)
        if kind == S.LINEAR_RESID:
            resid = resid.bfloat16()
    out = torch.full((M, N), float("nan"), device="cuda",
                     dtype=torch.float32 if kind == S.LINEAR_RESID else torch.bfloat16)
    S.sarathi_linear(S.BF16, kind, M, N, K, x.data_ptr(), w.data_ptr(), 0 if resid is None else resid.data_ptr(),
                     out.data_ptr(), 0, 0, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    z = x.double() @ w.double().t()
    if kind == S.LINEAR_SWIGLU:
        z = torch.nn.functional.silu(z[:, :N]) * z[:, N:]
    elif kind == S.LINEAR_GELU:
        z = torch.nn.functional.gelu(z)
    elif resid is not None:
        z += resid.double()
    assert _err(out, z.cpu()) <= 1e-2


@pytest.mark.parametrize("nh,T,tile,tail", [(72, 1021, (256, 256), (11264, 192)), (73, 700, (192, 256), (11648, 192))])
def test_quad_tail_rope_layer(nh, T, tile, tail):
    """The fused rotary + KV-append epilogue over wide tiles and a tail."""
    import numpy as np

    import workloads as wl
    from test_gpu_parity import run_and_check
    assert S.sarathi_linear_plan(S.BF16, S.LINEAR_PLAIN, T, 3 * nh * 128, 512, 0)[:2] == tile
    assert S.sarathi_linear_plan_tail(S.BF16, S.LINEAR_PLAIN, T, 3 * nh * 128, 512, 0) == tail
    shape = wl.LayerShape(hidden=512, n_heads=nh, head_dim=128, ffn=4096, dtype="bf16")
    b = wl.Batch(prefill_slot=0, chunk_offset=17, chunk_len=T - 21, decode_slots=np.arange(1, 22, dtype=np.int32),
                 decode_ctx=np.array([(53 * i) % 1000 for i in range(1, 22)], np.int32))
    run_and_check(wl.make_instance(shape, b, max_seq_len=1024, n_slots=22, seed=29), f"rope tail T={T}")
