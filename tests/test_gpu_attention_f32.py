"""fp32 chunk attention through the layer entry points: block and key-tile
edges (64-query blocks, 32-key tiles, key splits), both head sizes, rows
written directly and through the combine pass, against the oracle at the fp32
tolerance of the parity tests; and a non-finite value row, which the rows
before it must not see."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import workloads as wl  # noqa: E402
from paper_2308_16369_amd import sarathi as S  # noqa: E402
from test_gpu_parity import run_and_check  # noqa: E402


NH = 64   # enough heads that the plan takes the chunk kernel for short chunks too


def _takes_chunk_kernel(hd, offset, length):
    cfg = S.make_cfg(hidden=256, n_heads=NH, head_dim=hd, ffn=264, dtype=S.F32)
    return S.sarathi_attention_plan(cfg, S.make_batch(0, offset, length, [], [])[0])["chunk_items"] > 0


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("offset,length,decodes", [(200, 64, [3]), (231, 65, []), (200, 63, [511, 512]),
                                                   (900, 130, [10]), (0, 300, []), (767, 33, [])])
def test_f32_chunk_edges(hd, offset, length, decodes):
    assert _takes_chunk_kernel(hd, offset, length)
    b = wl.Batch(prefill_slot=1, chunk_offset=offset, chunk_len=length,
                 decode_slots=np.arange(2, 2 + len(decodes), dtype=np.int32), decode_ctx=np.array(decodes, np.int32))
    shape = wl.LayerShape(hidden=256, n_heads=NH, head_dim=hd, ffn=2048, dtype="f32")
    run_and_check(wl.make_instance(shape, b, max_seq_len=1100, n_slots=5, seed=offset + length),
                  f"f32 chunk hd={hd} {length}@{offset}")


def test_f32_chunk_rows_before_a_non_finite_row():
    """Row 40 of a 96-row chunk is infinite: rows 0..39 stay as in the run without it."""
    H, nh, hd, T, seq = 256, NH, 64, 96, 320
    assert _takes_chunk_kernel(hd, 200, T)
    cfg = S.make_cfg(hidden=H, n_heads=nh, head_dim=hd, ffn=264, dtype=S.F32)
    g = torch.Generator(device="cuda").manual_seed(1)
    rnd = lambda *d: torch.empty(*d, device="cuda").normal_(0, 0.05, generator=g)
    w = {"w_qkv": rnd(3 * nh * hd, H), "w_o": rnd(H, nh * hd), "w_up": rnd(2 * 264, H), "w_down": rnd(H, 264),
         "norm1_g": torch.ones(H, device="cuda"), "norm2_g": torch.ones(H, device="cuda")}
    x = rnd(T, H)
    ws_bytes = S.sarathi_workspace_bytes(cfg, T, 0, seq)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    out = []
    for poison in (False, True):
        kv_t = torch.zeros(1, 1, 2, nh, seq, hd, device="cuda")
        kv = S.sarathi_kv_alloc(cfg, 1, seq, kv_t.data_ptr(), kv_t.numel() * 4)
        xin = x.clone()
        if poison:
            xin[40] = float("inf")
        y = torch.empty_like(x)
        batch, keep = S.make_batch(0, 200, T, [], [])
        S.sarathi_hybrid_layer_forward(cfg, S.make_weights({k: t.data_ptr() for k, t in w.items()}), kv, 0, batch,
                                       xin.data_ptr(), y.data_ptr(), ws.data_ptr(), ws_bytes,
                                       torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        out.append(y)
    assert bool(torch.isfinite(out[0]).all()) and not bool(torch.isfinite(out[1][40]).any())
    # one key at a time instead of by matrix products: another summation order
    assert float((out[0][:40] - out[1][:40]).abs().max()) <= 1e-5 * float(out[0].abs().max())
