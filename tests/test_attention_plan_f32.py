"""fp32 attention plan on random single-chunk batches (CPU): its work items and
partial rows stay within what the workspace holds for the smallest cache the
batch fits, so no batch that fits its workspace is refused."""
import random

from paper_2308_16369_amd import sarathi as S


def test_f32_plan_fits_its_workspace():
    rng = random.Random(64)
    taken = set()
    for nh, hd in ((1, 64), (4, 64), (40, 128), (96, 128)):
        cfg = S.make_cfg(hidden=nh * hd, n_heads=nh, head_dim=hd, ffn=256, dtype=S.F32)
        for _ in range(150):
            C = rng.choice([0, 1, 63, 64, 65, rng.randint(2, 300), rng.randint(300, 3000)])
            off = rng.choice([0, rng.randint(1, 600), rng.randint(600, 30000)]) if C else 0
            B = rng.randint(0 if C else 1, 20)
            ctx = [rng.randint(0, 3000) for _ in range(B)]
            batch, keep = S.make_batch(0 if C else -1, off, C, list(range(1, B + 1)), ctx)
            p = S.sarathi_attention_plan(cfg, batch)
            T, seq = C + B, max([off + C] + [c + 1 for c in ctx])
            max_pre, max_dec = -(-T // 256) * -(-seq // 256), T * -(-seq // 512)
            assert 4 * p["chunk_items"] + p["decode_items"] <= 4 * max_pre + max_dec
            assert p["partial_rows_written"] <= 256 * max_pre + max_dec
            assert p["partial_rows_read"] == p["partial_rows_written"]
            splits = sum((c + 512) // 512 for c in ctx)
            if p["chunk_items"]:
                assert p["decode_items"] == splits
            else:       # the chunk's rows one by one, or no chunk
                assert p["decode_items"] == splits + sum((q + 512) // 512 for q in range(off, off + C))
            taken.add((C > 0, p["chunk_items"] > 0))
    assert taken == {(False, False), (True, False), (True, True)}


def test_f32_chunk_or_rows():
    """The two routes' measured ends: 64 rows of 4 heads at 128 cached positions one by one (7.7 us against 16.5), 128
    rows of 40 heads at 256 in blocks (27 us against 164)."""
    cfg = S.make_cfg(hidden=256, n_heads=4, head_dim=64, ffn=688, dtype=S.F32)
    assert S.sarathi_attention_plan(cfg, S.make_batch(0, 128, 64, [], [])[0])["chunk_items"] == 0
    cfg = S.make_cfg(hidden=5120, n_heads=40, head_dim=128, ffn=13824, dtype=S.F32)
    assert S.sarathi_attention_plan(cfg, S.make_batch(0, 256, 128, [], [])[0])["chunk_items"] > 0
