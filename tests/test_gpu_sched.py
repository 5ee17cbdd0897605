"""Work-list edges of the persistent scheduler against the naive grid.

Whatever way items reach the workgroups (by their index alone when there are
no more items than workgroups; else a first item by index and later ones from
the queue counters), every row must be run exactly once: with few enough kept
blocks that no row is split, the persistent launch equals the naive grid bit
for bit, and rows left out would keep the NaN that the output starts with.
Short rows that all fit on the device take the naive grid by themselves; more
than 32 blocks or more than 512 rows reach the work list. Shapes that take the
naive grid are compared with the same heads repeated until they no longer do:
more rows, on the work list, each wave with two query tiles.
"""

import numpy as np
import pytest

from oracle.compare import ATTN_MAX_ABS

from _gpu_util import custom_config, geometry_of, lib, tiling_of, to_dev, torch_mod, work_list_heads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize(
    "heads,grid,tile",
    [
        (1, (1, 8, 8), (1, 8, 8)),  # one row
        (8, (8, 16, 32), (2, 8, 8)),  # 256 full rows: the most that run on eight waves each
        (16, (1, 64, 32), (1, 8, 8)),  # 512 rows of 32 blocks: the last without a work list
        (1, (1, 8, 264), (1, 8, 8)),  # 33 rows of 33 blocks: the first with one
        (3, (1, 8, 280), (1, 8, 8)),  # 105 rows, uneven queues
        (12, (2, 16, 168), (2, 8, 8)),  # 504 rows: nearly every workgroup has its own
        (40, (1, 16, 52), (1, 8, 8)),  # 560 rows: counters
        (160, (2, 8, 40), (2, 8, 8)),  # 800 rows of five blocks
    ],
)
def test_every_item_runs_once(heads, grid, tile):
    torch, fva = torch_mod(), lib()
    cfg = custom_config("sched", heads, grid, tile, np.linspace(0.3, 5.0, heads), seed=61)
    geo = geometry_of(cfg)
    rng = np.random.default_rng(62)
    q, k, v = (torch.randn((1, heads, cfg.N, 128), generator=torch.Generator().manual_seed(63 + i)).bfloat16().cuda()
               for i in range(3))
    # uneven rows, some empty (an empty row's output is zero)
    mask = (rng.random((1, heads, geo.nb, geo.nb)) < rng.random((1, heads, geo.nb, 1))).astype(np.uint8)
    mask[np.cumsum(mask, -1) > 32] = 0  # the smallest automatic chunk: nothing is split
    m = torch.from_numpy(mask).cuda()
    want = fva.fva_attn(q, k, v, tiling_of(cfg), m, flags=fva.FVA_SCHED_NAIVE)
    calls = [(1, (q, k, v, m))]
    if geo.nb <= 32 and heads * geo.nb <= 512:
        calls.append(work_list_heads(heads * geo.nb, q, k, v, m))
    for n, (qn, kn, vn, mn) in calls:
        for flags in (0, fva.FVA_SCHED_UNPAIRED):
            out = torch.full_like(qn, float("nan"))
            fva.fva_attn(qn, kn, vn, tiling_of(cfg), mn, flags=flags, out=out)
            assert torch.equal(out, want.repeat(1, n, 1, 1))


@pytest.mark.parametrize(
    "heads,grid,tile,split",
    [
        (3, (1, 64, 64), (1, 8, 8), 0),  # nb 64: one whole round of rows per head, pairs
        (2, (1, 1, 64 * 65), (1, 1, 64), 3),  # nb 65: one row in the second round, every row split
        (2, (4, 64, 65), (2, 8, 8), 7),  # nb 144, partial last column
        (17, (1, 1, 64 * 257), (1, 1, 64), 90),  # nb 257 (the next number of rounds), more heads than waves
    ],
)
def test_work_list_over_row_rounds(heads, grid, tile, split):
    # The work list's workgroup takes a head's rows in rounds of 64, a lane
    # each: numbers of blocks around a whole round, forced and automatic
    # chunks, more heads than it has waves.
    torch, fva = torch_mod(), lib()
    cfg = custom_config("rounds", heads, grid, tile, np.linspace(0.3, 5.0, heads), seed=71)
    geo = geometry_of(cfg)
    rng = np.random.default_rng(72)
    q, k, v = (torch.randn((1, heads, cfg.N, 128), generator=torch.Generator().manual_seed(73 + i)).bfloat16().cuda()
               for i in range(3))
    mask = (rng.random((1, heads, geo.nb, geo.nb)) < rng.random((1, heads, geo.nb, 1))).astype(np.uint8)
    m = torch.from_numpy(mask).cuda()
    want = fva.fva_attn(q, k, v, tiling_of(cfg), m, flags=fva.FVA_SCHED_NAIVE)
    out = torch.full_like(q, float("nan"))
    fva.fva_attn(q, k, v, tiling_of(cfg), m, flags=fva.FVA_SPLIT_BLOCKS(split) if split else 0, out=out)
    # rows that are cut into chunks merge them in another order: within the
    # bar of the attention itself
    assert not torch.isnan(out).any()
    assert (out.float() - want.float()).abs().max().item() <= ATTN_MAX_ABS
    c = torch.from_numpy(mask.sum(-1).astype(np.int64))
    S = split or max(32, -(-int((c + 1).sum()) // 1024))
    tok = torch.from_numpy(np.concatenate(geo.block_tokens))
    whole = (c[0] <= S).numpy().repeat(geo.block_sizes, axis=1)
    for h in range(heads):
        rows = tok[torch.from_numpy(whole[h])].cuda()
        assert torch.equal(out[0, h, rows], want[0, h, rows])


@pytest.mark.parametrize("v", ["bf16", "e4m3"])
@pytest.mark.parametrize("grid,tile", [((3, 9, 13), (2, 8, 8)), ((1, 1, 1000), (1, 1, 128)), ((2, 8, 12), (1, 8, 8))])
def test_eight_waves_equal_four(v, grid, tile):
    # Up to a row per CU runs on eight waves of one query tile, more rows on four
    # of two: the same heads give the same bits alone and among others, for
    # blocks of every number of tiles (8 .. 128 tokens).
    torch, fva = torch_mod(), lib()
    heads = 72  # 72 x 8 (or 12) rows, then the first two heads of them alone
    cfg = custom_config("waves", heads, grid, tile, np.linspace(0.3, 5.0, heads), seed=91)
    geo = geometry_of(cfg)
    rng = np.random.default_rng(92)
    q, k, w = (torch.randn((1, heads, cfg.N, 128), generator=torch.Generator().manual_seed(93 + i)).bfloat16().cuda()
               for i in range(3))
    mask = torch.from_numpy((rng.random((1, heads, geo.nb, geo.nb)) < 0.6).astype(np.uint8)).cuda()
    assert heads * geo.nb > 256 >= 2 * geo.nb

    def attend(n):
        qn, kn, wn, mn = (x[:, :n].contiguous() for x in (q, k, w, mask))
        if v == "bf16":
            return fva.fva_attn(qn, kn, wn, tiling_of(cfg), mn, flags=fva.FVA_SCHED_NAIVE)
        return fva.fva_attn_fp8v(qn, kn, *fva.fva_quantize_v(wn, tiling_of(cfg)), tiling_of(cfg), mn,
                                 flags=fva.FVA_SCHED_NAIVE)

    assert torch.equal(attend(2), attend(heads)[:, :2])


@pytest.mark.parametrize("heads", [20, 40])  # union lists of 10.5 MB, and of 21 MB: more than the scratch
def test_noalloc_pairs_where_they_fit(heads):
    torch, fva = torch_mod(), lib()
    cfg = custom_config("fit", heads, (1, 128, 256), (1, 8, 8), np.ones(heads), seed=95)  # 512 blocks, 256 pairs per head
    nb = geometry_of(cfg).nb
    gen = torch.Generator(device="cuda").manual_seed(96)
    q, k, v = (torch.randn((1, heads, cfg.N, 128), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    mask = (torch.rand((1, heads, nb, nb), generator=gen, device="cuda") < 0.02).to(torch.uint8)
    mask *= (mask.cumsum(-1) <= 32).to(torch.uint8)  # nothing is split
    counts = mask.sum(-1, dtype=torch.int32)
    ids = torch.arange(nb, device="cuda", dtype=torch.int32)
    kv = torch.where(mask.bool(), ids, ids + nb).sort(-1).values.contiguous()
    kv = torch.where(kv < nb, kv, torch.zeros_like(kv))
    out = torch.full_like(q, float("nan"))
    fva.fva_attn_noalloc(q, k, v, tiling_of(cfg), counts, kv, out)
    assert torch.equal(out, fva.fva_attn(q, k, v, tiling_of(cfg), mask, counts, kv))


@pytest.mark.parametrize("heads", [20, 21])
def test_item_order_by_heads(heads):
    """Up to 20 heads the long rows of all heads start before the short ones of any; with more
    the heads run one after the other (in the order of their cost, here of their number)."""
    torch, fva = torch_mod(), lib()
    nb, long, short = 128, 32, 8  # (32: the smallest automatic chunk, so nothing is split)
    t = fva.Tiling.curve(nb * 128, 128)
    g = torch.Generator(device="cuda:0").manual_seed(91)
    q, k, v = (torch.randn(1, heads, nb * 128, 128, generator=g, device="cuda:0").bfloat16() for _ in range(3))
    is_long = torch.arange(nb, device="cuda:0") % 2 == 0
    counts = torch.where(is_long, long, short).int().expand(1, heads, nb).contiguous()
    ids = torch.arange(nb, dtype=torch.int32, device="cuda:0")
    kv = ids.expand(1, heads, nb, nb).contiguous()
    mask = (ids < counts[..., None]).to(torch.uint8)
    trace = torch.zeros(fva.fva_trace_words(fva._desc_of(q), t), dtype=torch.int64, device="cuda:0")
    out = fva.fva_attn(q, k, v, t, mask, counts, kv, flags=fva.FVA_TRACE, trace=trace)
    want = fva.fva_attn(q, k, v, t, mask, counts, kv, flags=fva.FVA_SCHED_NAIVE)
    assert torch.equal(out, want)
    start = trace.view(-1, 4)[: heads * nb, 0].cpu().numpy().reshape(heads, nb)
    assert (start > 0).all()
    is_long = is_long.cpu().numpy()
    first_short, last_long = np.median(start[0, ~is_long]), np.median(start[-1, is_long])
    assert (first_short > last_long) if heads <= 20 else (first_short < last_long)
