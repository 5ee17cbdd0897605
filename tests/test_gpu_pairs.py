"""Query-block pairs of the persistent scheduler.

Two neighbouring query blocks of at most 64 real tokens (x-neighbours, else
y-neighbours) run as one item over the union of their kept lists, each on
two of the four waves, each wave
skipping the key blocks its own block does not keep. Every row therefore
sees exactly its own key blocks in ascending order, as it does alone: the
paired launch must equal, bit for bit, the same launch under
FVA_SCHED_UNPAIRED and the naive grid, on every kind of workload that forms
pairs (one-frame last t-rows, the narrow last column of 480p, partial boxes
on every axis, 64-token boxes, 64-token curve runs, split rows next to
paired ones, E4M3 V). Pairs are formed only from 512 items on, so small clips
run with their heads several times over, and every comparison looks the pairs
up in the trace first. The oracle
parity of the same launches is covered by the other attention tests, which
run the default (paired) path.
"""

import numpy as np
import pytest

import synth

from _gpu_util import custom_config, geometry_of, lib, log, tiling_of, to_dev, torch_mod, workload

pytestmark = pytest.mark.gpu


def pairs_of(geo):
    """(first block, second block) of every pair of one head, by definition:
    x-neighbours (ix even, ix + 1) of one (t, y) line with at most 64 tokens
    each; then, among the blocks no x-pair holds, y-neighbours (iy even,
    iy + 1) of one (t, x) column with at most 64 tokens each."""
    n = geo.block_sizes.reshape(geo.nbt, geo.nby, geo.nbx)
    bid = lambda t, y, x: (t * geo.nby + y) * geo.nbx + x
    out, taken = [], set()
    for t in range(geo.nbt):
        for y in range(geo.nby):
            for x in range(0, geo.nbx - 1, 2):
                if n[t, y, x] <= 64 and n[t, y, x + 1] <= 64:
                    out.append((bid(t, y, x), bid(t, y, x + 1)))
                    taken |= {bid(t, y, x), bid(t, y, x + 1)}
    for t in range(geo.nbt):
        for x in range(geo.nbx):
            for y in range(0, geo.nby - 1, 2):
                a, b = bid(t, y, x), bid(t, y + 1, x)
                if a not in taken and b not in taken and n[t, y, x] <= 64 and n[t, y + 1, x] <= 64:
                    out.append((a, b))
    return sorted(out)


def chunk_size(mask_np):
    """The automatic chunk size: max(32, ceil(sum over rows of (kept + 1) / 1024))."""
    return max(32, -(-int((mask_np.sum(-1, dtype=np.int64) + 1).sum()) // 1024))


def split_rows(mask_np):
    """Rows the automatic chunk size splits: more kept blocks than it."""
    return mask_np.reshape(-1, mask_np.shape[-1]).sum(-1) > chunk_size(mask_np)


def assert_pairs_run(attend, desc, tiling, counts, S, geo):
    """The traced launch `attend(flags, trace)` runs every pair whose rows both
    keep at most S blocks as one item (the first row's record ends where the
    second's starts, in one workgroup), and there is such a pair: a call whose
    rows are too few for pairs, or that takes the plain grid, would compare a
    launch with itself. Returns the output."""
    fva, torch = lib(), torch_mod()
    trace = torch.zeros(fva.fva_trace_words(desc, tiling), dtype=torch.int64, device="cuda:0")
    O = attend(fva.FVA_TRACE, trace)
    torch.cuda.synchronize()
    tr = trace.view(-1, 4).cpu().numpy()
    whole = counts.reshape(-1, geo.nb) <= S
    formed = 0
    for a, b in pairs_of(geo):
        for bh in np.nonzero(whole[:, a] & whole[:, b])[0]:
            ra, rb = tr[bh * geo.nb + a], tr[bh * geo.nb + b]
            assert ra[0] > 0 and ra[1] == rb[0] and ra[2] == rb[2], (bh, a, b)
            formed += 1
    assert formed > 0
    return O


def repeated(x, copies):
    """The heads of host bits [batch, heads, ...] `copies` times over."""
    return np.tile(x, (1, copies) + (1,) * (x.ndim - 2))


def same_three_ways(q, k, v, tiling, mask, counts, kv, geo, split=0):
    """Paired (and pairs are formed) == FVA_SCHED_UNPAIRED everywhere; == the
    naive grid on the rows that are not split (a split row merges chunks in
    another order)."""
    fva, torch = lib(), torch_mod()
    extra = fva.FVA_SPLIT_BLOCKS(split) if split else 0
    O = fva.fva_attn(q, k, v, tiling, mask, counts, kv, flags=extra)
    O_u = fva.fva_attn(q, k, v, tiling, mask, counts, kv, flags=extra | fva.FVA_SCHED_UNPAIRED)
    torch.cuda.synchronize()
    assert torch.equal(O, O_u)
    m = mask.cpu().numpy()
    attend = lambda flags, trace: fva.fva_attn(q, k, v, tiling, mask, counts, kv, flags=extra | flags, trace=trace)
    assert torch.equal(O, assert_pairs_run(attend, fva._desc_of(q), tiling, m.sum(-1), split or chunk_size(m), geo))
    if not extra:
        O_n = fva.fva_attn(q, k, v, tiling, mask, counts, kv, flags=fva.FVA_SCHED_NAIVE)
        torch.cuda.synchronize()
        split = split_rows(m)
        if not split.any():
            assert torch.equal(O, O_n)
        else:
            a = O.view(torch.int16).cpu().numpy().reshape(-1, O.shape[-2], O.shape[-1])
            b = O_n.view(torch.int16).cpu().numpy().reshape(a.shape)
            for r in np.nonzero(~split)[0]:
                tok = geo.block_tokens[r % geo.nb]
                assert np.array_equal(a[r // geo.nb, tok], b[r // geo.nb, tok]), r
    return O


@pytest.mark.parametrize("name,heads", [("tiny", None), ("720p", [0, 9, 21, 39]), ("480p", [3, 11, 25, 38])])
def test_pairs_equal_unpaired_on_routed_workloads(name, heads):
    fva = lib()
    cfg = synth.get_config(name)
    geo = geometry_of(cfg)
    Qb, Kb, Vb = workload(name)
    if heads is not None:
        Qb, Kb, Vb = Qb[:, heads], Kb[:, heads], Vb[:, heads]
    else:
        # pairs are formed from 512 items on: the clip's two heads 43 times are 1032 rows in 516 pairs
        Qb, Kb, Vb = (repeated(x, 43) for x in (Qb, Kb, Vb))
    q, k, v = to_dev(Qb), to_dev(Kb), to_dev(Vb)
    mask, counts, kv = fva.fva_route(q, k, cfg.p, cfg.k_min, tiling_of(cfg))
    pairs = pairs_of(geo)
    assert pairs  # every one of these workloads forms pairs
    c = counts.cpu().numpy().reshape(-1, geo.nb)
    m = mask.cpu().numpy().reshape(-1, geo.nb, geo.nb)
    both = sum(int((m[h, a] & m[h, b]).sum()) for h in range(m.shape[0]) for a, b in pairs)
    union = sum(int((m[h, a] | m[h, b]).sum()) for h in range(m.shape[0]) for a, b in pairs)
    log(f"[pairs] {name}: {len(pairs)} pairs per head, union/shared kept blocks {union}/{both}, "
        f"mean count {c.mean():.1f}")
    same_three_ways(q, k, v, tiling_of(cfg), mask, counts, kv, geo)
    same_three_ways(q, k, v, tiling_of(cfg), mask, None, None, geo)  # lists rebuilt from the mask


@pytest.mark.parametrize("s", [2, 5])
def test_pairs_next_to_split_rows(s):
    # Partial boxes on all three axes (5 = 2*2 + 1 frames, 13 = 8 + 5 rows,
    # 21 = 2*8 + 5 columns): the one-frame t-row forms the x-pairs (12, 13)
    # and (15, 16) and the y-pair (14, 17) of its narrow last column. Random
    # masks elsewhere; in every head row 13 keeps s + 2 blocks (split into
    # chunks, so its pair is not formed) and rows 15 and 16 keep at most s
    # blocks, one shared and one of their own each (paired).
    # Each of the three heads 12 times over: 36 * 15 items with every pair formed.
    fva, torch = lib(), torch_mod()
    copies = 12
    cfg = custom_config("pairsplit", 3, (5, 13, 21), (2, 8, 8), (0.3, 1.5, 5.0), seed=41)
    geo = geometry_of(cfg)
    assert pairs_of(geo) == [(12, 13), (14, 17), (15, 16)]
    heads = 3 * copies
    Qb, Kb, Vb = (repeated(x, copies) for x in synth.gen_qkv(cfg))
    rng = np.random.default_rng(43 + s)
    m = (rng.random((1, heads, geo.nb, geo.nb)) < 0.25).astype(np.uint8)
    m[0, :, ::4, :] = 0
    m[0, :, 12:17, :] = 0
    m[0, :, 12, 0] = 1
    m[0, :, 13, :s + 2] = 1
    m[0, :, 15, [1, 3]] = 1
    m[0, :, 16, [3, 4]] = 1
    q, k, v = to_dev(Qb), to_dev(Kb), to_dev(Vb)
    mt = torch.from_numpy(m).to("cuda:0")
    same_three_ways(q, k, v, tiling_of(cfg), mt, None, None, geo, split=s)
    O = same_three_ways(q, k, v, tiling_of(cfg), mt, None, None, geo)
    O_split = fva.fva_attn(q, k, v, tiling_of(cfg), mt, flags=fva.FVA_SPLIT_BLOCKS(s))
    torch.cuda.synchronize()
    # rows cut into chunks merge them in another rounding order; whole rows
    # (paired or not) are the same bit for bit
    a = O.view(torch.int16).cpu().numpy()
    b = O_split.view(torch.int16).cpu().numpy()
    counts = m.sum(-1)
    for h in range(heads):
        for i in range(geo.nb):
            if counts[0, h, i] <= s:
                tok = geo.block_tokens[i]
                assert np.array_equal(a[0, h, tok], b[0, h, tok]), (h, i)


def test_pairs_64_token_curve_runs():
    # one-dimensional blocks of 64 consecutive tokens (the curve layout's
    # tiling): every block but a short last one pairs with its neighbour
    fva = lib()
    cfg = custom_config("run64", 4, (1, 1, 20000), (1, 1, 64), (0.5, 1.0, 2.0, 3.0), seed=47)
    Qb, Kb, Vb = synth.gen_qkv(cfg)
    q, k, v = to_dev(Qb), to_dev(Kb), to_dev(Vb)
    t = fva.Tiling(1, 1, 20000, 1, 1, 64)
    mask, counts, kv = fva.fva_route(q, k, cfg.p, cfg.k_min, t)
    same_three_ways(q, k, v, t, mask, counts, kv, geometry_of(cfg))


@pytest.mark.parametrize("name", ["720p", "partial boxes", "64-token runs"])
def test_pairs_fp8_v(name):
    fva, torch = lib(), torch_mod()
    if name == "720p":
        cfg = synth.get_config("720p")
        Qb, Kb, Vb = (x[:, [2, 17, 30]] for x in workload("720p"))
    elif name == "partial boxes":  # x- and y-pairs of a (5, 13, 21) clip, its three heads 12 times over
        cfg = custom_config("pairs8", 3, (5, 13, 21), (2, 8, 8), (0.3, 1.5, 5.0), seed=42)
        Qb, Kb, Vb = (repeated(x, 12) for x in synth.gen_qkv(cfg))
    else:
        cfg = custom_config("run64f", 4, (1, 1, 20000), (1, 1, 64), (0.5, 1.0, 2.0, 3.0), seed=48)
        Qb, Kb, Vb = synth.gen_qkv(cfg)
    geo = geometry_of(cfg)
    q, k, v = to_dev(Qb), to_dev(Kb), to_dev(Vb)
    t = tiling_of(cfg)
    mask, counts, kv = fva.fva_route(q, k, cfg.p, cfg.k_min, t)
    v8, vexp = fva.fva_quantize_v(v, t)
    attend = lambda flags, trace=None: fva.fva_attn_fp8v(q, k, v8, vexp, t, mask, counts, kv, flags=flags, trace=trace)
    m = mask.cpu().numpy()
    O = assert_pairs_run(attend, fva._desc_of(q), t, m.sum(-1), chunk_size(m), geo)
    O_u = attend(fva.FVA_SCHED_UNPAIRED)
    O_n = attend(fva.FVA_SCHED_NAIVE)
    torch.cuda.synchronize()
    assert torch.equal(O, attend(0)) and torch.equal(O, O_u)
    whole = torch.from_numpy(~split_rows(m).reshape(m.shape[:3]))
    for h in range(m.shape[1]):
        tok = torch.from_numpy(np.concatenate([geo.block_tokens[i] for i in np.nonzero(whole[0, h])[0]])).cuda()
        assert torch.equal(O[0, h, tok], O_n[0, h, tok]), h


def test_pair_trace_records_split_the_item():
    fva, torch = lib(), torch_mod()
    cfg = synth.get_config("720p")
    geo = geometry_of(cfg)
    heads = [5, 12, 33, 38]
    Qb, Kb, Vb = workload("720p")
    q, k, v = to_dev(Qb[:, heads]), to_dev(Kb[:, heads]), to_dev(Vb[:, heads])
    t = tiling_of(cfg)
    mask, counts, kv = fva.fva_route(q, k, cfg.p, cfg.k_min, t)
    desc = fva._desc_of(q)
    trace = torch.zeros(fva.fva_trace_words(desc, t), dtype=torch.int64, device="cuda:0")
    fva.fva_attn(q, k, v, t, mask, counts, kv, flags=fva.FVA_TRACE, trace=trace)
    torch.cuda.synchronize()
    tr = trace.view(-1, 4).cpu().numpy()
    c = counts.cpu().numpy().reshape(-1)
    rows = c.size
    # the automatic chunk size; rows keeping more are split (no row record)
    S = max(32, -(-int((c + 1).sum()) // 1024))
    whole = c <= S
    assert np.all(tr[:rows][whole, 0] > 0) and np.all(tr[:rows][whole, 3] > 0)
    assert np.all(tr[:rows, 1] >= tr[:rows, 0]) and not tr[:rows][~whole].any()
    formed = 0
    for h in range(len(heads)):
        for a, b in pairs_of(geo):
            ra, rb = h * geo.nb + a, h * geo.nb + b
            if whole[ra] and whole[rb]:
                # one item: the same workgroup, the first record ends where the second starts
                assert tr[ra, 1] == tr[rb, 0] and tr[ra, 2] == tr[rb, 2], (h, a)
                formed += 1
    log(f"[pairs] 720p trace: S = {S}, {formed} pairs formed, {int((~whole).sum())} rows split")
    assert formed > 0
