"""GPU check of fva_attn_noalloc, the allocation-free attention call.

The call runs fva_attn on the library's static device scratch. Calls in a
row, each on a smaller input (the scratch keeps the earlier calls' contents),
each compared with fva_attn on the same
inputs and lists: identical where fva_attn splits no row, and within the
attention bar (max 2e-2, mean 1e-3 against the fp64 oracle) where its
automatic chunk size splits rows that the allocation-free call keeps whole.
"""

import ctypes

import numpy as np
import pytest

import synth
from oracle import attn_ref_rows
from oracle.compare import ATTN_MAX_ABS, ATTN_MEAN_ABS

from _gpu_util import custom_config, f64, geometry_of, lib, log, tiling_of, to_dev, torch_mod, workload
from test_gpu_pairs import pairs_of

pytestmark = pytest.mark.gpu


def routed(cfg, Qb, Kb, Vb):
    fva = lib()
    q, k, v = to_dev(Qb), to_dev(Kb), to_dev(Vb)
    mask, counts, kv = fva.fva_route(q, k, cfg.p, cfg.k_min, tiling_of(cfg))
    return q, k, v, mask, counts, kv


def noalloc(q, k, v, cfg, counts, kv, **kw):
    torch = torch_mod()
    out = torch.full_like(q, float("nan"))  # every real row must be written
    lib().fva_attn_noalloc(q, k, v, tiling_of(cfg), counts, kv, out, **kw)
    torch.cuda.synchronize()
    return out


def oracle_errors(cfg, Qb, Kb, Vb, mask, O, heads, blocks):
    geo = geometry_of(cfg)
    errs = []
    for h in heads:
        ref = attn_ref_rows(f64(Qb[0, h]), f64(Kb[0, h]), f64(Vb[0, h]), mask[0, h], geo, blocks)
        for i, o in ref.items():
            errs.append(np.abs(O[0, h][geo.block_tokens[i]] - o).ravel())
    e = np.concatenate(errs)
    return float(e.max()), float(e.mean())


def test_noalloc_two_calls_second_smaller():
    torch, fva = torch_mod(), lib()
    # call 1: the 480p layer (40 heads, nb 308); fva_attn splits nothing here
    cfg1 = synth.get_config("480p")
    Q1, K1, V1 = workload("480p")
    q, k, v, mask, counts, kv = routed(cfg1, Q1, K1, V1)
    O_ref = fva.fva_attn(q, k, v, tiling_of(cfg1), mask, counts, kv)
    O_na = noalloc(q, k, v, cfg1, counts, kv)
    assert torch.equal(O_na, O_ref)
    emax, emean = oracle_errors(cfg1, Q1, K1, V1, mask.cpu().numpy(), O_na.float().cpu().numpy(), [0, 17, 39],
                                [0, 150, 307])
    log(f"[noalloc] 480p: identical to fva_attn; oracle rows max {emax:.3e} mean {emean:.3e}")
    assert emax <= ATTN_MAX_ABS and emean <= ATTN_MEAN_ABS
    del q, k, v, mask, counts, kv, O_ref, O_na
    # call 2: a smaller work list over the first one's, on the scratch it left:
    # the 3x16x16 clip's two heads 43 times over, 1032 rows
    cfg2 = synth.get_config("tiny")
    Q2, K2, V2 = workload("tiny")
    q, k, v, mask, counts, kv = routed(cfg2, *(np.tile(x, (1, 43, 1, 1)) for x in (Q2, K2, V2)))
    O_ref = fva.fva_attn(q, k, v, tiling_of(cfg2), mask, counts, kv, flags=fva.FVA_SCHED_NAIVE)
    O_na = noalloc(q, k, v, cfg2, counts, kv)
    assert torch.equal(O_na, O_ref)
    O_many = O_na
    # call 3: the two heads alone, which take the plain grid
    q, k, v, mask, counts, kv = routed(cfg2, Q2, K2, V2)
    O_ref = fva.fva_attn(q, k, v, tiling_of(cfg2), mask, counts, kv)
    O_na = noalloc(q, k, v, cfg2, counts, kv)
    assert torch.equal(O_na, O_ref)
    assert torch.equal(O_na.repeat(1, 43, 1, 1), O_many)
    emax, emean = oracle_errors(cfg2, Q2, K2, V2, mask.cpu().numpy(), O_na.float().cpu().numpy(), [0, 1],
                                range(12))
    log(f"[noalloc] tiny after 480p: identical to fva_attn; every element max {emax:.3e} mean {emean:.3e}")
    assert emax <= ATTN_MAX_ABS and emean <= ATTN_MEAN_ABS


def test_noalloc_where_fva_attn_splits_rows():
    # One flat head of the 480p shape: fva_attn's automatic chunk size splits
    # its long rows; the allocation-free call keeps them whole.
    torch, fva = torch_mod(), lib()
    cfg = custom_config("one_head", 1, (21, 30, 52), (2, 8, 8), (0.5,), seed=24)
    Qb, Kb, Vb = synth.gen_qkv(cfg)
    q, k, v, mask, counts, kv = routed(cfg, Qb, Kb, Vb)
    O_ref = fva.fva_attn(q, k, v, tiling_of(cfg), mask, counts, kv)
    O_na = noalloc(q, k, v, cfg, counts, kv)
    d = (O_na.float() - O_ref.float()).abs()
    assert not torch.isnan(O_na).any()
    m = mask.cpu().numpy()
    c = counts.cpu().numpy()[0, 0]
    rows = sorted(set(int(i) for i in np.argsort(-c)[:8]) | {0, 307})
    emax, emean = oracle_errors(cfg, Qb, Kb, Vb, m, O_na.float().cpu().numpy(), [0], rows)
    log(f"[noalloc] one flat head: |noalloc - fva_attn| max {d.max().item():.3e} mean {d.mean().item():.3e}; "
        f"oracle rows max {emax:.3e} mean {emean:.3e}")
    assert d.max().item() <= ATTN_MAX_ABS and d.mean().item() <= ATTN_MEAN_ABS
    assert emax <= ATTN_MAX_ABS and emean <= ATTN_MEAN_ABS


def test_noalloc_trace_and_repeat():
    torch, fva = torch_mod(), lib()
    cfg = synth.get_config("tiny")
    Qb, Kb, Vb = workload("tiny")
    q, k, v, mask, counts, kv = routed(cfg, Qb, Kb, Vb)
    desc = fva._desc_of(q)
    trace = torch.zeros(fva.fva_trace_words(desc, tiling_of(cfg)), dtype=torch.int64, device="cuda:0")
    O1 = noalloc(q, k, v, cfg, counts, kv, flags=fva.FVA_TRACE, trace=trace)
    O2 = noalloc(q, k, v, cfg, counts, kv)
    assert torch.equal(O1, O2)
    tr = trace.view(-1, 4).cpu().numpy()
    rows = cfg.heads * geometry_of(cfg).nb
    assert np.all(tr[:rows, 0] > 0) and np.all(tr[:rows, 1] >= tr[:rows, 0]) and not tr[rows:].any()


def test_noalloc_graph_holds_two_launches():
    # No row of the allocation-free call is split: the work list and the
    # attention are all it launches, and replays of the captured pair follow
    # the inputs' contents.
    torch, fva = torch_mod(), lib()
    cfg = custom_config("captured", 6, (4, 32, 96), (1, 8, 8), np.linspace(0.5, 4.0, 6), seed=25)
    Qb, Kb, Vb = synth.gen_qkv(cfg)
    q, k, v, mask, counts, kv = routed(cfg, Qb, Kb, Vb)
    assert q.shape[1] * counts.shape[2] > 512 and counts.shape[2] > 32  # a work list, rows long enough to be split
    out = torch.empty_like(q)
    fva.fva_attn_noalloc(q, k, v, tiling_of(cfg), counts, kv, out)  # (the first call finds the scratch's address)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        fva.fva_attn_noalloc(q, k, v, tiling_of(cfg), counts, kv, out)
    hip = ctypes.CDLL(fva.LIB_PATH)  # (and the HIP runtime it is bound to)
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    assert n.value == 2
    graph.instantiate()
    for scale in (1.0, -2.0, 0.5):
        v.copy_(to_dev(Vb) * scale)
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, noalloc(q, k, v, cfg, counts, kv))


@pytest.mark.parametrize("heads, grid, tile", [(2, (21, 30, 52), (2, 8, 8)), (4, (16, 26, 43), (2, 8, 8))])
def test_noalloc_pairs_start_first(heads, grid, tile):
    """No row is split here, so a query-block pair is the longest item there is: with all rows
    equally long, and more of them than workgroups, every pair starts before any item ends (the
    items that begin later are single rows)."""
    torch, fva = torch_mod(), lib()
    cfg = custom_config("pairs_first", heads, grid, tile, [1.0] * heads, 5)
    geo, t = geometry_of(cfg), tiling_of(cfg)
    nb, kept = geo.nb, geo.nb // 2
    pairs = pairs_of(geo)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert pairs and 2 * len(pairs) < nb  # (a tiling with pairs at its edges only)
    assert 2 * cus < heads * (nb - len(pairs))  # pairs are formed, and some items have to wait
    g = torch.Generator(device="cuda:0").manual_seed(11)
    N = geo.block_sizes.sum()
    q, k, v = (torch.randn(1, heads, int(N), 128, generator=g, device="cuda:0").bfloat16() for _ in range(3))
    counts = torch.full((1, heads, nb), kept, dtype=torch.int32, device="cuda:0")
    kv = torch.zeros((1, heads, nb, nb), dtype=torch.int32, device="cuda:0")
    kv[..., :kept] = torch.arange(kept, dtype=torch.int32, device="cuda:0")
    desc = fva._desc_of(q)
    trace = torch.zeros(fva.fva_trace_words(desc, t), dtype=torch.int64, device="cuda:0")
    for _ in range(2):  # (the first launch of a process starts its workgroups later)
        out = torch.full_like(q, float("nan"))
        fva.fva_attn_noalloc(q, k, v, t, counts, kv, out, flags=fva.FVA_TRACE, trace=trace)
        torch.cuda.synchronize()
    tr = trace.view(-1, 4)[: heads * nb].cpu().numpy()
    first = np.zeros(nb, bool)
    first[[a for a, _ in pairs]] = True
    second = np.zeros(nb, bool)
    second[[b for _, b in pairs]] = True
    start, end = tr[:, 0].reshape(heads, nb), tr[:, 1].reshape(heads, nb)
    assert (start[:, first] < end[:, ~first & ~second].min()).all()
