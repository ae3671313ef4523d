"""GPU parity of the whole-set conversions (start / end of a round, and a change of the set of
quantized variables between rounds, Sec. 2.5) against per-variable oracle calls."""
import numpy as np
import pytest
import torch

from oracle import omc_oracle as orc
from paper_2205_03494_amd import omc, synth
from gpu_util import bits_equal, to_dev

pytestmark = pytest.mark.gpu


def build(specs, mask, fmts, use_pvt=True):
    gfs = [omc.fmt(*fmts[i]) if mask[i] else None for i in range(len(specs))]
    sizes = iter([omc.omc_packed_bytes(gfs[i], specs[i].n) for i in range(len(specs)) if mask[i]])
    lay = synth.make_layout(specs, mask, lambda n: next(sizes))
    table = [dict(data_offset=int(lay.data_offset[i]), aux_offset=int(lay.aux_offset[i]), n=s.n, fmt=gfs[i],
                  quantized=bool(mask[i]), use_pvt=use_pvt) for i, s in enumerate(specs)]
    return lay, omc.omc_plan_build(omc.make_var_table(table))


def oracle_arena(specs, mask, fmts, lay, vals):
    arena = np.zeros(lay.arena_bytes, np.uint8)
    sbt = np.zeros((len(specs), 2), np.float32)
    for i, s in enumerate(specs):
        a, d = int(lay.aux_offset[i]), int(lay.data_offset[i])
        x = vals[a:a + s.n]
        if mask[i]:
            p, sb = orc.compress(x, orc.Format(*fmts[i]))
            arena[d:d + p.size] = p
            sbt[i] = sb
        else:
            arena[d:d + 4 * s.n] = x.view(np.uint8)
    return arena, sbt


def gpu_compress_set(lay, plan, vals, nvars):
    arena = torch.full((lay.arena_bytes,), 0, dtype=torch.uint8, device="cuda")
    sb = torch.full((nvars, 2), 7.0, device="cuda")
    ws = torch.empty(max(plan.workspace_bytes, 16), dtype=torch.uint8, device="cuda")
    omc.omc_compress_set(to_dev(vals), plan, arena, sb, ws)
    torch.cuda.synchronize()
    return arena, sb


def ragged_specs():
    # sizes around the tile and chunk borders, a tail-only variable, vectors
    ns = [1, 31, 2047, 2048, 2049, 4096, 4097, 8192, 8193, 5 * 8192 + 77, 3 * 2048, 40000, 100, 2048 * 9 + 1]
    return [synth.VarSpec(f"v{i}", (n,), max(n, 1), i % 4 != 3) for i, n in enumerate(ns)]


@pytest.mark.parametrize("case", ["conformer", "ragged", "fp32_only", "tails_only"])
def test_compress_set_and_decompress_set(case):
    if case == "conformer":
        specs = synth.conformer_varset(96, 2, 384, 8, frontend=True)
        mask = synth.ppq_mask(specs, 0.6, 4)
    elif case == "ragged":
        specs = ragged_specs()
        mask = np.array([s.is_matrix for s in specs])
    elif case == "fp32_only":
        specs = ragged_specs()
        mask = np.zeros(len(specs), bool)
    else:
        specs = [synth.VarSpec(f"t{i}", (n,), n, True) for i, n in enumerate([5, 700, 2047, 33])]
        mask = np.ones(len(specs), bool)
    choices = [(4, 3), (3, 7), (5, 10), (2, 3), (8, 7)]
    fmts = [choices[i % len(choices)] for i in range(len(specs))]
    lay, plan = build(specs, mask, fmts)
    vals = synth.init_values(lay, 9)
    want_arena, want_sb = oracle_arena(specs, mask, fmts, lay, vals)
    arena, sb = gpu_compress_set(lay, plan, vals, len(specs))
    assert np.array_equal(arena.cpu().numpy(), want_arena)
    gsb = sb.cpu().numpy()
    assert bits_equal(gsb[mask], want_sb[mask])
    assert np.all(gsb[~mask] == 7.0)                       # untouched for fp32 variables
    assert plan.transport_bytes == sum(orc.packed_bytes(s.n, 1 + sum(fmts[i])) + 8 if mask[i] else 4 * s.n
                                       for i, s in enumerate(specs))
    # and back
    out = torch.full((lay.aux_elems,), float("nan"), device="cuda")
    omc.omc_decompress_set(arena, plan, sb, out)
    torch.cuda.synchronize()
    o = out.cpu().numpy()
    for i, s in enumerate(specs):
        a, d = int(lay.aux_offset[i]), int(lay.data_offset[i])
        if mask[i]:
            of = orc.Format(*fmts[i])
            nb = orc.packed_bytes(s.n, of.bits)
            want = orc.decompress(want_arena[d:d + nb], s.n, of, want_sb[i])
        else:
            want = vals[a:a + s.n]
        assert bits_equal(o[a:a + s.n], want), s.name
        pad = o[a + s.n:int(lay.aux_offset[i + 1]) if i + 1 < len(specs) else lay.aux_elems]
        assert np.all(np.isnan(pad))                       # nothing written between variables


def test_reselection_between_rounds():
    """The set of quantized variables changes (Sec. 2.5): decompress with the old plan, compress with
    the new one; every variable must come out as the oracle's conversion of the same values."""
    specs = synth.conformer_varset(64, 2, 256, 8, frontend=False)
    fmts = [(3, 7)] * len(specs)
    mask_a, mask_b = synth.ppq_mask(specs, 0.9, 1), synth.ppq_mask(specs, 0.9, 2)
    assert np.any(mask_a != mask_b)
    lay_a, plan_a = build(specs, mask_a, fmts)
    lay_b, plan_b = build(specs, mask_b, fmts)
    vals = synth.init_values(lay_a, 3)
    arena_a, sb_a = gpu_compress_set(lay_a, plan_a, vals, len(specs))
    mid = torch.zeros(lay_a.aux_elems, device="cuda")
    omc.omc_decompress_set(arena_a, plan_a, sb_a, mid)
    arena_b = torch.zeros(lay_b.arena_bytes, dtype=torch.uint8, device="cuda")
    sb_b = torch.zeros((len(specs), 2), device="cuda")
    ws = torch.empty(max(plan_b.workspace_bytes, 16), dtype=torch.uint8, device="cuda")
    omc.omc_compress_set(mid, plan_b, arena_b, sb_b, ws)
    torch.cuda.synchronize()
    oa, osb = oracle_arena(specs, mask_a, fmts, lay_a, vals)
    mid_ref = np.zeros(lay_a.aux_elems, np.float32)
    of = orc.Format(3, 7)
    for i, s in enumerate(specs):
        a, d = int(lay_a.aux_offset[i]), int(lay_a.data_offset[i])
        mid_ref[a:a + s.n] = (orc.decompress(oa[d:d + orc.packed_bytes(s.n, 11)], s.n, of, osb[i]) if mask_a[i]
                              else vals[a:a + s.n])
    ob, osb_b = oracle_arena(specs, mask_b, fmts, lay_b, mid_ref)
    assert np.array_equal(arena_b.cpu().numpy(), ob)
    assert bits_equal(sb_b.cpu().numpy()[mask_b], osb_b[mask_b])


@pytest.mark.parametrize("many", [False, True])
def test_parts_of_the_copies(many):
    """Copies of fp32 variables that end around the 1024 elements of a part, the 256 of a piece and the four of a lane's, in few work items
    (parts of all items in turn) and in many (an item's parts one after the other)."""
    plain = [1, 3, 4, 5, 255, 257, 1021, 1023, 1024, 1025, 1283, 4095, 4096, 4097, 2 * 4096 + 1024 + 2] + ([1100 * 4096 + 6] if many else [])
    specs = [synth.VarSpec("w", (2 * 2048 + 5,), 2 * 2048 + 5, True)] + [synth.VarSpec(f"b{n}", (n,), n, False) for n in plain]
    mask = np.array([s.is_matrix for s in specs])
    lay, plan = build(specs, mask, [(3, 7)] * len(specs))
    vals = synth.init_values(lay, 12)
    want, want_sb = oracle_arena(specs, mask, [(3, 7)] * len(specs), lay, vals)
    arena, sb = gpu_compress_set(lay, plan, vals, len(specs))
    assert np.array_equal(arena.cpu().numpy(), want)
    out = torch.full((lay.aux_elems,), float("nan"), device="cuda")
    omc.omc_decompress_set(arena, plan, sb, out)
    torch.cuda.synchronize()
    o = out.cpu().numpy()
    for i, s in enumerate(specs):
        a, end = int(lay.aux_offset[i]), int(lay.aux_offset[i + 1]) if i + 1 < len(specs) else lay.aux_elems
        if not mask[i]:
            assert bits_equal(o[a:a + s.n], vals[a:a + s.n]), s.name
        assert np.all(np.isnan(o[a + s.n:end]))


def many_small_variables(count, quantized):
    """A table of `count` variables of one to seven elements, 32 bytes apart in the arena and eight elements in the aux order; no layout helper, which
    would take minutes."""
    rows = np.zeros(count, np.dtype([("data", "<u8"), ("aux", "<u8"), ("n", "<u8"), ("E", "u1"), ("M", "u1"), ("bias", "<i2"), ("flags", "<u4")]))
    rows["data"] = 32 * np.arange(count, dtype=np.uint64)
    rows["aux"] = 8 * np.arange(count, dtype=np.uint64)
    rows["n"] = 1 + np.arange(count) % 7
    rows["E"], rows["M"], rows["bias"] = 4, 3, 7
    rows["flags"] = np.where(quantized, omc.OMC_VAR_QUANTIZED, 0)
    live = (np.arange(8)[None, :] < rows["n"][:, None].astype(np.int64)).ravel()
    return (omc.omc_var * count).from_buffer(rows), torch.from_numpy(live).cuda()


@pytest.mark.parametrize("count,full_tile", [((1 << 19) + 11, True), ((1 << 23) + 11, False)])
def test_millions_of_small_fp32_variables(count, full_tile):
    """Every fp32 item is eight workgroups' work.  More than 2^19 of them take several launches, with a launch of full tiles before them and without; a grid of 2^32
    work-items or more (more than 2^23 items in one launch) would run only what is left of it modulo 2^32."""
    table, live = many_small_variables(count, np.zeros(count, bool))
    if full_tile:                                           # the last variable: quantized, one tile, in room of its own behind the others
        table[count - 1].n, table[count - 1].flags = 2048, omc.OMC_VAR_QUANTIZED
    plan = omc.omc_plan_build(table)
    g = torch.Generator(device="cuda").manual_seed(3)
    aux = max(8 * count, plan.aux_elems)
    w = torch.zeros(aux, device="cuda").normal_(0, 1, generator=g)
    grad = torch.zeros(aux, device="cuda").normal_(0, 1, generator=g)
    arena = torch.zeros(max(32 * count, plan.arena_bytes), dtype=torch.uint8, device="cuda")
    sb = torch.tensor([1.0, 0.0], device="cuda").repeat(count, 1).contiguous()
    ws = torch.empty(max(plan.workspace_bytes, 16), dtype=torch.uint8, device="cuda")
    omc.omc_compress_set(w, plan, arena, sb, ws)
    omc.omc_step_update_recompress(arena, plan, sb, grad, None, None, omc.opt(omc.OMC_SGD, 0.5), ws)
    out = torch.full((aux,), float("nan"), device="cuda")
    omc.omc_decompress_set(arena, plan, sb, out)
    last = 8 * (count - 1) if full_tile else 8 * count
    want = w - 0.5 * grad
    got, mask = out[:last], live[:last]
    assert torch.equal(got[mask], want[:last][mask])        # (0.5 times a float is exact)
    assert torch.isnan(got[~mask]).all()


@pytest.mark.parametrize("quantized", ["nowhere", "at one client"])
def test_mean_of_millions_of_small_variables(quantized):
    """2^20 and more all-fp32 items, four workgroups each, and as many ragged tails, eight each: more than one launch's share."""
    count = (1 << 20) + 11
    masks = [np.full(count, quantized == "at one client"), np.zeros(count, bool)]
    plans, arenas, sbs, values = [], [], [], []
    for r, mask in enumerate(masks):
        table, live = many_small_variables(count, mask)
        plan = omc.omc_plan_build(table)
        w = torch.zeros(8 * count, device="cuda").normal_(0, 1, generator=torch.Generator(device="cuda").manual_seed(r))
        arena = torch.zeros(32 * count, dtype=torch.uint8, device="cuda")
        sb = torch.tensor([1.0, 0.0], device="cuda").repeat(count, 1).contiguous()
        ws = torch.empty(max(plan.workspace_bytes, 16), dtype=torch.uint8, device="cuda")
        omc.omc_compress_set(w, plan, arena, sb, ws)
        back = torch.zeros(8 * count, device="cuda")
        omc.omc_decompress_set(arena, plan, sb, back)
        if not mask.any():
            assert torch.equal(back[live], w[live])
        plans.append(plan), arenas.append(arena), sbs.append(sb), values.append(back)
    agg = omc.omc_aggregate_plan_build(plans)
    out = torch.full((8 * count,), float("nan"), device="cuda")
    omc.omc_aggregate_mean(agg, arenas, sbs, out)
    assert torch.equal(out[live], ((values[0] + values[1]) / 2)[live])
    assert torch.isnan(out[~live]).all()
