"""GPU parity of the server-side aggregation against the oracle: every client's copy decompressed
by the oracle, then its fp32 left-to-right mean, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import omc_oracle as orc
from paper_2205_03494_amd import omc, synth
from gpu_util import bits_equal, to_dev
from test_gpu_sets import build, oracle_arena, ragged_specs

pytestmark = pytest.mark.gpu


def client_values(lay, base, r):
    """Client r's trained copy: the shared starting point plus its own small update."""
    d = synth.gradients(lay, 2e-3, 500 + r)
    return (base + d).astype(np.float32)


def run_case(specs, fmts, masks, seed=0):
    R = len(masks)
    lays, plans, arenas, sbs, ref_src = [], [], [], [], []
    base = None
    for r, mask in enumerate(masks):
        lay, plan = build(specs, mask, fmts)
        if base is None:
            base = synth.init_values(lay, seed)
        vals = client_values(lay, base, r)
        arena, sb = oracle_arena(specs, mask, fmts, lay, vals)     # what client r transports
        lays.append(lay); plans.append(plan)
        arenas.append(to_dev(arena)); sbs.append(to_dev(sb))
        ref_src.append((lay, arena, sb, vals))
    agg = omc.omc_aggregate_plan_build(plans)
    out = torch.full((lays[0].aux_elems,), float("nan"), device="cuda")
    omc.omc_aggregate_mean(agg, arenas, sbs, out)
    torch.cuda.synchronize()
    o = out.cpu().numpy()
    for i, s in enumerate(specs):
        a = int(lays[0].aux_offset[i])
        copies = []
        for r in range(R):
            lay, arena, sb, vals = ref_src[r]
            d = int(lay.data_offset[i])
            if masks[r][i]:
                of = orc.Format(*fmts[i])
                copies.append(orc.decompress(arena[d:d + orc.packed_bytes(s.n, of.bits)], s.n, of, sb[i]))
            else:
                copies.append(arena[d:d + 4 * s.n].view(np.float32))
        want = orc.aggregate_mean(copies)
        assert bits_equal(o[a:a + s.n], want), (s.name, s.n)
        end = int(lays[0].aux_offset[i + 1]) if i + 1 < len(specs) else lays[0].aux_elems
        assert np.all(np.isnan(o[a + s.n:end]))
    return o


@pytest.mark.parametrize("R", [1, 2, 3, 8, 16])
def test_conformer_shaped_set_with_per_client_subsets(R):
    specs = synth.conformer_varset(96, 2, 384, 8, frontend=True)
    fmts = [(4, 3)] * len(specs)
    masks = [synth.ppq_mask(specs, 0.9, 10 + r) for r in range(R)]
    run_case(specs, fmts, masks)


@pytest.mark.parametrize("EM", [(4, 3), (3, 7), (2, 3), (4, 14), (5, 10), (8, 7), (8, 23)])
def test_ragged_sizes_and_formats(EM):
    specs = ragged_specs()
    fmts = [EM] * len(specs)
    rng = np.random.default_rng(5)
    masks = [np.array([s.is_matrix and rng.random() < 0.7 for s in specs]) for _ in range(3)]
    masks[0][:] = [s.is_matrix for s in specs]              # client 0 quantizes every matrix
    masks[1][:] = False                                     # client 1 sends everything in fp32
    run_case(specs, fmts, masks)


def test_mixed_formats_across_variables_and_everyone_fp32():
    specs = ragged_specs()
    choices = [(4, 3), (3, 7), (5, 10), (2, 3)]
    fmts = [choices[i % 4] for i in range(len(specs))]
    masks = [np.array([s.is_matrix for s in specs]), np.array([s.is_matrix and i % 2 == 0 for i, s in enumerate(specs)])]
    run_case(specs, fmts, masks)
    run_case(specs, fmts, [np.zeros(len(specs), bool)] * 3)  # no client quantizes anything


def test_top_codes_and_non_finite_copies_in_the_byte_path():
    """S1E4M3 copies are decoded by the hardware conversion, which reads the top code as NaN; slabs that
    meet one are redone generically.  A NaN / Inf in an fp32 copy must come out as the oracle's NaN / Inf."""
    specs = [synth.VarSpec("w", (8192 * 2 + 2048 * 3,), 8192 * 2 + 2048 * 3, True),
             synth.VarSpec("u", (4096,), 4096, True)]
    fmts = [(4, 3), (4, 3)]
    masks = [np.array([True, True]), np.array([False, True]), np.array([True, False])]
    R = len(masks)
    lays, plans, arenas, sbs, copies = [], [], [], [], [[None] * R for _ in specs]
    for r, mask in enumerate(masks):
        lay, plan = build(specs, mask, fmts)
        vals = synth.init_values(lay, 40 + r)
        a0, a1 = int(lay.aux_offset[0]), int(lay.aux_offset[1])
        vals[a0 + 5] = 480.0; vals[a0 + 3000] = -480.0; vals[a0 + 9000:a0 + 9040] = 1e4     # top codes where quantized
        vals[a1 + 7] = 500.0
        if r == 1:
            vals[a0 + 12345] = np.nan; vals[a0 + 12346] = np.inf; vals[a0 + 20000] = -np.inf  # fp32 copy of variable 0
        arena, sb = oracle_arena(specs, mask, fmts, lay, vals)
        lays.append(lay); plans.append(plan); arenas.append(to_dev(arena)); sbs.append(to_dev(sb))
        for i, s in enumerate(specs):
            d = int(lay.data_offset[i])
            if mask[i]:
                of = orc.Format(4, 3)
                copies[i][r] = orc.decompress(arena[d:d + orc.packed_bytes(s.n, 8)], s.n, of, sb[i])
            else:
                copies[i][r] = arena[d:d + 4 * s.n].view(np.float32)
    agg = omc.omc_aggregate_plan_build(plans)
    out = torch.zeros(lays[0].aux_elems, device="cuda")
    omc.omc_aggregate_mean(agg, arenas, sbs, out)
    torch.cuda.synchronize()
    o = out.cpu().numpy()
    for i, s in enumerate(specs):
        a = int(lays[0].aux_offset[i])
        want = orc.aggregate_mean(copies[i])
        got = o[a:a + s.n]
        nan = np.isnan(want)
        assert np.array_equal(np.isnan(got), nan)
        assert bits_equal(got[~nan], want[~nan])
    assert np.isnan(o[int(lays[0].aux_offset[0]) + 12345])


@pytest.mark.parametrize("R", [1, 4, 5, 8, 9])
@pytest.mark.parametrize("EM", [(4, 3), (3, 9)])
def test_parts_of_tails_and_batches_of_clients(R, EM):
    """Ragged tails around the 256 elements that one workgroup takes of them, all-fp32 variables around the 256 of one of their
    pieces, and numbers of clients around the batches whose loads are in flight together."""
    sizes = [1, 31, 255, 256, 257, 2047, 2048, 2049, 2048 + 511, 2 * 2048 + 1793, 5 * 2048]
    specs = [synth.VarSpec("w%d" % n, (n,), n, True) for n in sizes] + [synth.VarSpec("b%d" % n, (n,), n, False) for n in (1, 3, 255, 257, 1030, 4099)]
    rng = np.random.default_rng(R)
    masks = [np.array([s.is_matrix and (r == R - 1 or rng.random() < 0.6) for s in specs]) for r in range(R)]
    run_case(specs, [EM] * len(specs), masks)


@pytest.mark.parametrize("EM", [(3, 7), (2, 3), (5, 10)])
def test_more_work_items_than_the_chip_holds(EM):
    """More than 8192 items of full tiles, each one workgroup's, which goes on from tile to tile in the same LDS.  (Smaller sets share an item's tiles out.)
    Against the mean of what omc_decompress_set gives, which other tests hold to the oracle."""
    item = 4096 if EM != (2, 3) else 8192
    sizes = [5000 * item + 2048 + 5, 3300 * item + 77, 4097]
    gf = omc.fmt(*EM)
    plans, arenas, sbs, total = [], [], [], None
    for r, mask in enumerate(((True, True, False), (False, True, True))):
        at, table = 0, []
        aux = [sum((n + 3) // 4 * 4 for n in sizes[:i]) for i in range(4)]
        for i, n in enumerate(sizes):
            table.append(dict(data_offset=at, aux_offset=aux[i], n=n, fmt=gf, quantized=mask[i]))
            at += (omc.omc_packed_bytes(gf, n) if mask[i] else 4 * n) + 15 & ~15
        plan = omc.omc_plan_build(omc.make_var_table(table))
        w = torch.zeros(aux[3], device="cuda").normal_(0, 0.05, generator=torch.Generator(device="cuda").manual_seed(r))
        arena, sb = torch.zeros(at, dtype=torch.uint8, device="cuda"), torch.zeros((3, 2), device="cuda")
        omc.omc_compress_set(w, plan, arena, sb, torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda"))
        omc.omc_decompress_set(arena, plan, sb, w)
        total = w if total is None else total + w
        plans.append(plan), arenas.append(arena), sbs.append(sb)
    out = torch.full((aux[3],), float("nan"), device="cuda")
    omc.omc_aggregate_mean(omc.omc_aggregate_plan_build(plans), arenas, sbs, out)
    for i, n in enumerate(sizes):
        assert torch.equal(out[aux[i]:aux[i] + n], (total / 2)[aux[i]:aux[i] + n]), i
