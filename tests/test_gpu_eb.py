"""GPU parity of the ABFT-checked EmbeddingBag (include/abft_eb.h) against the CPU oracle
(oracle/eb_oracle.*), through the C ABI.

Bar: R is compared element by element with the operator's definition evaluated in double
(Section III-C) within the derived binary32 round-off tolerance - that is the parity claim; the
table's row sums and the batch kernel's CSum are bit-exact; RSum agrees to double rounding (the
kernels add the same doubles in a tree, the oracle in sequence); the flags are equal wherever the
oracle says the comparison cannot depend on that order, which the tests require to be everywhere
for their seeds.  On top of that R is checked bit for bit against a binary32 evaluation in the
kernels' documented order: a reproducibility check, not the oracle."""
import numpy as np
import pytest
import torch

from oracle import eb_oracle as eb
from paper_2103_00130_amd import eb_workloads as w

pytestmark = pytest.mark.gpu

VARIANTS = {"auto": 0, "batch": 0x100, "group": 0x200}


@pytest.fixture(scope="module")
def b():
    from paper_2103_00130_amd import binding
    assert torch.cuda.is_available()
    return binding


def dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


class GpuTable:
    def __init__(self, b, T, scale, bias, aligned=False, bits=8):
        self.b = b
        self.Tp = b.abft_eb_pack_rowsum(dev(T), dev(scale), dev(bias), (b.ABFT_EB_PACK_LINE_ALIGNED if aligned else 0) |
                                        (b.ABFT_EB_PACK_INT4 if bits == 4 else 0))
        torch.cuda.synchronize()

    def rowsums(self):
        out = torch.empty(self.Tp.rows, dtype=torch.int32, device="cuda")
        self.b.abft_eb_table_get_rowsums(self.Tp, out)
        return out.cpu().numpy()

    def run(self, indices, offsets, weights=None, variant="auto", check=True, bound=1e-5, ldr=None):
        b, d = self.b, self.Tp.d
        n_bags = offsets.size - 1
        ldr = d if ldr is None else ldr
        Rbuf = torch.full((max(n_bags, 1), ldr), -7.0, dtype=torch.float32, device="cuda")
        R = Rbuf[:, :d]
        flags = torch.full((max(n_bags, 1),), -1, dtype=torch.int32, device="cuda")
        rsum = torch.full((max(n_bags, 1),), -1.0, dtype=torch.float64, device="cuda")
        csum = torch.full((max(n_bags, 1),), -1.0, dtype=torch.float64, device="cuda")
        b.abft_eb_u8_checked(self.Tp, dev(indices) if indices.size else torch.empty(0, dtype=torch.int64, device="cuda"),
                             dev(offsets), R[:n_bags] if n_bags else R[:0], flags, dev(weights), rsum, csum, bound,
                             VARIANTS[variant] | (0 if check else b.ABFT_EB_NOCHECK))
        torch.cuda.synchronize()
        return {"R": R[:n_bags].cpu().numpy(), "flags": flags[:n_bags].cpu().numpy(), "rsum": rsum[:n_bags].cpu().numpy(),
                "csum": csum[:n_bags].cpu().numpy(), "pad": Rbuf[:, d:].cpu().numpy()}


def same_bits(x, y):
    return np.array_equal(np.ascontiguousarray(x).view(np.uint32), np.ascontiguousarray(y).view(np.uint32))


def compare(out, ref, T, scale, bias, indices, offsets, weights, bits=8, csum_in_index_order=False):
    """THE PARITY BAR for R: element by element against the operator's definition evaluated in double
    (Section III-C: R = sum_i (alpha_i * eb_i + beta_i * e_d), `forward(..., "f64")`), within the
    round-off bound of a binary32 evaluation of that sum that roundoff_tolerance() derives.
    Row sums, flags: equal to the oracle's.  CSum: its terms are exact to one rounding on both sides; the
    batch kernel adds them in index order like the oracle (bit for bit), the group kernel adds them lanes
    in parallel, which moves the sum by at most m * 2^-53 * sum|term| (|term| <= d * (|scale| * code_max +
    |bias|): the magnitude roundoff_tolerance() is built on).  RSum: a binary64 sum of d binary32 values in
    the kernel's own order.
    After the parity checks, one REPRODUCIBILITY check that is not the oracle: R bit for bit against the
    binary32 evaluation in the one order the kernels document (one fused multiply-add per pooled row in
    index order, biases summed apart) - it pins that order from run to run and between the two kernels."""
    tol = eb.roundoff_tolerance(T, scale, bias, indices, offsets, weights, bits)
    R64 = eb.forward(T, scale, bias, indices, offsets, weights, "f64", bits)
    ok = np.isfinite(R64)
    assert np.array_equal(np.isfinite(out["R"]), ok)
    assert np.all(np.abs(out["R"].astype(np.float64) - R64)[ok] <= (tol[:, None] + np.zeros_like(R64))[ok] + 1e-30), \
        "R differs from the definition (double) by more than the binary32 round-off bound"
    if csum_in_index_order:
        assert np.array_equal(out["csum"].view(np.uint64), ref.csum.view(np.uint64)), "CSum differs"
    else:
        d = out["R"].shape[1]
        fin_c = np.isfinite(ref.csum)
        assert np.array_equal(np.isfinite(out["csum"]), fin_c)
        assert np.all(np.abs(out["csum"] - ref.csum)[fin_c] <= (tol * d * 2.0 ** -29)[fin_c]), "CSum differs"
    fin = np.isfinite(ref.rsum)
    assert np.allclose(out["rsum"][fin], ref.rsum[fin], rtol=1e-13, atol=0)
    assert ref.robust.all(), "seed gives a comparison that depends on summation order; pick another"
    assert np.array_equal(out["flags"], ref.flags)
    # reproducibility of the documented evaluation order (not the parity bar)
    assert same_bits(out["R"], ref.R), "R is not reproducible against the binary32 evaluation in the documented order"


@pytest.mark.parametrize("d", [16, 32, 64, 128, 256, 512])
@pytest.mark.parametrize("variant", ["batch", "group"])
def test_eb_matches_oracle(b, d, variant):
    for weighted, regime, lengths in ((False, "uniform", "spread"), (True, "gauss", "ragged"), (False, "integer", "ragged")):
        rng = w.rng_for(100 + d, 0, int(weighted))
        T, scale, bias = w.draw_table(rng, 3000, d, regime)
        indices, offsets = w.draw_bags(rng, 3000, 150, 40, lengths)
        # one lookup long enough to span several staging chunks of the group kernel at every d
        extra = rng.integers(0, 3000, size=1300, dtype=np.int64)
        indices = np.concatenate([indices, extra])
        offsets = np.concatenate([offsets, [indices.size]]).astype(np.int64)
        weights = w.draw_weights(rng, indices.size) if weighted else None
        aligned = regime == "gauss"     # one of the three passes runs on line-aligned records
        g = GpuTable(b, T, scale, bias, aligned)
        stride = {16: 32, 32: 64, 64: 128}.get(d, d + 16) if aligned else d + 16
        assert b.abft_eb_table_dims(g.Tp) == (3000, d, stride, 8)
        assert np.array_equal(g.rowsums(), eb.table_rowsums(T))
        ref = eb.checked_eb(T, scale, bias, indices, offsets, weights)
        out = g.run(indices, offsets, weights, variant)
        compare(out, ref, T, scale, bias, indices, offsets, weights, csum_in_index_order=variant == "batch")
        if regime != "gauss":
            assert not out["flags"].any()


def test_variants_agree_and_nocheck_is_the_same_lookup(b):
    rng = w.rng_for(7)
    T, scale, bias = w.draw_table(rng, 5000, 64, "gauss")
    indices, offsets = w.draw_bags(rng, 5000, 700, 30, "ragged")
    weights = w.draw_weights(rng, indices.size)
    g = GpuTable(b, T, scale, bias)
    outs = [g.run(indices, offsets, weights, v, check=c, ldr=72) for v in ("batch", "group") for c in (True, False)]
    for o in outs[1:]:
        assert same_bits(o["R"], outs[0]["R"])
        assert np.all(o["pad"] == -7.0)          # columns past d are not written
    assert np.array_equal(outs[0]["flags"], outs[2]["flags"])
    assert not outs[1]["flags"].any() and not outs[3]["flags"].any()   # no check: only bad indices are reported
    assert np.all(outs[1]["rsum"] == -1.0)                              # and the diagnostics are left alone


def test_bad_indices_empty_batches_and_clamped_offsets(b):
    rng = w.rng_for(8)
    T, scale, bias = w.draw_table(rng, 100, 32, "uniform")
    g = GpuTable(b, T, scale, bias)
    indices = np.array([5, 100, 7, -3, 9, 2**40, 11, 12], dtype=np.int64)
    offsets = np.array([0, 2, 2, 5, 8], dtype=np.int64)
    ref = eb.checked_eb(T, scale, bias, indices, offsets)
    assert ref.flags.tolist() == [2, 0, 2, 2]
    for v in ("batch", "group"):
        out = g.run(indices, offsets, None, v)
        assert same_bits(out["R"], ref.R) and np.array_equal(out["flags"], ref.flags)
        assert np.all(out["R"][1] == 0.0)
        nc = g.run(indices, offsets, None, v, check=False)
        assert nc["flags"].tolist() == [2, 0, 2, 2]
        # offsets beyond the index array are clamped: the last lookup pools what exists
        wild = np.array([0, 2, 2, 5, 1000], dtype=np.int64)
        out = g.run(indices, wild, None, v)
        assert same_bits(out["R"], ref.R)
        # no lookups at all
        empty = g.run(np.zeros(0, dtype=np.int64), np.zeros(1, dtype=np.int64), None, v)
        assert empty["R"].shape == (0, 32)
        # only empty lookups
        out = g.run(np.zeros(0, dtype=np.int64), np.zeros(6, dtype=np.int64), None, v)
        assert np.all(out["R"] == 0.0) and not out["flags"].any()
    with pytest.raises(b.AbftError):
        R = torch.empty((4, 32), dtype=torch.float32, device="cuda")
        b.abft_eb_u8_checked(g.Tp, dev(indices), dev(offsets), R, None)    # flags are required when checking
    with pytest.raises(b.AbftError):
        R = torch.empty((4, 33), dtype=torch.float32, device="cuda")[:, :32]  # ldr not a multiple of 4
        b.abft_eb_u8_checked(g.Tp, dev(indices), dev(offsets), R, torch.empty(4, dtype=torch.int32, device="cuda"))


def test_non_finite_parameters_are_reported(b):
    rng = w.rng_for(9)
    T, scale, bias = w.draw_table(rng, 200, 64, "uniform")
    scale[17] = np.inf
    bias[23] = np.nan
    indices, offsets = w.draw_bags(rng, 200, 40, 20, "fixed")
    indices[5], indices[45] = 17, 23      # lookups 0 and 2
    g = GpuTable(b, T, scale, bias)
    ref = eb.checked_eb(T, scale, bias, indices, offsets)
    assert ref.flags[0] == 1 and ref.flags[2] == 1
    for v in ("batch", "group"):
        out = g.run(indices, offsets, None, v)
        assert np.array_equal(out["flags"], ref.flags)
        assert np.array_equal(np.isnan(out["R"]), np.isnan(ref.R))
        ok = ~np.isnan(ref.R)
        assert np.array_equal(out["R"][ok], ref.R[ok])


def test_zero_bound_and_threshold_on_integer_table(b):
    """Integer table: RSum and CSum are the same integer, so even bound 0 passes a clean lookup;
    a planted flip is caught or passed exactly as the closed form says."""
    rng = w.rng_for(10)
    T, scale, bias = w.draw_table(rng, 400, 64, "integer")
    indices, offsets = w.draw_bags(rng, 400, 6, 100, "fixed")
    g = GpuTable(b, T, scale, bias)
    C_T = eb.table_rowsums(T)
    for v in ("batch", "group"):
        assert not g.run(indices, offsets, None, v, bound=0.0)["flags"].any()
    bag0 = indices[offsets[0]:offsets[1]]
    row, col = int(next(i for i in bag0 if (bag0 == i).sum() == 1)), 5   # pooled exactly once by lookup 0
    for bit in range(8):
        b.abft_eb_table_flip_bit(g.Tp, row, col, bit)
        T2 = T.copy()
        T2[row, col] ^= np.uint8(1 << bit)
        ref = eb.checked_eb(T2, scale, bias, indices, offsets, C_T=C_T)
        for v in ("batch", "group"):
            out = g.run(indices, offsets, None, v)
            assert same_bits(out["R"], ref.R) and np.array_equal(out["flags"], ref.flags)
            assert out["flags"][0] == int(bit >= 4)     # CSum is about 816000: 1e-5 of it lies between 8 and 16
        b.abft_eb_table_flip_bit(g.Tp, row, col, bit)
    assert np.array_equal(g.rowsums(), C_T)
    assert not g.run(indices, offsets, None, "group")["flags"].any()


@pytest.mark.parametrize("regime", ["uniform", "gauss"])
def test_table_flip_campaign_matches_oracle(b, regime):
    """Section VI-B-2 at reduced size: 100 flips in the upper and 100 in the lower four bits of
    pooled table elements, one per launch, plus clean launches; every flag vector equals the oracle's."""
    wl = w.EbWorkload("campaign", 20000, 64, 10, 100, False, regime)
    x = w.make_inputs(wl, tag=20)
    g = GpuTable(b, x.T, x.scale, x.bias, aligned=(regime == "gauss"))
    C_T = eb.table_rowsums(x.T)
    clean = eb.checked_eb(x.T, x.scale, x.bias, x.indices, x.offsets)
    assert clean.robust.all()
    assert np.array_equal(g.run(x.indices, x.offsets, None, "auto")["flags"], clean.flags)
    rates = {}
    for bits in ("high", "low"):
        rng = w.rng_for(20, 0, 1 + (bits == "low"))
        f_row, f_col, f_bit = w.draw_table_flips(rng, x.indices, 64, 100, bits)
        want = eb.campaign_table_flips(x.T, x.scale, x.bias, C_T, x.indices, x.offsets, None, f_row, f_col, f_bit)
        got = np.empty_like(want)
        for t in range(100):
            b.abft_eb_table_flip_bit(g.Tp, f_row[t], f_col[t], f_bit[t])
            got[t] = g.run(x.indices, x.offsets, None, "auto")["flags"]
            b.abft_eb_table_flip_bit(g.Tp, f_row[t], f_col[t], f_bit[t])
        assert np.array_equal(got, want)
        rates[bits] = float((got != 0).any(axis=1).mean())
    print(f"\n[eb campaign, {regime}] detected: high bits {rates['high']:.0%}, low bits {rates['low']:.0%}, "
          f"false positives {float((clean.flags != 0).mean()):.0%}")
    assert rates["high"] >= rates["low"]
    assert np.array_equal(g.rowsums(), C_T)


@pytest.mark.parametrize("d", [64, 256])
def test_table1_shapes_full_size(b, d):
    """The benchmark's own configurations: 4,000,000 rows, pooling 100, batch 10 (Table I) and
    the large batch of 16384 lookups, weighted and not, in the variant the library picks."""
    x = w.make_inputs(w.TABLE1[d], tag=30 + d)
    g = GpuTable(b, x.T, x.scale, x.bias)
    C_T = eb.table_rowsums(x.T)
    sample = np.concatenate([np.arange(0, 4_000_000, 40_009), x.indices[:200]])
    assert np.array_equal(g.rowsums()[sample], C_T[sample])
    ref = eb.checked_eb(x.T, x.scale, x.bias, x.indices, x.offsets, C_T=C_T)
    compare(g.run(x.indices, x.offsets), ref, x.T, x.scale, x.bias, x.indices, x.offsets, None)
    rng = w.rng_for(30 + d, 1)
    indices, offsets = w.draw_bags(rng, 4_000_000, 16384 if d == 64 else 4096, 100, "spread")
    weights = w.draw_weights(rng, indices.size)
    for wts in (None, weights):
        ref = eb.checked_eb(x.T, x.scale, x.bias, indices, offsets, wts, C_T=C_T)
        compare(g.run(indices, offsets, wts), ref, x.T, x.scale, x.bias, indices, offsets, wts)


@pytest.mark.parametrize("d", [32, 64, 128, 256, 512, 1024])
@pytest.mark.parametrize("variant", ["batch", "group"])
def test_int4_tables_match_oracle(b, d, variant):
    """4-bit codes, two per byte: same bar as the 8-bit tables, plus flips of each of the four bits of
    codes in even and odd columns."""
    for weighted, regime, lengths, aligned in ((False, "uniform", "spread", False), (True, "gauss", "ragged", True)):
        rng = w.rng_for(200 + d, 0, int(weighted))
        T, scale, bias = w.draw_table(rng, 2000, d, regime, bits=4)
        assert T.shape == (2000, d // 2)
        indices, offsets = w.draw_bags(rng, 2000, 100, 40, lengths)
        extra = rng.integers(0, 2000, size=1300, dtype=np.int64)
        indices = np.concatenate([indices, extra])
        offsets = np.concatenate([offsets, [indices.size]]).astype(np.int64)
        weights = w.draw_weights(rng, indices.size) if weighted else None
        g = GpuTable(b, T, scale, bias, aligned, bits=4)
        stride = {16: 32, 32: 64, 64: 128}.get(d // 2, d // 2 + 16) if aligned else d // 2 + 16
        assert b.abft_eb_table_dims(g.Tp) == (2000, d, stride, 4)
        C_T = eb.table_rowsums(T, bits=4)
        assert np.array_equal(g.rowsums(), C_T)
        ref = eb.checked_eb(T, scale, bias, indices, offsets, weights, bits=4)
        compare(g.run(indices, offsets, weights, variant), ref, T, scale, bias, indices, offsets, weights, bits=4,
                csum_in_index_order=variant == "batch")
        for col, bit in ((0, 0), (1, 3), (d - 1, 2), (d // 2, 1)):
            row = int(indices[offsets[-2] + 5])
            b.abft_eb_table_flip_bit(g.Tp, row, col, bit)
            T2 = T.copy()
            T2[row, col // 2] ^= np.uint8(1 << (bit + 4 * (col & 1)))
            ref = eb.checked_eb(T2, scale, bias, indices, offsets, weights, C_T=C_T, bits=4)
            out = g.run(indices, offsets, weights, variant)
            assert same_bits(out["R"], ref.R)
            assert np.array_equal(out["flags"][ref.robust], ref.flags[ref.robust])
            b.abft_eb_table_flip_bit(g.Tp, row, col, bit)
        with pytest.raises(b.AbftError):
            b.abft_eb_table_flip_bit(g.Tp, 0, 0, 4)     # a 4-bit code has bits 0..3


def test_large_batch_takes_the_batch_kernel_by_itself(b):
    """70000 short lookups at d = 32: the library picks the batch kernel (lookups alone fill the chip);
    same bar as everywhere."""
    rng = w.rng_for(40)
    T, scale, bias = w.draw_table(rng, 50000, 32, "uniform")
    indices, offsets = w.draw_bags(rng, 50000, 70000, 6, "spread")
    weights = w.draw_weights(rng, indices.size)
    g = GpuTable(b, T, scale, bias)
    ref = eb.checked_eb(T, scale, bias, indices, offsets, weights)
    out = g.run(indices, offsets, weights, "auto")
    compare(out, ref, T, scale, bias, indices, offsets, weights, csum_in_index_order=True)   # (only the batch kernel does)
    assert same_bits(g.run(indices, offsets, weights, "group")["R"], out["R"])


def test_table_beyond_4_gib(b):
    """Record offsets that do not fit 32 bits: a table of 17,000,000 records of 272 bytes (4.6 GB) built
    on the device; the rows a batch pools are brought back and the oracle runs on that compacted table."""
    rows, d = 17_000_000, 256
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    T = torch.randint(0, 256, (rows, d), dtype=torch.uint8, device="cuda", generator=gen)
    scale = torch.rand(rows, device="cuda", generator=gen) * 0.015 + 0.005
    bias = -0.5 * torch.rand(rows, device="cuda", generator=gen)
    Tp = b.abft_eb_pack_rowsum(T, scale, bias)
    torch.cuda.synchronize()
    assert b.abft_eb_table_dims(Tp)[2] * rows > 2 ** 32
    rng = w.rng_for(41)
    indices, offsets = w.draw_bags(rng, rows, 300, 40, "spread")
    indices[:50] = rows - 1 - np.arange(50)              # the far end of the table
    uniq, inv = np.unique(indices, return_inverse=True)
    sel = torch.from_numpy(uniq).cuda()
    T_small, scale_small, bias_small = T[sel].cpu().numpy(), scale[sel].cpu().numpy(), bias[sel].cpu().numpy()
    del T
    ref = eb.checked_eb(T_small, scale_small, bias_small, inv.astype(np.int64), offsets)
    rowsums = torch.empty(rows, dtype=torch.int32, device="cuda")
    b.abft_eb_table_get_rowsums(Tp, rowsums)
    assert np.array_equal(rowsums[sel].cpu().numpy(), ref.C_T)
    for variant in ("group", "batch"):
        R = torch.empty((300, d), dtype=torch.float32, device="cuda")
        flags = torch.empty(300, dtype=torch.int32, device="cuda")
        b.abft_eb_u8_checked(Tp, dev(indices), dev(offsets), R, flags, flags=VARIANTS[variant])
        torch.cuda.synchronize()
        assert same_bits(R.cpu().numpy(), ref.R) and np.array_equal(flags.cpu().numpy(), ref.flags)
    # a planted fault at the far end is seen
    b.abft_eb_table_flip_bit(Tp, rows - 1, 255, 7)
    b.abft_eb_u8_checked(Tp, dev(indices), dev(offsets), R, flags)
    torch.cuda.synchronize()
    assert flags[0].item() == 1
    Tp.destroy()


# (one wavefront per lookup, two of them)
@pytest.mark.parametrize("n_bags,mean", [(1500, 20), (1100, 60)])
@pytest.mark.parametrize("code_bytes,bits", [(32, 8), (128, 4), (256, 8), (512, 4)])
def test_tables_whose_records_pass_the_caches_by(b, code_bytes, bits, n_bags, mean):
    """Tables just above 1.5 GiB: the same lookups as on a small table of the pooled rows, within the round-off bound of the definition and
    with the same bits, plain and weighted, checked and not; a planted fault and a bad index are reported."""
    d = code_bytes * 8 // bits
    rows = (3 << 29) // (code_bytes + 16) + 1
    gen = torch.Generator(device="cuda").manual_seed(code_bytes)
    T = torch.randint(0, 256, (rows, code_bytes), dtype=torch.uint8, device="cuda", generator=gen)
    scale = torch.rand(rows, device="cuda", generator=gen) * 0.015 + 0.005
    bias = -0.5 * torch.rand(rows, device="cuda", generator=gen)
    Tp = b.abft_eb_pack_rowsum(T, scale, bias, b.ABFT_EB_PACK_INT4 if bits == 4 else 0)
    torch.cuda.synchronize()
    assert (3 << 29) < b.abft_eb_table_dims(Tp)[2] * rows < (3 << 29) + 4096
    rng = w.rng_for(43 + mean, code_bytes)
    indices, offsets = w.draw_bags(rng, rows, n_bags, mean, "spread")
    indices[:20] = rows - 1 - np.arange(20)
    uniq, inv = np.unique(indices, return_inverse=True)
    inv = inv.astype(np.int64)
    sel = torch.from_numpy(uniq).cuda()
    small = T[sel].cpu().numpy(), scale[sel].cpu().numpy(), bias[sel].cpu().numpy()
    del T
    g = GpuTable.__new__(GpuTable)
    g.b, g.Tp = b, Tp
    for weights in (None, w.draw_weights(rng, indices.size)):
        ref = eb.checked_eb(*small, inv, offsets, weights, bits=bits)
        compare(g.run(indices, offsets, weights), ref, *small, inv, offsets, weights, bits)
        assert same_bits(g.run(indices, offsets, weights, check=False)["R"], ref.R)
    wrong = indices.copy()
    wrong[int(offsets[7])] = rows
    b.abft_eb_table_flip_bit(Tp, int(indices[0]), d - 1, 3 if bits == 4 else 7)
    flags = g.run(wrong, offsets, weights)["flags"]
    assert flags[0] & 1 and flags[7] & b.ABFT_EB_BAD_INDEX
    Tp.destroy()


@pytest.mark.parametrize("n_bags,mean", [(2 ** 25 + 3, 47), (2 ** 26 + 3, 30)])
def test_more_lookups_than_wavefronts_in_a_launch(b, n_bags, mean):
    """So many lookups that one or two wavefronts each would be more work-items than a launch takes: the call runs all the same,
    and the variant that asks for four each is refused.  (The index array has `mean` entries per lookup, one of them pooled.)"""
    rows, d = 1000, 16
    g = torch.Generator("cuda").manual_seed(n_bags)
    T = torch.randint(0, 256, (rows, d), dtype=torch.uint8, device="cuda", generator=g)
    scale, bias = torch.rand(rows, device="cuda", generator=g), torch.rand(rows, device="cuda", generator=g) - 0.5
    Tp = b.abft_eb_pack_rowsum(T, scale, bias)
    indices = torch.zeros(n_bags * mean, dtype=torch.int64, device="cuda")
    indices[:n_bags] = torch.randint(0, rows, (n_bags,), device="cuda", generator=g)
    offsets = torch.arange(n_bags + 1, device="cuda")
    R, flags = torch.empty(n_bags, d, device="cuda"), torch.empty(n_bags, dtype=torch.int32, device="cuda")
    with pytest.raises(b.AbftError) as e:
        b.abft_eb_u8_checked(Tp, indices, offsets, R, flags, flags=VARIANTS["group"])
    assert e.value.code == b.ABFT_EUNSUPPORTED
    b.abft_eb_u8_checked(Tp, indices, offsets, R, flags)
    torch.cuda.synchronize()
    assert not flags.any()
    rows_f32 = scale[:, None] * T.float() + bias[:, None]      # (one row: a product and a sum, each rounded once)
    for at in range(0, n_bags, 1 << 22):
        assert torch.equal(R[at:at + (1 << 22)], rows_f32[indices[at:min(at + (1 << 22), n_bags)]])
    Tp.destroy()


# (numbers of lookups and mean lengths on either side of every line of the choice; the lengths themselves sit at the edges
# of the eight rows that are pooled at a time and of the chunks that are staged)
@pytest.mark.parametrize("n_bags,mean", [(999, 10), (40, 30), (999, 17), (1000, 40), (1000, 60), (6000, 4), (16000, 9), (5999, 5)])
@pytest.mark.parametrize("code_bytes,bits", [(16, 8), (32, 4), (64, 8), (64, 4), (128, 8), (256, 4), (512, 8)])
def test_every_choice_by_size(b, code_bytes, bits, n_bags, mean):
    """The kernel that the library picks by itself, with and without weights: every one within the round-off bound of the
    definition, with the same bits as the documented order, bad indices reported and left out."""
    d = code_bytes * 8 // bits
    if n_bags * mean * d > 40_000_000:
        mean = 6     # (wide rows: the same side of the line with shorter lookups)
    rng = w.rng_for(60 + code_bytes + bits, n_bags + mean)
    rows = 4000
    T, scale, bias = w.draw_table(rng, rows, d, "uniform", bits)
    n = rng.integers(max(mean // 2, 0), mean + mean // 2 + 1, size=n_bags)
    edge = np.array([0, 1, 7, 8, 9, 16, 17, 24, 31, 33, 56, 57, 96, 97, 104, 105, 120, 128, 129, 200, 201, 208, 700])
    n[1:1 + len(edge)] = edge
    offsets = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    indices = rng.integers(0, rows, size=int(offsets[-1]), dtype=np.int64)
    g = GpuTable(b, T, scale, bias, aligned=bits == 4, bits=bits)
    for weights in (None, w.draw_weights(rng, indices.size)):
        ref = eb.checked_eb(T, scale, bias, indices, offsets, weights, bits=bits)
        compare(g.run(indices, offsets, weights), ref, T, scale, bias, indices, offsets, weights, bits)
        assert same_bits(g.run(indices, offsets, weights, check=False)["R"], ref.R)
    # bad indices: at the start of a lookup, in its last row, and a lookup of nothing else
    wrong = indices.copy()
    wrong[[int(offsets[5]), int(offsets[24]) - 1, int(offsets[2])]] = [rows, -1, 2 ** 40]
    out = g.run(wrong, offsets, weights)
    flagged = np.zeros(n_bags, dtype=bool)
    flagged[[5, 23, 2]] = True
    assert np.array_equal((out["flags"] & b.ABFT_EB_BAD_INDEX) != 0, flagged)
    keep = np.ones(indices.size, dtype=bool)
    keep[[int(offsets[5]), int(offsets[24]) - 1, int(offsets[2])]] = False
    left = np.concatenate([[0], np.cumsum(keep)])[offsets].astype(np.int64)
    ref = eb.checked_eb(T, scale, bias, indices[keep], left, weights[keep], bits=bits)
    assert same_bits(out["R"], ref.R)


# (a chunk of four wavefronts holds 512, 341, 204, 113, 120 and 62 rows of 16, 32, .. 512 bytes, one of two wavefronts 256, 168, 96, 56,
# 56 and 24, one of one 128, 80, 96, 56, 24 and 24: lookups of one row less and more than one and two of them; four wavefronts are
# asked for, one and two are chosen for many lookups, short ones and long ones)
@pytest.mark.parametrize("code_bytes,bits", [(16, 8), (32, 4), (64, 8), (64, 4), (128, 8), (256, 4), (256, 8), (512, 8), (512, 4)])
@pytest.mark.parametrize("fill,variant", [(None, "group"), (20, "auto"), (48, "auto")])
def test_chunk_edges(b, code_bytes, bits, fill, variant):
    """R with the same bits as the documented order, bad indices in the first and last rows of chunks reported and left out."""
    d = code_bytes * 8 // bits
    G = code_bytes // 16
    four = (8 if G >= 16 else 4) * 256 // (G + 1)
    two = (8 if G >= 16 else 4) * 128 // (G + 1) // 8 * 8
    one = (16 if G >= 32 else 8 if G >= 4 else 4) * 64 // (G + 1) // 8 * 8
    n = sorted({max(m * c + o, 1) for c in (four, two, one) for m in (1, 2) for o in (-1, 0, 1, 2)})
    if fill is not None:
        n += [fill] * (1700 if G < 32 else 4100)
    rng = w.rng_for(90 + code_bytes + bits, len(n))
    rows = 3000
    T, scale, bias = w.draw_table(rng, rows, d, "uniform", bits)
    offsets = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    indices = rng.integers(0, rows, size=int(offsets[-1]), dtype=np.int64)
    g = GpuTable(b, T, scale, bias, bits=bits)
    for weights in (None, w.draw_weights(rng, indices.size)):
        ref = eb.checked_eb(T, scale, bias, indices, offsets, weights, bits=bits)
        compare(g.run(indices, offsets, weights, variant), ref, T, scale, bias, indices, offsets, weights, bits)
    wrong = indices.copy()
    hit = [int(offsets[3]), int(offsets[6]) - 1, int(offsets[8]) + min(four, n[8]) - 1]
    wrong[hit] = [rows, -1, 2 ** 40]
    out = g.run(wrong, offsets, weights, variant)
    flagged = np.zeros(len(n), dtype=bool)
    flagged[[3, 5, 8]] = True
    assert np.array_equal((out["flags"] & b.ABFT_EB_BAD_INDEX) != 0, flagged)
    keep = np.ones(indices.size, dtype=bool)
    keep[hit] = False
    left = np.concatenate([[0], np.cumsum(keep)])[offsets].astype(np.int64)
    assert same_bits(out["R"], eb.checked_eb(T, scale, bias, indices[keep], left, weights[keep], bits=bits).R)


def test_operands_of_the_native_call(b, monkeypatch):
    """The natively marshalled lookup takes what the Python code takes and leaves to it, errors and all, what it does not: the
    native function says which (a return code, or None)."""
    native, said = b._fastcall.eb, []

    def watched(*args):
        said.append(native(*args))
        return said[-1]
    monkeypatch.setattr(b._fastcall, "eb", watched)
    rows, d, n = 500, 64, 20
    rng = w.rng_for(7, 1)
    T, scale, bias = w.draw_table(rng, rows, d, "uniform", 8)
    offsets = np.arange(n + 1, dtype=np.int64) * 5
    indices = rng.integers(0, rows, size=5 * n, dtype=np.int64)
    weights = w.draw_weights(rng, indices.size)
    g = GpuTable(b, T, scale, bias)
    i, o, wt = dev(indices), dev(offsets), dev(weights)
    R, flags = torch.zeros(n, d, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
    sums = torch.zeros(n, dtype=torch.float64, device="cuda")
    wide = torch.zeros(n + 1, d + 4, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    call = b.abft_eb_u8_checked
    for weighted, out, stream in ((None, R, None), (wt, R, side), (wt, wide[:, :d], None)):
        call(g.Tp, i, o, out, flags, weighted, sums, sums.clone(), stream=stream)
        assert said.pop() == b.ABFT_OK
        torch.cuda.synchronize()
        want = eb.checked_eb(T, scale, bias, indices, offsets, None if weighted is None else weights)
        assert same_bits(out[:n].cpu().numpy(), want.R) and np.array_equal(flags.cpu().numpy(), want.flags)
    call(g.Tp, i, o, R, None, flags=b.ABFT_EB_NOCHECK)
    assert said.pop() == b.ABFT_OK
    for args, kw, error in (((i.int(), o, R, flags), {}, TypeError), ((i.cpu(), o, R, flags), {}, TypeError), ((i, o[::2], R, flags), {}, ValueError),
                            ((i, o, R[:, :-1], flags), {}, ValueError), ((i, o, R[:-1], flags), {}, ValueError), ((i, o, R.double(), flags), {}, TypeError),
                            ((i, o, R, flags[:-1]), {}, ValueError), ((i, o, R, flags.float()), {}, TypeError), ((i, o, R, flags, wt[:-1]), {}, ValueError),
                            ((i, o, R, flags, wt.double()), {}, TypeError), ((i, o, R, flags), {"rsum": sums.float()}, TypeError),
                            ((i, o, R, flags), {"csum": sums[:-1]}, ValueError)):
        with pytest.raises(error):
            call(g.Tp, *args, **kw)
        assert said.pop() is None
    for args, kw in (((i, o, R, None), {}), ((i, o, R, flags), {"flags": 0x300}), ((i, o, R, flags), {"rel_bound": -1.0}), ((i, o, wide[:, 1:1 + d], flags), {})):
        with pytest.raises(b.AbftError) as e:
            call(g.Tp, *args, **kw)
        assert e.value.code == b.ABFT_EINVAL and said.pop() == b.ABFT_EINVAL
    call(g.Tp, i, o, R, flags, flags=np.int64(0))     # (a number that is no plain int)
    call(g.Tp, i, o, R, flags, rel_bound=np.float32(1e-5))
    assert said == [None, None]
    torch.cuda.synchronize()
    assert same_bits(R.cpu().numpy(), eb.checked_eb(T, scale, bias, indices, offsets, None).R)
