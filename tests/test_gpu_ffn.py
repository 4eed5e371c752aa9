"""End-to-end parity of elas_lowrank_ffn_fwd / elas_lowrank_ffn_bwd with the
oracle (bf16 inputs, fp32 accumulation).

* Mask gate: every group where the GPU's 2:4 mask differs from the oracle's
  must be the stable top-2 of some h that binary32 accumulation of the up
  projection can produce (oracle.bounds.h_range, a bound derived from the
  arithmetic); disagreements beyond the 1e-2 relative window on the
  oracle's keys are counted and reported.
* Numeric gate: relative Frobenius error <= 2e-2 for Y, dx, P, Z and the
  four weight gradients against the oracle with the same bf16 rounding
  points; with ``legs`` also against the plain float64 block with the same
  selection (gate 2e-2) and with its own selection (reported only).
* Dense activations: every GPU value of s lies in the range the
  accumulation bound allows.
* Inputs for which every binary32 sum of the block is exact (checked from
  the oracle's intermediates): every output, including the four fp32 weight
  gradients, matches the oracle bit for bit.
* Small token counts at the 1B shape exercise the wave-split kernel (256, 512)
  and the split-K 128 x 128 tiles (1100, 3000) in every activation mode; T = 4096
  at the 1B shape runs the weight gradients over every token.
* Full-size workloads run in the benchmarked configuration: the 1B shape is
  checked on every token and group; the others on sampled tokens (every
  output row depends only on its own token, and the weight gradients are
  checked with dY zero outside the sampled tokens, so that they are exact
  sums over those tokens).
"""
import numpy as np
import pytest
import torch

import paper_2605_03667_amd as elas
from oracle import bf16 as obf
from oracle import bounds as obd
from oracle import ffn as offn
from oracle import sparsify as osp
from synthetic import (CONFIGS, config_inputs, exact_p_inputs, ffn_inputs, sparse_sign_bf16,
                       uniform_int_bf16)
from tests.helpers import check_padding, dev_bf16, host_bits, mask_gate, rel_fro, s_in_range, untile

pytestmark = pytest.mark.gpu

TOL = 2e-2
GRADS = ("dU_up", "dV_up", "dU_down", "dV_down")


def run_gpu(bits, rows=None, mode="sparse", fwd_flags=0):
    """Forward + backward through the C ABI; returns host copies (float64 for
    numbers) of the outputs, restricted to the token rows ``rows`` if given.
    mode: "sparse" (default), "ste" (sparse forward, Eq. 4 backward) or
    "dense" (dense activations); fwd_flags are or-ed into the forward's flags
    (ELAS_FWD_FUSED / ELAS_FWD_UNFUSED)."""
    fflags = (elas.ELAS_MODE_DENSE if mode == "dense" else 0) | fwd_flags
    bflags = {"sparse": 0, "ste": elas.ELAS_BWD_STE, "dense": elas.ELAS_MODE_DENSE}[mode]
    t = {k: dev_bf16(v) for k, v in bits.items()}
    fwd = elas.elas_lowrank_ffn_fwd(t["x"], t["U_up"], t["V_up"], t["U_down"], t["V_down"], flags=fflags)
    bwd = elas.elas_lowrank_ffn_bwd(t["dY"], t["x"], t["U_up"], t["V_up"], t["U_down"], t["V_down"], fwd,
                                    flags=bflags)
    torch.cuda.synchronize()
    del t
    F = bits["V_up"].shape[1]
    idx = None if rows is None else torch.as_tensor(rows, device="cuda:0")

    def rows_of(x):
        return x if idx is None else x.index_select(0, idx)

    T = bits["x"].shape[0]
    # the compressed S is tiled (include/elas.h); the dense one is row-major
    sv = fwd["s_vals"] if mode == "dense" else untile(fwd["s_vals"], T, fwd["s_vals"].shape[1], 32)
    out = {
        "Y": obf.to_f64(host_bits(rows_of(fwd["y"]))), "P": obf.to_f64(host_bits(rows_of(fwd["P"]))),
        "Z": obf.to_f64(host_bits(rows_of(fwd["Z"]))), "dx": obf.to_f64(host_bits(rows_of(bwd["dx"]))),
        "s_vals": host_bits(rows_of(sv)),
    }
    for k in GRADS:
        out[k] = bwd[k].cpu().numpy().astype(np.float64)
    if mode == "dense":
        out["S"] = obf.to_f64(out["s_vals"])
        out["mask"] = np.ones(out["S"].shape, dtype=bool)
    else:
        out["s_meta"] = rows_of(untile(fwd["s_meta"], T, fwd["s_meta"].shape[1], 8)).cpu().numpy()
        check_padding(out["s_vals"], out["s_meta"], F)
        dense, mask = osp.decompress(out["s_vals"][:, : F // 2], out["s_meta"][:, : F // 8], F)
        out["mask"] = mask
        out["S"] = obf.to_f64(dense)
    del fwd, bwd
    return out


def h_range_of(bits):
    """h_range(rows, cols) of the inputs (oracle.bounds)."""
    a = offn.from_bits({k: bits[k] for k in ("x", "U_up", "V_up")})
    return lambda rows, cols: obd.h_range(a["x"], a["U_up"], a["V_up"], rows, cols)


def compare(gpu, f, b, bits, grads=True, report=None, legs=False, mode="sparse"):
    """Mask gate and numeric gate (gpu, oracle and bits hold the same token
    rows).  legs: also the plain float64 block with the oracle's selection
    (gated) and with its own selection (reported)."""
    gate = mask_gate(gpu["mask"], f["mask"], f["s"], h_range_of(bits))
    assert gate["unexplained"] == 0, f"mask disagreements the accumulation bound does not explain: {gate}"
    if mode == "dense":
        a = offn.from_bits({k: bits[k] for k in ("x", "U_up", "V_up")})
        assert s_in_range(gpu["S"], *obd.s_range(*obd.h_range(a["x"], a["U_up"], a["V_up"])))
    errs = {"Y": rel_fro(gpu["Y"], f["Y"]), "dx": rel_fro(gpu["dx"], b["dx"]),
            "P": rel_fro(gpu["P"], f["P"]), "Z": rel_fro(gpu["Z"], f["Z"])}
    if grads:
        for k in GRADS:
            errs[k] = rel_fro(gpu[k], b[k])
    if legs:
        sparse, ste = mode != "dense", mode == "ste"
        f2, b2 = offn.run(bits, bf16io=False, sparse=sparse, ste=ste, mask=f["mask"])
        f3, b3 = offn.run(bits, bf16io=False, sparse=sparse, ste=ste)
        for tag, ff, bb in (("f64_same_mask", f2, b2), ("f64_own_mask", f3, b3)):
            errs[f"{tag}:Y"] = rel_fro(gpu["Y"], ff["Y"])
            errs[f"{tag}:dx"] = rel_fro(gpu["dx"], bb["dx"])
            if grads:
                for k in GRADS:
                    errs[f"{tag}:{k}"] = rel_fro(gpu[k], bb[k])
    rep = dict(errs, **gate)
    if report is not None:
        report.update(rep)
    print("parity", {k: (f"{v:.2e}" if isinstance(v, float) else v) for k, v in rep.items()})
    for k, e in errs.items():
        if not k.startswith("f64_own_mask"):      # the own-selection leg is reported only
            assert e <= TOL, (k, e, errs)
    return errs


def all_sums_exact(bits, f, b):
    """True when every product of the block (forward and backward) sums
    exactly in binary32 in any order and the masked dH product is a binary32
    value: then the GPU's fp32 sums equal the oracle's float64 ones and every
    bf16 rounding sees the same value (oracle.bounds.exact_product)."""
    a = offn.from_bits(bits)
    prods = [(a["x"], a["U_up"]), (f["P"], a["V_up"]), (f["S"], a["U_down"]), (f["Z"], a["V_down"]),
             (a["dY"], a["V_down"].T), (f["Z"].T, a["dY"]), (b["dZ"], a["U_down"].T), (f["S"].T, b["dZ"]),
             (b["dH"], a["V_up"].T), (f["P"].T, b["dH"]), (a["x"].T, b["dP"]), (b["dP"], a["U_up"].T)]
    if not all(np.all(obd.exact_product(A, B)) for A, B in prods):
        return False
    g = b["dS"] * 2.0 * np.where(f["H"] > 0, f["H"], 0.0)
    return bool(np.all(g.astype(np.float32).astype(np.float64) == g))


def assert_bit_exact(gpu, f, b, F):
    """Every output equals the oracle's: P, Z, Y, dx, the kept values, the
    metadata and the four fp32 weight gradients."""
    for k in ("P", "Z", "Y"):
        np.testing.assert_array_equal(gpu[k], f[k], err_msg=k)
    np.testing.assert_array_equal(gpu["dx"], b["dx"], err_msg="dx")
    ref_vals, ref_meta = osp.compress(obf.from_f64(f["S"]), f["mask"])
    np.testing.assert_array_equal(gpu["s_meta"][:, : F // 8], ref_meta)
    np.testing.assert_array_equal(gpu["s_vals"][:, : F // 2], ref_vals)
    for k in GRADS:
        np.testing.assert_array_equal(gpu[k], b[k], err_msg=k)


def sparse_sign_inputs(T, d, F, r, density, scale_log2, seed):
    """x, U_up, V_up, U_down, V_down, dY as sparse +-2**scale (densities and
    scales in that order): small exact values for the bit-exact tests."""
    names = ["x", "U_up", "V_up", "U_down", "V_down", "dY"]
    shapes = [(T, d), (d, r), (r, F), (F, r), (r, d), (T, d)]
    return {n: sparse_sign_bf16(shp, de, seed + i, sc)
            for i, (n, shp, de, sc) in enumerate(zip(names, shapes, density, scale_log2))}


def exact_int_inputs(T, d, F, r):
    return {
        "x": uniform_int_bf16((T, d), -1, 1, 1), "U_up": uniform_int_bf16((d, r), -1, 1, 2),
        "V_up": uniform_int_bf16((r, F), -1, 1, 3), "U_down": uniform_int_bf16((F, r), -1, 1, 4, -12),
        "V_down": uniform_int_bf16((r, d), -1, 1, 5, -4), "dY": uniform_int_bf16((T, d), -1, 1, 6),
    }


@pytest.mark.parametrize("T,d,F,r", [(5, 16, 24, 8), (1, 64, 64, 16), (700, 136, 1000, 72),
                                     (256, 256, 256, 256), (300, 512, 1376, 128), (129, 768, 2048, 256),
                                     (16417, 128, 320, 256)])
def test_small_shapes(T, d, F, r):
    bits = ffn_inputs(T, d, F, r, seed_base=T + d if T != 16417 else T + 7 * d)
    f, b = offn.run(bits)
    compare(run_gpu(bits), f, b, bits)


@pytest.mark.parametrize("cfg", ["llama60m"])
def test_llama60m_full(cfg):
    bits = config_inputs(cfg)
    f, b = offn.run(bits)
    compare(run_gpu(bits), f, b, bits, legs=True)


@pytest.mark.parametrize("cfg", ["llama130m", "llama350m", "llama1b"])
def test_model_shapes_reduced_tokens(cfg):
    bits = config_inputs(cfg, T=1024)
    f, b = offn.run(bits)
    compare(run_gpu(bits), f, b, bits, legs=True)


def test_exact_fused_epilogue():
    """Small integers for which every sum of the block is exact in binary32:
    every output, the four fp32 weight gradients included, is bit-exact."""
    T, d, F, r = 700, 64, 1000, 40
    bits = exact_int_inputs(T, d, F, r)
    f, b = offn.run(bits)
    assert all_sums_exact(bits, f, b)
    gpu = run_gpu(bits)
    assert_bit_exact(gpu, f, b, F)
    compare(gpu, f, b, bits)


def test_exact_1b_shape_every_token():
    """The 1B shape at T = 4096 with sparse +-1 inputs whose every sum is exact
    in binary32: every output, including the four fp32 weight gradients (sums
    over every token), must match the oracle bit for bit."""
    T, d, F, r = 4096, 2048, 5464, 512
    bits = sparse_sign_inputs(T, d, F, r, [1 / 16, 1 / 16, 1 / 64, 1 / 8, 1 / 8, 1 / 4], [0, 0, 0, -8, -4, 0], 51)
    bits["V_up"][:, 5461:] = 0
    bits["U_down"][5461:, :] = 0
    f, b = offn.run(bits)
    assert all_sums_exact(bits, f, b)
    gpu = run_gpu(bits)
    assert_bit_exact(gpu, f, b, F)
    for k in GRADS:
        assert np.mean(b[k] != 0) > 0.99, k          # the gradients are dense: every token contributes


def test_all_h_nonpositive_gives_exact_zeros():
    T, d, F, r = 300, 64, 136, 24
    bits = ffn_inputs(T, d, F, r, seed_base=5)
    bits["x"] = bits["x"] & np.uint16(0x7FFF)
    bits["U_up"] = bits["U_up"] & np.uint16(0x7FFF)
    bits["V_up"] = bits["V_up"] | np.uint16(0x8000)
    gpu = run_gpu(bits)
    assert np.all(gpu["Y"] == 0) and np.all(gpu["dx"] == 0)
    for k in GRADS:
        assert np.all(gpu[k] == 0), k


def test_deterministic():
    bits = ffn_inputs(700, 136, 1000, 72, seed_base=3)
    a, b = run_gpu(bits), run_gpu(bits)
    for k in ("Y", "dx", "s_vals", "s_meta") + GRADS:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


def _sample_rows(T, n, seed):
    g = np.random.default_rng(seed)
    return np.unique(np.concatenate([[0, T - 1], g.integers(0, T, n)]))


@pytest.mark.parametrize("cfg", ["llama130m", "llama350m", "llama1b", "llama1b_t262144"])
def test_full_size_sampled(cfg):
    bits = config_inputs(cfg)
    T = CONFIGS[cfg]["T"]
    rows = _sample_rows(T, 94, 1)
    # outputs per token: y, dx, saved P and Z, the mask
    sub = {k: (v[rows] if k in ("x", "dY") else v) for k, v in bits.items()}
    f, b = offn.run(sub)
    gpu = run_gpu(bits, rows)
    rep = {}
    compare(gpu, f, b, sub, grads=False, report=rep)
    del gpu
    # weight gradients: dY zero outside the sampled tokens
    dY = np.zeros_like(bits["dY"])
    dY[rows] = bits["dY"][rows]
    bits["dY"] = dY
    gpu = run_gpu(bits, rows)
    sub["dY"] = dY[rows]
    f, b = offn.run(sub)
    for k in GRADS:
        e = rel_fro(gpu[k], b[k])
        rep[k] = e
        assert e <= TOL, (k, e)
    print(cfg, rep)


@pytest.mark.parametrize("inputs", ["llama1b", "llama1b_exact_p"])
def test_llama1b_every_token_and_group(inputs):
    """The 1B workload in the benchmarked configuration (T = 65536 tokens),
    checked everywhere: the mask gate on all 89.5 M groups, the kept values
    against the range of s the accumulation bound allows, Y, P, Z and dx on
    every row, and the four weight gradients as sums over every token.  The
    oracle runs on chunks of tokens.  ``llama1b_exact_p``: the same shapes and
    distributions with x and U_up drawn on grids that make P exact in
    binary32 (synthetic.exact_p_inputs), so that the accumulation range of
    the mask gate covers H's own sum only."""
    c = CONFIGS["llama1b"]
    T, d, F, r = c["T"], c["d"], c["d_ff"], c["r"]
    bits = config_inputs("llama1b") if inputs == "llama1b" else exact_p_inputs(T, d, F, r, c["d_ff_true"], 3)
    t = {k: dev_bf16(v) for k, v in bits.items()}
    fwd = elas.elas_lowrank_ffn_fwd(t["x"], t["U_up"], t["V_up"], t["U_down"], t["V_down"])
    bwd = elas.elas_lowrank_ffn_bwd(t["dY"], t["x"], t["U_up"], t["V_up"], t["U_down"], t["V_down"], fwd)
    torch.cuda.synchronize()
    del t
    sv = untile(fwd["s_vals"], T, fwd["s_vals"].shape[1], 32)
    sm = untile(fwd["s_meta"], T, fwd["s_meta"].shape[1], 8)
    a = offn.from_bits({k: bits[k] for k in ("x", "U_up", "V_up")})
    sq = {k: [0.0, 0.0] for k in ("Y", "P", "Z", "dx")}
    gref = {k: 0.0 for k in GRADS}
    tot = {"groups": 0, "flips": 0, "outside_rel": 0, "unexplained": 0}
    CH = 8192
    for t0 in range(0, T, CH):
        sub = {k: (v[t0:t0 + CH] if k in ("x", "dY") else v) for k, v in bits.items()}
        f, b = offn.run(sub)
        gpu = {"Y": obf.to_f64(host_bits(fwd["y"][t0:t0 + CH])), "P": obf.to_f64(host_bits(fwd["P"][t0:t0 + CH])),
               "Z": obf.to_f64(host_bits(fwd["Z"][t0:t0 + CH])), "dx": obf.to_f64(host_bits(bwd["dx"][t0:t0 + CH]))}
        ref = {"Y": f["Y"], "P": f["P"], "Z": f["Z"], "dx": b["dx"]}
        for k in sq:
            sq[k][0] += float(np.sum((gpu[k] - ref[k]) ** 2))
            sq[k][1] += float(np.sum(ref[k] ** 2))
        for k in GRADS:
            gref[k] = gref[k] + b[k]
        vals, meta = host_bits(sv[t0:t0 + CH]), sm[t0:t0 + CH].cpu().numpy()
        check_padding(vals, meta, F)
        dense, mask = osp.decompress(vals[:, : F // 2], meta[:, : F // 8], F)
        xs = a["x"][t0:t0 + CH]
        gate = mask_gate(mask, f["mask"], f["s"],
                         lambda rows, cols: obd.h_range(xs, a["U_up"], a["V_up"], rows, cols))
        for k in tot:
            tot[k] += gate[k]
        s_lo, s_hi = obd.s_range(*obd.h_range(xs, a["U_up"], a["V_up"]))
        assert s_in_range(obf.to_f64(dense)[mask], s_lo[mask], s_hi[mask]), t0
        print(f"tokens {t0}..{t0 + CH}: {gate}", flush=True)
    errs = {k: (v[0] / v[1]) ** 0.5 for k, v in sq.items()}
    for k in GRADS:
        errs[k] = rel_fro(bwd[k].cpu().numpy().astype(np.float64), gref[k])
    print(inputs, "mask gate", tot, {k: f"{v:.2e}" for k, v in errs.items()})
    assert tot["unexplained"] == 0, tot
    for k, e in errs.items():
        assert e <= TOL, (k, e, errs)


def test_zero_tokens():
    """T = 0: the forward is a no-op and the backward writes zero weight
    gradients (over whatever the buffers held)."""
    d, F, r = 64, 136, 24
    bits = ffn_inputs(0, d, F, r, seed_base=9)
    t = {k: dev_bf16(v) for k, v in bits.items()}
    fwd = elas.elas_lowrank_ffn_fwd(t["x"], t["U_up"], t["V_up"], t["U_down"], t["V_down"])
    grads = {"dx": torch.empty((0, d), dtype=torch.bfloat16, device="cuda:0")}
    for k, shp in (("dU_up", (d, r)), ("dV_up", (r, F)), ("dU_down", (F, r)), ("dV_down", (r, d))):
        grads[k] = torch.full(shp, float("nan"), dtype=torch.float32, device="cuda:0")
    elas.elas_lowrank_ffn_bwd(t["dY"], t["x"], t["U_up"], t["V_up"], t["U_down"], t["V_down"], fwd,
                              grads=grads)
    torch.cuda.synchronize()
    for k in GRADS:
        assert torch.all(grads[k] == 0), k


@pytest.mark.parametrize("mode", ["sparse", "dense", "ste"])
@pytest.mark.parametrize("T", [256, 512, 1100, 3000])
def test_small_token_counts_1b_shape(mode, T):
    """The 1B shape at token counts where the long-K products split K over waves
    (256, 512) or over the CUs (fp32 partials reduced to bf16; 1100, 3000) and
    the K = T products use 128 x 128 tiles: parity with the oracle in each
    activation mode."""
    bits = config_inputs("llama1b", T=T, seed_base=60 + T)
    f, b = offn.run(bits, sparse=(mode != "dense"), ste=(mode == "ste"))
    compare(run_gpu(bits, mode=mode), f, b, bits, mode=mode)


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("T,d,F,r,cfg", [(700, 136, 1000, 72, None), (1024, 2048, 5464, 512, "llama1b"),
                                         (256, 2048, 5464, 512, "llama1b")])
def test_factors_ab_identical(T, d, F, r, cfg, dense):
    """ELAS_FACTORS_AB (factors passed as the A, B of Eq. 1, i.e. transposed)
    reads the same operands as the copies the default forward makes, with the
    unpadded d_ff read as zero beyond its end: every output is bit-identical."""
    bits = config_inputs(cfg, T=T) if cfg else ffn_inputs(T, d, F, r, seed_base=3)
    t = {k: dev_bf16(v) for k, v in bits.items()}
    mode = elas.ELAS_MODE_DENSE if dense else 0
    ref = elas.elas_lowrank_ffn_fwd(t["x"], t["U_up"], t["V_up"], t["U_down"], t["V_down"], flags=mode)
    tr = {k: t[k].t().contiguous() for k in ("U_up", "V_up", "U_down", "V_down")}
    got = elas.elas_lowrank_ffn_fwd(t["x"], tr["U_up"], tr["V_up"], tr["U_down"], tr["V_down"],
                                    flags=mode | elas.ELAS_FACTORS_AB)
    torch.cuda.synchronize()
    for k in ("y", "P", "s_vals", "s_meta", "Z"):
        if ref[k] is None:
            continue
        assert torch.equal(ref[k].view(torch.int16) if ref[k].dtype == torch.bfloat16 else ref[k],
                           got[k].view(torch.int16) if got[k].dtype == torch.bfloat16 else got[k]), k


@pytest.mark.parametrize("T,d,F,r", [(64, 64, 65536, 16), (40, 65536, 64, 8)])
def test_maximum_widths(T, d, F, r):
    """d_ff and d at the ABI's maximum (65536): 32 Ki kept values per row,
    1024-step contractions, the long-K split of the forward and backward."""
    bits = ffn_inputs(T, d, F, r, seed_base=7)
    f, b = offn.run(bits)
    compare(run_gpu(bits), f, b, bits)


@pytest.mark.parametrize("mode", ["dense", "ste"])
@pytest.mark.parametrize("T,d,F,r", [(5, 16, 24, 8), (700, 136, 1000, 72), (300, 512, 1376, 128),
                                     (129, 2048, 5464, 512)])
def test_modes_small(mode, T, d, F, r):
    """Dense activations (the paper's warm-up phase) and the straight-through
    backward of Eq. 4, against the oracle in the same mode."""
    bits = ffn_inputs(T, d, F, r, seed_base=T + r)
    f, b = offn.run(bits, sparse=(mode != "dense"), ste=(mode == "ste"))
    compare(run_gpu(bits, mode=mode), f, b, bits, mode=mode)


@pytest.mark.parametrize("mode", ["dense", "ste"])
def test_modes_llama60m_full(mode):
    bits = config_inputs("llama60m")
    f, b = offn.run(bits, sparse=(mode != "dense"), ste=(mode == "ste"))
    compare(run_gpu(bits, mode=mode), f, b, bits, mode=mode, legs=True)


def test_ste_equals_masked_when_at_most_two_positives():
    """When every group has <= 2 positive h, pruned slots have relu(h) = 0, so
    the straight-through and masked backward agree (GPU vs GPU)."""
    T, d, F, r = 300, 64, 136, 8
    bits = ffn_inputs(T, d, F, r, seed_base=21)
    # H = P V_up with P's column 0 > 0 only and V_up row 0 signed (+ + - -) per group
    g = np.random.default_rng(5)
    x = np.zeros((T, d), dtype=np.float32); x[:, 0] = np.abs(g.standard_normal(T)) + 0.1
    U = np.zeros((d, r), dtype=np.float32); U[0, 0] = 1.0
    V = np.zeros((r, F), dtype=np.float32); V[0] = np.tile([1, 1, -1, -1], F // 4) * (np.abs(g.standard_normal(F)) + 0.1)
    to_bits = lambda a: (a.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    bits["x"], bits["U_up"], bits["V_up"] = to_bits(x), to_bits(U), to_bits(V)
    a, s = run_gpu(bits, mode="sparse"), run_gpu(bits, mode="ste")
    for k in ("dx",) + GRADS:
        assert rel_fro(s[k], a[k]) < 1e-2, k



@pytest.mark.parametrize("mode", ["sparse", "dense"])
def test_subnormal_activations_recover_relu(mode):
    """x scaled by c = 2^-64 (exact in bf16) scales h by c, so most stored
    s = bf16(h^2) are subnormal.  The backward recovers relu(h) from s as the
    correctly rounded bf16 square root, which for subnormal s needs the
    pre-scaled root (the raw one flushes them).  Expected: c times the
    oracle's backward at c = 1 with relu(h) replaced by that root / c at the
    GPU's kept positions; a flushing root would lose most of dx."""
    T, d, F, r = 300, 512, 1376, 128
    bits = ffn_inputs(T, d, F, r, seed_base=33)
    sparse = mode == "sparse"
    a = offn.from_bits(bits)
    f = offn.forward(a["x"], a["U_up"], a["V_up"], a["U_down"], a["V_down"], sparse=sparse)
    c = 2.0 ** -64
    scaled = dict(bits)
    scaled["x"] = obf.from_f64(a["x"] * c)
    assert np.array_equal(obf.to_f64(scaled["x"]), a["x"] * c)   # every scaled x is a normal bf16
    gpu = run_gpu(scaled, mode=mode)
    kept = gpu["S"][gpu["mask"]]
    assert np.mean(kept[kept > 0] < 2.0 ** -126) > 0.5, "most stored s should be subnormal"
    root = obf.to_f64(obf.from_f64(np.sqrt(gpu["S"])))   # relu(h) as the kernel recovers it

    def expected_dx(relu_h):
        fe = dict(f, H=relu_h / c, mask=gpu["mask"])
        return c * offn.backward(a["dY"], a["x"], a["U_up"], a["V_up"], a["U_down"], a["V_down"], fe)["dx"]

    want = expected_dx(root)
    assert rel_fro(gpu["dx"], want) <= TOL
    # the check can tell a flushing root apart (CPU-side counterfactual)
    flushed = expected_dx(np.where(gpu["S"] < 2.0 ** -126, 0.0, root))
    assert rel_fro(flushed, want) > 0.5


# ---- the fused forward (ELAS_FWD_FUSED) ---------------------------------------
# Shapes: ragged token counts (a partial block of 32), d_ff not a multiple of
# 64 (zero padding) or of 128 (a half chunk), both r (128, 256), d up to 1024,
# and more than 16384 tokens (two token blocks per workgroup).  The backward
# runs on the fused forward's saved P, S and Z, so their layouts are checked
# end to end.  (T = 16417 is the case where P differs from the oracle's by one
# bf16 ulp in one element, which moves one h onto an exact tie: a selection
# difference the accumulation bound of the mask gate explains.)
FUSED_SHAPES = [(5, 64, 64, 128), (100, 128, 200, 128), (300, 512, 1376, 128), (129, 768, 2048, 256),
                (700, 1024, 2736, 256), (20000, 64, 192, 128), (16449, 128, 320, 256), (16417, 128, 320, 256)]


@pytest.mark.parametrize("T,d,F,r", FUSED_SHAPES)
def test_fused_forward_parity(T, d, F, r):
    bits = ffn_inputs(T, d, F, r, seed_base=T + 7 * d)
    f, b = offn.run(bits)
    compare(run_gpu(bits, fwd_flags=elas.ELAS_FWD_FUSED), f, b, bits)


@pytest.mark.parametrize("cfg", ["llama60m", "llama130m", "llama350m"])
def test_fused_forward_model_shapes(cfg):
    bits = config_inputs(cfg, T=None if cfg == "llama60m" else 2048)
    f, b = offn.run(bits)
    compare(run_gpu(bits, fwd_flags=elas.ELAS_FWD_FUSED), f, b, bits)


@pytest.mark.parametrize("T", [700, 17000])
def test_fused_forward_exact(T):
    """Small integers for which every sum of the block is exact in binary32:
    every output of the fused forward and of the backward on its saved
    tensors equals the oracle's bit for bit."""
    d, F, r = 64, 1000, 128
    bits = sparse_sign_inputs(T, d, F, r, [1 / 8, 1 / 4, 1 / 4, 1 / 4, 1 / 4, 1 / 16], [0, 0, 0, -8, -4, 0], 61)
    f, b = offn.run(bits)
    assert all_sums_exact(bits, f, b)
    gpu = run_gpu(bits, fwd_flags=elas.ELAS_FWD_FUSED)
    assert_bit_exact(gpu, f, b, F)
    compare(gpu, f, b, bits)


@pytest.mark.parametrize("T,d,F,r", [(300, 512, 1376, 128), (129, 768, 2000, 256)])
def test_fused_forward_factors_ab_identical(T, d, F, r):
    """The fused forward reads pre-arranged factors (unpadded d_ff, read as
    zero beyond its end) exactly like the copies it makes otherwise."""
    bits = ffn_inputs(T, d, F, r, seed_base=11)
    t = {k: dev_bf16(v) for k, v in bits.items()}
    fused = elas.ELAS_FWD_FUSED
    ref = elas.elas_lowrank_ffn_fwd(t["x"], t["U_up"], t["V_up"], t["U_down"], t["V_down"], flags=fused)
    tr = {k: t[k].t().contiguous() for k in ("U_up", "V_up", "U_down", "V_down")}
    got = elas.elas_lowrank_ffn_fwd(t["x"], tr["U_up"], tr["V_up"], tr["U_down"], tr["V_down"],
                                    flags=fused | elas.ELAS_FACTORS_AB)
    torch.cuda.synchronize()
    for k in ("y", "P", "s_vals", "s_meta", "Z"):
        assert torch.equal(ref[k].view(torch.int16) if ref[k].dtype == torch.bfloat16 else ref[k],
                           got[k].view(torch.int16) if got[k].dtype == torch.bfloat16 else got[k]), k


def test_fused_forward_deterministic():
    """Two calls agree bit for bit (no atomics, fixed summation order)."""
    T, d, F, r = 77, 128, 320, 128
    bits = ffn_inputs(T, d, F, r, seed_base=5)
    a = run_gpu(bits, fwd_flags=elas.ELAS_FWD_FUSED)
    c = run_gpu(bits, fwd_flags=elas.ELAS_FWD_FUSED)
    for k in ("Y", "dx", "s_vals", "s_meta") + GRADS:
        np.testing.assert_array_equal(a[k], c[k], err_msg=k)

