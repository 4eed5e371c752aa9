"""Infinities and NaN of one token stay with that token: with non-finite values in
two rows of x and dY (the last row, which kernels re-read in place of rows past the
end, and one in the middle), P, Z, S, y and dx of every other token are the same
bits as without them, whichever kernel the token count and rank select."""
import pytest
import torch

import paper_2605_03667_amd as elas
from synthetic import ffn_inputs
from tests.helpers import dev_bf16, untile

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["sparse", "dense", "ste"])
@pytest.mark.parametrize("T,d,F,r", [(17, 520, 1000, 512), (250, 264, 200, 72), (1100, 136, 328, 128), (2300, 520, 456, 512),
                                     (4351, 72, 200, 256)])
def test_nonfinite_tokens_stay_alone(T, d, F, r, mode):
    t = {k: dev_bf16(v) for k, v in ffn_inputs(T, d, F, r, seed_base=T).items()}
    w = [t[k] for k in ("U_up", "V_up", "U_down", "V_down")]
    fflags = elas.ELAS_MODE_DENSE if mode == "dense" else 0
    bflags = elas.ELAS_BWD_STE if mode == "ste" else fflags

    def run():
        o = elas.elas_lowrank_ffn_fwd(t["x"], *w, flags=fflags)
        g = elas.elas_lowrank_ffn_bwd(t["dY"], t["x"], *w, o, flags=bflags)
        rows = {"P": o["P"], "Z": o["Z"], "y": o["y"], "dx": g["dx"]}
        if mode == "dense":
            rows["S"] = o["s_vals"]
        else:
            rows["S"] = untile(o["s_vals"], T, o["s_vals"].shape[1], 32)
            rows["codes"] = untile(o["s_meta"], T, o["s_meta"].shape[1], 8)
        return {k: v.clone() for k, v in rows.items()}

    clean = run()
    bad = [T // 2, T - 1]
    t["x"][bad[0], 3], t["x"][bad[0], 5], t["x"][bad[1], 0] = float("inf"), float("-inf"), float("nan")
    t["dY"][bad[0], 1], t["dY"][bad[1], 2] = float("nan"), float("inf")
    got = run()
    others = torch.ones(T, dtype=torch.bool, device="cuda:0")
    others[bad] = False
    for k, v in clean.items():
        assert torch.equal(got[k][others], v[others]), k
    assert not torch.isfinite(got["P"][bad].float()).all(dim=1).any()
    assert not torch.isfinite(got["dx"][bad].float()).all(dim=1).any()
