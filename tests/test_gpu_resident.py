"""The token-resident products at the edges of their blocks: token counts
around 128, 2048 and 4096 (where the products to the model width change kernel), d
and d_ff that are not multiples of 64, each rank, each activation mode, against
the oracle with the gates of the other parity tests."""
import ctypes

import pytest
import torch

import paper_2605_03667_amd as elas
from oracle import ffn as offn
from synthetic import ffn_inputs
from tests.helpers import dev_bf16
from tests.test_gpu_ffn import compare, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["sparse", "dense"])
@pytest.mark.parametrize("T,d,F,r", [(1, 64, 64, 128), (127, 72, 72, 256), (129, 200, 1000, 512), (2049, 136, 328, 128),
                                     (2303, 72, 200, 256), (2431, 520, 456, 512), (4097, 136, 328, 128),
                                     (4351, 72, 200, 256), (4479, 520, 456, 512)])
def test_resident_edges(T, d, F, r, mode):
    bits = ffn_inputs(T, d, F, r, seed_base=T + r)
    f, b = offn.run(bits, sparse=(mode != "dense"))
    compare(run_gpu(bits, mode=mode), f, b, bits, mode=mode)


@pytest.mark.parametrize("T,d,F,r", [(2049, 136, 328, 128), (2431, 520, 456, 512), (4099, 72, 25000, 128),
                                     (4223, 200, 4104, 256), (4479, 520, 456, 512)])
def test_resident_factors_ab_identical(T, d, F, r):
    """Factors given as A and B are laid out by another job of the same launch."""
    t = {k: dev_bf16(v) for k, v in ffn_inputs(T, d, F, r, seed_base=5).items()}
    w = [t[k] for k in ("U_up", "V_up", "U_down", "V_down")]
    a = elas.elas_lowrank_ffn_fwd(t["x"], *w)
    b = elas.elas_lowrank_ffn_fwd(t["x"], *[x.t().contiguous() for x in w], flags=elas.ELAS_FACTORS_AB)
    for k in a:
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("mode", [0, elas.ELAS_MODE_DENSE])
def test_noalloc_at_the_scratch_limit(mode):
    """The weights in fragment order exceed the static scratch (64 MiB): the
    forward takes the kernels that need less, whose sums over r run in the same
    order.  (The long sums of Z are the same kernel's either way.)"""
    T, d, F, r, flags = 2049, 64, 65536, 512, elas.ELAS_FACTORS_AB | mode
    assert elas.elas_lowrank_ffn_fwd_workspace_bytes(T, d, F, r, flags) > elas.elas_noalloc_scratch_bytes()
    t = {k: dev_bf16(v) for k, v in ffn_inputs(T, d, F, r, seed_base=9).items()}
    w = [t[k].t().contiguous() for k in ("U_up", "V_up", "U_down", "V_down")]
    a = elas.elas_lowrank_ffn_fwd(t["x"], *w, flags=flags)
    out = {k: None if v is None else torch.full_like(v, 7) for k, v in a.items()}
    b = elas.elas_lowrank_ffn_fwd_noalloc(t["x"], *w, flags=flags, out=out)
    for k in a:
        assert a[k] is None or torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("T,d,F,r,mode,copies", [
    (4096, 768, 2048, 256, 0, 0), (8192, 512, 1376, 128, 0, 0), (12000, 512, 1376, 128, 0, 1), (6000, 768, 2048, 256, 0, 1),
    (2049, 2048, 5464, 512, 0, 1), (8192, 512, 1376, 128, elas.ELAS_MODE_DENSE, 0),
    (4096, 2048, 5464, 512, elas.ELAS_MODE_DENSE, 0), (6000, 2048, 5464, 512, elas.ELAS_MODE_DENSE, 1)])
def test_layout_launch_only_where_it_pays(T, d, F, r, mode, copies):
    """With factors as a linear layer stores them, a launch that lays weights out
    is a cost of the token-resident kernel alone: there is none where the tiled
    kernel is the faster of the two with it."""
    bf = dict(dtype=torch.bfloat16, device="cuda:0")
    w = [torch.zeros(s, **bf) for s in ((r, d), (F, r), (r, F), (d, r))]
    elas.elas_timing_enable(True)
    try:
        elas.elas_lowrank_ffn_fwd(torch.zeros((T, d), **bf), *w, flags=elas.ELAS_FACTORS_AB | mode)
        torch.cuda.synchronize()
        launches = elas.elas_timing_collect()
    finally:
        elas.elas_timing_enable(False)
    assert launches.get("weight_transpose", (0, 0.0))[0] == copies


@pytest.mark.parametrize("mode", [0, elas.ELAS_MODE_DENSE])
def test_factors_ab_need_no_workspace(mode):
    """Factors as a linear layer stores them are the tiled kernels' operands: a
    call without a workspace runs those, with the same results; and a workspace
    short of what even they need is refused."""
    T, d, F, r, flags = 4479, 520, 5464, 512, elas.ELAS_FACTORS_AB | mode
    need = elas.elas_lowrank_ffn_fwd_workspace_bytes(T, d, F, r, flags)
    assert need > 0
    t = {k: dev_bf16(v) for k, v in ffn_inputs(T, d, F, r, seed_base=8).items()}
    w = [t[k].t().contiguous() for k in ("U_up", "V_up", "U_down", "V_down")]
    a = elas.elas_lowrank_ffn_fwd(t["x"], *w, flags=flags)
    b = {k: None if v is None else torch.full_like(v, 7) for k, v in a.items()}

    def ptr(v):
        return ctypes.c_void_p(None if v is None else v.data_ptr())

    args = [ptr(v) for v in (t["x"], *w)]
    out = [ptr(b[k]) for k in ("y", "P", "s_vals", "s_meta", "Z")]
    torch.cuda.synchronize()
    assert elas.lib().elas_lowrank_ffn_fwd(*args, T, d, F, r, flags, *out, None, 0, None) == 0
    torch.cuda.synchronize()
    for k in a:
        assert a[k] is None or torch.equal(a[k], b[k]), k
    flags = mode   # the other orientation always needs its copies
    need = elas.elas_lowrank_ffn_fwd_workspace_bytes(T, d, F, r, flags)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    assert elas.lib().elas_lowrank_ffn_fwd(*args, T, d, F, r, flags, *out, ptr(ws), d * r * 2, None) == 4
