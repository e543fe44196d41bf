"""GPU parity on both sides of the rules that pick a kernel variant by size: the whole problem runs on the GPU in the
variant that its size selects, the fp64 oracle is evaluated on two (batch, head) slices of it (the first and the last).
The tolerance is the suite's own per-tensor bar (gpu_util.TOL): the variants round the same operands at the same places."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import mlstm_oracle as orc

pytestmark = pytest.mark.gpu


def _scan_noise(oi, rb, w):
    """What the rounding of bf16 operands may leave in the forget gate's gradient, per step: a reversed sum of q dq - k dk over
    the steps up to the end of a block of four chunks (two for heads wider than 512), where an exact anchor takes over.  Each
    product carries the independent roundings of a weight, a state and a result, sqrt(3) 2^-9 together; four standard
    deviations of their sum, times sigma(-f~)."""
    G = 2 if max(w.dqk, w.dhv) > 512 else 4
    var = ((oi["q"] * rb["dq"]) ** 2).sum(-1) + ((oi["k"] * rb["dk"]) ** 2).sum(-1)
    out = np.zeros_like(var)
    for t0 in range(0, w.T, G * w.chunk):
        out[:, t0:t0 + G * w.chunk] = np.cumsum(var[:, t0:t0 + G * w.chunk][:, ::-1], axis=1)[:, ::-1]
    return 4 * 3 ** 0.5 * 2.0 ** -9 * np.sqrt(out) / (1.0 + np.exp(oi["f_pre"]))


def _check_slices(w, dCn=False, keep=True, scan=False):
    import paper_2503_14376_amd as tfla
    from tests import gpu_util as gu
    d = wl.make_inputs(w)
    dev = gu.dev_inputs(w, d)
    print("rule", w.variant, w.dtype, (w.B, w.NH, w.T, w.dqk, w.dhv, w.chunk), flush=True)
    st = [dev.get(x) for x in ("C0", "n0", "m0")]
    dC = torch.randn((w.B, w.NH, w.dqk, w.dhv), device="cuda", generator=torch.Generator("cuda").manual_seed(5)) if dCn else None
    f = tfla.mlstm_fwd(dev["q"], dev["k"], dev["v"], dev["i_pre"], dev["f_pre"], *st, chunk=w.chunk, variant=w.variant, eps=1e-6)
    b = tfla.mlstm_bwd(dev["q"], dev["k"], dev["v"], dev["i_pre"], dev["f_pre"], dev["dH"], f["n_out"], f["m_out"], *st, dC,
                       chunk=w.chunk, variant=w.variant, eps=1e-6, fwd_workspace=f["workspace"] if keep else None)
    torch.cuda.synchronize()
    idx = sorted({0, w.B * w.NH - 1})
    sub = lambda t: t.reshape((-1,) + tuple(t.shape[2:]))[idx]
    oi = gu.oracle_inputs(wl.make_inputs(w, slices=idx))
    tol = gu.TOL[w.dtype]
    ref = orc.recurrent_fwd(**oi, variant=w.variant, eps=1e-6)
    rb = orc.chunkwise_bwd(**oi, dH=gu.flat(wl.make_inputs(w, slices=idx)["dH"]), variant=w.variant, eps=1e-6, chunk=128,
                           **({"dCn": sub(dC).double().cpu().numpy()} if dCn else {}))
    errs = {k: gu.rel_err(sub(f[k]), ref[k]) for k in ("H", "Cn") + (("nn", "n_out") if w.variant == wl.EXP else ())}
    names = dict(dq="dq", dk="dk", dv="dv", d_i_pre="di", d_f_pre="df")
    if w.init_state:
        names["dC0"] = "dC0"
    errs.update({k: gu.rel_err(sub(b[k]), rb[r]) for k, r in names.items()})
    print("   ", errs, flush=True)
    if scan and w.dtype == wl.BF16:
        # (an upstream state gradient of the size of the states themselves makes the sum cancel to where its noise shows)
        off = np.abs(sub(b["d_f_pre"]).double().cpu().numpy() - rb["df"])
        bound = np.maximum(_scan_noise(oi, rb, w), tol * np.abs(rb["df"]).max())
        print("    scan: error over bound", float((off / bound).max()), flush=True)
        assert np.all(off <= bound), float((off / bound).max())
        del errs["d_f_pre"]
    for k, e in errs.items():
        assert e <= tol, (k, e, errs)


# contractions over 1024 columns.  The weighted matrix lies where a split contraction would leave its partial results, if it fits:
# for H up to chunk 448 at d_hv = 256 and 960 at 512; several blocks per chunk on and off the diagonal, of 64 and of 128 rows,
# whole and ragged
@pytest.mark.parametrize("keep", [True, False])
@pytest.mark.parametrize("variant,B,NH,T,dqk,dhv,chunk", [
    (wl.EXP, 1, 2, 900, 1024, 256, 448),
    (wl.EXP, 1, 2, 1024, 1024, 256, 512),       # does not fit
    (wl.EXP, 1, 1, 2000, 1000, 512, 960),
    (wl.SIG, 1, 1, 2048, 1024, 504, 1024),      # does not fit
    (wl.EXP, 2, 1, 640, 520, 1000, 320),
    (wl.SIG, 1, 3, 1152, 264, 1024, 384),
])
def test_wide_contractions(keep, variant, B, NH, T, dqk, dhv, chunk):
    w = wl.small(variant, wl.BF16, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=1500 + T + dqk)
    _check_slices(w, dCn=True, keep=keep, scan=True)


# heads wider than 512 with chunks above 1024: a block of the forget-gate gradient scan is two chunks, up to 4096 steps
@pytest.mark.parametrize("variant,B,NH,T,dqk,dhv,chunk", [
    (wl.EXP, 1, 2, 3 * 1088, 64, 1024, 1088),   # blocks of 2176 steps, the last one half full
    (wl.SIG, 1, 1, 4000, 1000, 256, 1536),
    (wl.EXP, 1, 1, 2 * 2048, 520, 64, 2048),    # one block of 4096
    (wl.EXP, 1, 1, 2 * 2048 + 100, 128, 1024, 2048),
    (wl.EXP, 1, 1, 2 * 1088, 1024, 1024, 1088),
])
def test_wide_heads_long_chunks(variant, B, NH, T, dqk, dhv, chunk):
    w = wl.small(variant, wl.BF16, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=2500 + T + dqk)
    _check_slices(w, dCn=True, keep=T % 64 == 0, scan=True)


# 128 x 256 state tiles of the recurrent kernel: from 129 of them on, but not from 257 to 320; one piece and several per chunk,
# fewer pieces than ring stages, anchors, whole and ragged
@pytest.mark.parametrize("variant,B,NH,T,dqk,dhv,chunk,state", [
    (wl.EXP, 3, 43, 320, 128, 256, 64, True),        # 129
    (wl.EXP, 8, 16, 320, 128, 256, 64, True),        # 128: the smaller tiles
    (wl.SIG, 13, 20, 128, 128, 256, 128, False),     # 260: the smaller tiles
    (wl.EXP, 8, 41, 192, 128, 256, 192, False),      # 328
    (wl.EXP, 19, 7, 64, 128, 256, 64, True),         # one piece
    (wl.EXP, 19, 7, 100, 120, 248, 128, True),
    (wl.EXP, 4, 8, 700, 456, 504, 128, True),
    (wl.SIG, 4, 8, 1100, 512, 512, 256, True),
    (wl.EXP, 2, 3, 900, 1000, 1024, 128, True),      # 32 workgroups per head: with the L2 prefetch where whole
    (wl.EXP, 2, 3, 1152, 1024, 1024, 128, True),
    (wl.SIG, 2, 3, 1152, 1024, 1024, 192, False),
])
def test_large_state_tiles(variant, B, NH, T, dqk, dhv, chunk, state):
    w = wl.small(variant, wl.BF16, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=1700 + T + dqk, init_state=state)
    _check_slices(w, dCn=state, keep=T % 128 == 0, scan=True)


# every (batch, head) of a problem, not two of them: the slices hold two slices' inputs in turn, and each one's results are,
# bit for bit, those of the first two, which the oracle has checked in the tests around
@pytest.mark.parametrize("variant,B,NH,T,dqk,dhv,chunk", [
    (wl.EXP, 3, 43, 320, 128, 256, 64),         # large state tiles
    (wl.SIG, 19, 7, 100, 120, 248, 128),
    (wl.EXP, 2, 3, 900, 1000, 1024, 128),
    (wl.EXP, 3, 3, 1024, 1024, 1024, 256),      # 256 rows per workgroup
    (wl.SIG, 2, 5, 1100, 1000, 1024, 512),
    (wl.EXP, 1, 5, 900, 1024, 256, 448),        # 64 rows
    (wl.EXP, 5, 13, 700, 64, 64, 64),           # few state tiles
    (wl.EXP, 9, 37, 320, 64, 64, 64),           # ... and more than CUs
    (wl.EXP, 3, 5, 256 * 17 - 3, 64, 128, 256), # gate kernels of more than sixteen chunks
])
def test_every_slice(variant, B, NH, T, dqk, dhv, chunk):
    import paper_2503_14376_amd as tfla
    from tests import gpu_util as gu
    w = wl.small(variant, wl.BF16, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=2900 + T + dqk)
    dev = gu.dev_inputs(w, wl.make_inputs(wl.small(variant, wl.BF16, B=1, NH=2, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=w.seed)))
    which = torch.arange(B * NH, device="cuda") % 2
    dev = {k: x.reshape((2,) + x.shape[2:])[which].reshape((B, NH) + x.shape[2:]).contiguous() for k, x in dev.items()}
    args, kw = [dev[x] for x in ("q", "k", "v", "i_pre", "f_pre")], dict(chunk=chunk, variant=variant, eps=1e-6)
    st = [dev.get(x) for x in ("C0", "n0", "m0")]
    f = tfla.mlstm_fwd(*args, *st, **kw)
    b = tfla.mlstm_bwd(*args, dev["dH"], f["n_out"], f["m_out"], *st, **kw, fwd_workspace=f["workspace"])
    torch.cuda.synchronize()
    for o in (f, b):
        for k, x in o.items():
            if k == "workspace":
                continue
            x = x.reshape((B * NH,) + x.shape[2:])
            assert torch.isfinite(x.float()).all(), k
            assert torch.equal(x, x[:2][which]), k


# Few state tiles: the reversed launch's anchors arrive through a ring of LDS buffers.  The first one belongs to piece 1, 2, 3, 4, ...
# (the chunks past the last whole block), the next to one four or (heads wider than 512) two chunks on, and there may be none
@pytest.mark.parametrize("B,NH,T,dqk,dhv,chunk", [
    (1, 2, 64 * n, 64, 64, 64) for n in (2, 4, 5, 6, 7, 8, 9)] + [(1, 2, 128 * n, 64, 128, 128) for n in (4, 5, 6, 7)] + [
    (1, 1, 64 * n, 64, 1024, 64) for n in (2, 3, 4, 9)] + [(1, 1, 128 * n, 64, 1024, 128) for n in (3, 8)] + [
    (1, 1, 256 * 5, 1024, 64, 256), (1, 3, 700, 64, 128, 64), (1, 3, 900, 120, 64, 128),
])
def test_anchors_through_lds(B, NH, T, dqk, dhv, chunk):
    w = wl.small(wl.EXP, wl.BF16, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=1900 + T + dqk)
    _check_slices(w, keep=T % 256 == 0, scan=True)


# Gate kernels of more than sixteen chunks: chunks of 64, 128, 256 and 512 move a lane's steps as vectors, others do not; several
# chunks per lane of the recurrence over the chunks (more than 64), a last block of the gradient scan with fewer chunks, ragged ends
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("variant,T,chunk", [
    (wl.EXP, 64 * 19, 64), (wl.SIG, 64 * 67 - 3, 64), (wl.EXP, 64 * 131 - 1, 64), (wl.EXP, 128 * 17 - 100, 128), (wl.SIG, 256 * 18, 256),
    (wl.EXP, 256 * 17 - 255, 256), (wl.EXP, 512 * 17 - 77, 512), (wl.EXP, 192 * 18 - 5, 192), (wl.SIG, 320 * 17, 320),
])
def test_gates_of_many_chunks(dtype, variant, T, chunk):
    w = wl.small(variant, dtype, B=1, NH=2, T=T, dqk=64, dhv=64, chunk=chunk, seed=2100 + T)
    _check_slices(w, keep=T % 2 == 0, scan=True)


# m_out and n_out are any float pointers: outputs that lie one float into a buffer are those of a call with aligned ones
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("T,chunk", [(64 * 17, 64), (128 * 17, 128), (256 * 17, 256), (512 * 17, 512), (256 * 3, 256)])
def test_unaligned_per_step_outputs(dtype, T, chunk):
    import paper_2503_14376_amd as tfla
    from tests import gpu_util as gu
    w = wl.small(wl.EXP, dtype, B=1, NH=2, T=T, dqk=64, dhv=64, chunk=chunk, seed=2700 + T)
    dev = gu.dev_inputs(w, wl.make_inputs(w))
    args = [dev[x] for x in ("q", "k", "v", "i_pre", "f_pre", "C0", "n0", "m0")]
    kw = dict(chunk=w.chunk, variant=w.variant, eps=1e-6)
    ref = tfla.mlstm_fwd(*args, **kw)
    out = {k: torch.empty_like(ref[k]) for k in ("H", "Cn", "nn", "mn")}
    for k in ("n_out", "m_out"):
        out[k] = torch.empty(ref[k].numel() + 1, device="cuda")[1:].view(ref[k].shape)
        assert out[k].data_ptr() % 8 == 4
    res = tfla.mlstm_fwd(*args, **kw, out=out)
    a, b = (tfla.mlstm_bwd(*args[:5], dev["dH"], f["n_out"], f["m_out"], *args[5:], **kw, fwd_workspace=f["workspace"]) for f in (ref, res))
    torch.cuda.synchronize()
    for k in ("H", "Cn", "nn", "mn", "n_out", "m_out"):
        assert torch.equal(ref[k], res[k]), k
    for k in ("dq", "dk", "dv", "d_i_pre", "d_f_pre"):
        assert torch.equal(a[k], b[k]), k


# 256 rows per workgroup for contractions over 1024 columns: chunks of 256 and multiples, more than 128 workgroups, whole and ragged
@pytest.mark.parametrize("variant,B,NH,T,dqk,dhv,chunk", [
    (wl.EXP, 3, 3, 1024, 1024, 1024, 256),      # 144 workgroups
    (wl.SIG, 2, 2, 2300, 1000, 1016, 256),      # 160 with the last chunk ragged
    (wl.EXP, 2, 5, 1536, 1024, 768, 768),       # (three row blocks per chunk)
    (wl.EXP, 1, 17, 1024, 1024, 512, 512),      # H and dV only, 136
    (wl.EXP, 1, 17, 1000, 512, 1024, 512),      # dQ and dK only
    (wl.EXP, 1, 24, 1000, 1024, 1024, 256),     # 384 workgroups: the last with 128 rows
    (wl.SIG, 1, 33, 1000, 1024, 1024, 256),     # 528
])
def test_wide_contractions_256_rows(variant, B, NH, T, dqk, dhv, chunk):
    w = wl.small(variant, wl.BF16, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=2300 + T + dqk)
    _check_slices(w, dCn=True, keep=T % 512 != 0, scan=True)


# 256-wide output blocks of the tiled kernels: rows / 128 * (columns / 256) >= 256 workgroups, chunk a multiple of 128
@pytest.mark.parametrize("variant,B,NH,T,dqk,dhv,chunk", [
    (wl.EXP, 1, 4, 2048, 1024, 1024, 256),      # exactly 256 workgroups in every mode (weights from memory)
    (wl.SIG, 1, 4, 1920, 1024, 1024, 128),      # 240: below the line
    (wl.EXP, 1, 8, 2048, 512, 512, 256),        # exactly 256, one launch per mode
    (wl.EXP, 3, 5, 2304, 512, 512, 384),        # an odd number of heads, three row blocks per chunk
    (wl.SIG, 1, 16, 2048, 512, 256, 128),       # dQ / dK contract over 256 columns, H / dV over 512
])
def test_wide_output_blocks(variant, B, NH, T, dqk, dhv, chunk):
    w = wl.small(variant, wl.BF16, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=700 + T + dqk)
    _check_slices(w)


# dV, dQ and dK in one launch: all kernel widths up to 256 on either side, two- and four-wavefront workgroups, several row
# blocks, a number of heads that is no multiple of the XCDs, tensors that end inside a block; and the first shape past the rule
@pytest.mark.parametrize("variant,NH,T,dqk,dhv,chunk", [
    (wl.EXP, 3, 512, 64, 64, 256), (wl.SIG, 8, 192, 64, 128, 64), (wl.EXP, 2, 300, 64, 256, 128),
    (wl.SIG, 5, 384, 128, 64, 384), (wl.EXP, 8, 130, 120, 128, 64), (wl.EXP, 1, 1000, 128, 200, 512),
    (wl.EXP, 3, 256, 256, 64, 64), (wl.SIG, 2, 449, 256, 128, 128), (wl.EXP, 8, 512, 256, 256, 256),
    (wl.EXP, 3, 256, 256, 264, 128),
])
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
def test_gradients_in_one_launch(dtype, variant, NH, T, dqk, dhv, chunk):
    w = wl.small(variant, dtype, B=1, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=600 + T + dqk)
    _check_slices(w, dCn=True)


# dK written over an input that dV and dQ read takes three launches and gives the same bits (what the header allows: over K in
# bf16; over V where a workgroup reads its own rows only; over Q and dH where a chunk is one row block)
@pytest.mark.parametrize("dtype,T,dqk,dhv,chunk,name", [
    (wl.BF16, 1024, 64, 64, 128, "k"), (wl.BF16, 1024, 256, 128, 128, "k"),
    (wl.BF16, 1024, 64, 64, 256, "v"), (wl.BF16, 1024, 128, 128, 256, "v"), (wl.BF16, 1000, 96, 96, 128, "v"), (wl.F32, 1024, 64, 64, 128, "v"),
    (wl.BF16, 1024, 128, 128, 128, "q"), (wl.BF16, 1000, 64, 256, 64, "q"), (wl.F32, 1024, 64, 64, 64, "q"),
    (wl.BF16, 1024, 64, 64, 64, "dH"), (wl.BF16, 1024, 128, 128, 128, "dH"), (wl.F32, 1000, 64, 64, 128, "dH"),
])
def test_key_gradient_in_place(dtype, T, dqk, dhv, chunk, name):
    import paper_2503_14376_amd as tfla
    from tests import gpu_util as gu
    w = wl.small(wl.EXP, dtype, B=4, NH=16, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=630 + dqk)
    print("dK over", name, (dtype, T, dqk, dhv, chunk), flush=True)
    dev = gu.dev_inputs(w, wl.make_inputs(w))
    x = [dev[n] for n in ("q", "k", "v", "i_pre", "f_pre")]
    f = tfla.mlstm_fwd(*x, chunk=chunk, variant=w.variant, eps=1e-6)
    call = lambda out: tfla.mlstm_bwd(*x, dev["dH"], f["n_out"], f["m_out"], chunk=chunk, variant=w.variant, eps=1e-6,
                                      fwd_workspace=f["workspace"], out=out)
    apart = call(None)
    over = call(dict({n: torch.empty_like(apart[n]) for n in ("dq", "dv", "d_i_pre", "d_f_pre", "dC0")}, dk=dev[name]))
    torch.cuda.synchronize()
    assert over["dk"].data_ptr() == dev[name].data_ptr()
    for n in ("dq", "dk", "dv", "d_i_pre", "d_f_pre", "dC0"):
        assert torch.equal(apart[n], over[n]), n


# fp32: 128-wide blocks in the one launch (512 workgroups of two wavefronts and more), and both sides of the rules that keep
# three launches
@pytest.mark.parametrize("variant,B,NH,T,dqk,dhv,chunk", [
    (wl.SIG, 2, 8, 1024, 128, 256, 64),         # one launch, 128-wide blocks
    (wl.EXP, 2, 8, 512, 128, 256, 64),          # exactly 512 workgroups
    (wl.EXP, 1, 15, 512, 128, 256, 64),         # 480
    (wl.EXP, 2, 8, 500, 256, 104, 128),
    (wl.SIG, 2, 16, 1024, 128, 256, 64),        # 32768 rows: three launches
    (wl.EXP, 4, 16, 1024, 256, 64, 256),        # 65536 rows
    (wl.EXP, 4, 16, 1024, 128, 128, 64),        # 65536 rows of narrow heads: one launch
])
def test_gradients_in_one_launch_fp32_rules(variant, B, NH, T, dqk, dhv, chunk):
    w = wl.small(variant, wl.F32, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=650 + T + dqk)
    _check_slices(w, dCn=True)


# fp32 forget-gate scan: the blocks of 1024 steps after a block summed by itself (up to four blocks) or by a launch before it
@pytest.mark.parametrize("variant,T", [(wl.EXP, 1024), (wl.SIG, 1100), (wl.EXP, 4096), (wl.SIG, 4097)])
def test_fp32_gate_gradient_blocks(variant, T):
    _check_slices(wl.small(variant, wl.F32, B=1, NH=2, T=T, dqk=64, dhv=64, chunk=64, seed=640 + T), dCn=True)


# fp32 recurrent kernels: 256 state tiles of 64 x 64 and fewer (split pieces), more of them, and 128 x 128 ones; two and more
# pieces per chunk, one chunk, numbers of pieces that are no multiple of four, tensors that end inside a tile and a piece
@pytest.mark.parametrize("keep", [True, False])
@pytest.mark.parametrize("variant,B,NH,T,dqk,dhv,chunk", [
    (wl.EXP, 1, 1, 64, 64, 64, 64), (wl.SIG, 1, 3, 300, 72, 40, 192), (wl.EXP, 1, 16, 256, 256, 256, 128),
    (wl.EXP, 1, 17, 200, 256, 256, 64), (wl.SIG, 1, 64, 128, 128, 128, 64), (wl.EXP, 2, 24, 130, 256, 256, 64),
])
def test_fp32_state_tiles(keep, variant, B, NH, T, dqk, dhv, chunk):
    w = wl.small(variant, wl.F32, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=660 + T + dqk, init_state=True)
    _check_slices(w, dCn=True, keep=keep)


# recurrent kernels that bring the lines of later pieces into L2.  On: 64 x 64 state tiles, 16 and 32 sharers, pieces of 64 and
# 128 rows, one and more per chunk (from 24 on), and 64 x 128 ones, d_hv from 512 on, pieces of 128 rows (from 16 on).  Off: a piece
# too few, pieces of 64 rows or d_hv = 256 with 64 x 128 tiles, 128 sharers, sequences and head dimensions that end inside a piece
@pytest.mark.parametrize("variant,B,NH,T,dqk,dhv,chunk", [
    (wl.SIG, 1, 8, 3072, 256, 512, 128), (wl.EXP, 1, 8, 3072, 256, 512, 256), (wl.EXP, 1, 8, 1536, 256, 512, 64),
    (wl.SIG, 1, 8, 1728, 256, 512, 192), (wl.EXP, 1, 5, 1600, 256, 256, 64), (wl.EXP, 1, 3, 3200, 128, 512, 128),
    (wl.EXP, 3, 8, 2048, 256, 512, 128), (wl.SIG, 3, 8, 2304, 256, 512, 256), (wl.EXP, 1, 8, 2560, 512, 512, 512),
    (wl.EXP, 1, 8, 2944, 256, 512, 128), (wl.SIG, 3, 8, 1920, 256, 512, 128), (wl.EXP, 3, 8, 1152, 256, 512, 192),
    (wl.EXP, 2, 16, 2048, 512, 256, 128), (wl.SIG, 1, 4, 1024, 1024, 1024, 64),
    (wl.EXP, 1, 3, 1600, 256, 512, 192), (wl.EXP, 1, 4, 3500, 256, 320, 256), (wl.EXP, 3, 8, 1100, 200, 456, 192),
])
def test_recurrent_prefetch(variant, B, NH, T, dqk, dhv, chunk):
    w = wl.small(variant, wl.BF16, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=680 + T + dqk)
    _check_slices(w)


# tensors that end before the kernels' blocks do: whole row blocks, pieces and column blocks past the end, odd remainders,
# initial state and upstream state gradient, both ways of the backward pass (kept and recomputed states)
@pytest.mark.parametrize("keep", [True, False])
@pytest.mark.parametrize("variant,dtype,T,dqk,dhv,chunk", [
    (wl.EXP, wl.BF16, 130, 256, 512, 512),      # two of four row blocks empty
    (wl.SIG, wl.BF16, 257, 40, 520, 256),       # one step in the last chunk; a contraction split behind 512 of 520 columns
    (wl.EXP, wl.BF16, 3, 64, 64, 2048),         # almost everything past the end
    (wl.EXP, wl.BF16, 700, 1000, 72, 192),      # two-wavefront workgroups, 64-row pieces
    (wl.EXP, wl.F32, 70, 72, 136, 192),
    (wl.SIG, wl.F32, 333, 264, 328, 64),        # fp32 contraction split behind 256 of 264 / 328 columns
])
def test_tensors_that_end_inside_a_block(keep, variant, dtype, T, dqk, dhv, chunk):
    w = wl.small(variant, dtype, B=1, NH=3, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=800 + T + dqk)
    _check_slices(w, dCn=True, keep=keep)


# the row kernels of the layer: one and two groups of 512 columns per wavefront, several rows side by side, row blocks that
# end early, one row only; forward through the layer's own entry point against the fp64 norm of the rounded cell output
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("B,NH,T,dhv", [(1, 1, 1, 512), (1, 2, 129, 264), (2, 1, 33, 1024), (1, 3, 77, 128), (8, 16, 1030, 256)])
def test_layer_rows(dtype, kind, B, NH, T, dhv):
    import paper_2503_14376_amd as tfla
    if dtype == wl.F32 and dhv > 512:
        dhv = 512
    g = torch.Generator(device="cuda").manual_seed(900 + T + dhv)
    td = torch.bfloat16 if dtype == wl.BF16 else torch.float32
    mk = lambda *s: torch.randn(s, device="cuda", generator=g)
    q, k, v, o, dY = mk(B, NH, T, 64).to(td), mk(B, NH, T, 64).to(td), *(mk(B, NH, T, dhv).to(td) for _ in range(3))
    o = o * 8                                   # gates from closed to open
    ip, fp, gamma, beta = mk(B, NH, T), mk(B, NH, T) + 3, 1 + 0.1 * mk(NH, dhv), 0.1 * mk(NH, dhv)
    print("rows", dtype, kind, (B, NH, T, dhv), flush=True)
    kw = dict(chunk=64, norm_kind=kind, norm_eps=1e-6)
    f = tfla.mlstm_layer_fwd(q, k, v, ip, fp, o, gamma, beta, **kw)
    b = tfla.mlstm_layer_bwd(q, k, v, ip, fp, f["H"], dY, o, gamma, beta, f["n_out"], f["m_out"], fwd_workspace=f["workspace"], **kw)
    torch.cuda.synchronize()
    h, od, gd, bd, dy = (t.double().cpu() for t in (f["H"], o, gamma, beta, dY))
    od.requires_grad_(); gd.requires_grad_(); bd.requires_grad_()
    x = h - h.mean(-1, keepdim=True) if kind == 1 else h
    y = torch.sigmoid(od) * (x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-6) * gd[None, :, None] + (bd[None, :, None] if kind else 0))
    (y * dy).sum().backward()
    # one rounding to the element type (2^-9, 2^-24) of the largest value, and for the sums over B T rows of products of
    # rounded operands the fp32 spacing times sqrt(rows); a factor of four on each
    tol = 4 * 2.0 ** -9 if dtype == wl.BF16 else 4e-6
    err = lambda a, r: float((a.double().cpu() - r).abs().max() / r.abs().max().clamp_min(1e-30))
    errs = {"Y": err(f["Y"], y.detach()), "do": err(b["do_pre"], od.grad), "dgamma": err(b["dgamma"], gd.grad)}
    if kind == 1:
        errs["dbeta"] = err(b["dbeta"], bd.grad)
    else:
        assert float(b["dbeta"].abs().max()) == 0.0
    print("   ", errs, flush=True)
    for key, e in errs.items():
        assert e <= (tol if key in ("Y", "do") else 4e-6 * max(1.0, (B * T) ** 0.5 / 8)), (key, errs)


# generation step: both slab widths (64 columns from 2^24 state values on), batches of 64, 128 and 256 rows and row counts
# that end inside a batch; one step against the fp64 recurrence on the first and the last head, fp32 bar on the state
@pytest.mark.parametrize("variant", [wl.EXP, wl.SIG])
@pytest.mark.parametrize("B,NH,dqk,dhv", [(1, 1, 64, 64), (16, 8, 256, 512), (2, 3, 192, 64), (64, 64, 64, 64), (3, 64, 320, 320),
                                          (16, 64, 128, 128), (1, 2, 576, 960), (17, 1, 1024, 1024)])
def test_step_slabs(variant, B, NH, dqk, dhv):
    import paper_2503_14376_amd as tfla
    g = torch.Generator(device="cuda").manual_seed(950 + dqk + dhv)
    mk = lambda *s: torch.randn(s, device="cuda", generator=g)
    q, k, v = mk(B, NH, dqk), mk(B, NH, dqk), mk(B, NH, dhv)
    ip, fp, C, n, m = mk(B, NH), mk(B, NH) + 3, mk(B, NH, dqk, dhv), mk(B, NH, dqk), mk(B, NH)
    print("step slabs", variant, (B, NH, dqk, dhv), flush=True)
    o = tfla.mlstm_step(q, k, v, ip, fp, C, n, m, variant=variant, eps=1e-6)
    torch.cuda.synchronize()
    for b, h in ((0, 0), (B - 1, NH - 1)):
        s = lambda t: t[b, h].double().cpu().numpy()[None]
        r = orc.recurrent_fwd(s(q)[:, None], s(k)[:, None], s(v)[:, None], s(ip)[:, None], s(fp)[:, None], s(C), s(n), s(m),
                              variant=variant, eps=1e-6)
        from tests import gpu_util as gu
        for key, ref in (("h", r["H"][0, 0]), ("C", r["Cn"][0])) + ((("n", r["nn"][0]),) if variant == wl.EXP else ()):
            e = gu.rel_err(o[key][b, h], ref)
            assert e <= gu.TOL[wl.F32], (key, e)
    if variant == wl.SIG:
        assert float(o["n"].abs().max()) == 0.0 and float(o["m"].abs().max()) == 0.0


# the two recurrent kernels: 64 x 64 state tiles up to 256 of them, 64 x 128 beyond (where d_hv is a multiple of 128), with
# 64- and 128-row pieces, piece counts that are no multiple of the four a producer keeps on its way, whole and ragged
@pytest.mark.parametrize("variant,B,NH,T,dqk,dhv,chunk", [
    (wl.EXP, 2, 8, 320, 256, 256, 64),          # exactly 256 tiles of 64 x 64, five 64-row pieces
    (wl.SIG, 1, 17, 384, 256, 256, 128),        # 272: 64 x 128 tiles, three 128-row pieces
    (wl.EXP, 3, 7, 200, 256, 256, 64),          # 336, ragged
    (wl.SIG, 4, 8, 700, 248, 200, 256),         # 512, ragged in every direction, 128-row pieces
    (wl.EXP, 8, 40, 130, 64, 64, 64),           # 320 tiles, d_hv = 64: 64 x 64 whatever their number
    (wl.EXP, 1, 1, 64, 64, 64, 64),             # one piece
])
def test_recurrent_tiles(variant, B, NH, T, dqk, dhv, chunk):
    w = wl.small(variant, wl.BF16, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=1000 + T + dqk)
    _check_slices(w, dCn=True)


# the gate pre-pass in one launch (up to 16 chunks of 64, 128, 256 or 512) and in two
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("variant,T,chunk", [(wl.EXP, 1024, 64), (wl.EXP, 1025, 64), (wl.SIG, 2048, 128), (wl.EXP, 1000, 512),
                                             (wl.EXP, 576, 192)])
def test_gate_launches(dtype, variant, T, chunk):
    w = wl.small(variant, dtype, B=1, NH=3, T=T, dqk=64, dhv=64, chunk=chunk, seed=1100 + T)
    _check_slices(w)


# a state that is continued in place (the final state's buffers are the initial state's): up to 16 chunks the gate pre-pass
# is one workgroup per (batch, head), whose wavefronts all need the initial max state that one of them replaces; beyond, and at
# other chunk sizes, all workgroups of a second launch do
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("T,chunk", [(64, 64), (128, 64), (250, 64), (512, 128), (1024, 64), (1088, 64), (4000, 64), (1100, 192), (5000, 1024)])
def test_state_continued_in_place(dtype, T, chunk):
    import paper_2503_14376_amd as tfla
    from tests import gpu_util as gu
    w = wl.small(wl.EXP, dtype, B=2, NH=3, T=T, dqk=64, dhv=64, chunk=chunk, seed=1200 + T)
    dev = gu.dev_inputs(w, wl.make_inputs(w))
    args = [dev[x] for x in ("q", "k", "v", "i_pre", "f_pre")]
    st = [dev[x] for x in ("C0", "n0", "m0")]
    st[2] = st[2] + 40.0                        # an initial max state that decides the stabilisation of every chunk
    two = tfla.mlstm_fwd(*args, *st, chunk=chunk, eps=1e-6)
    cur = [t.clone() for t in st]
    one = tfla.mlstm_fwd(*args, *cur, chunk=chunk, eps=1e-6, out=dict(zip(("Cn", "nn", "mn"), cur)))
    torch.cuda.synchronize()
    for key in ("H", "Cn", "nn", "mn", "n_out", "m_out"):
        assert torch.equal(one[key], two[key]), key


# steps past the end of a ragged sequence have no q: with eps = 0 and a max state above 104, where exp(-m) is zero in fp32,
# their denominator is no number, and what the H kernel leaves for them must not reach the gradients.  The backward pass from
# the forward call's workspace against the one that recomputes everything (same operands; the suite's bar)
@pytest.mark.parametrize("dtype,dqk,dhv,chunk", [(wl.BF16, 64, 64, 64), (wl.BF16, 256, 512, 128), (wl.BF16, 1024, 64, 128), (wl.F32, 64, 64, 64), (wl.F32, 512, 64, 128)])
def test_ragged_length_without_epsilon(dtype, dqk, dhv, chunk):
    import paper_2503_14376_amd as tfla
    from tests import gpu_util as gu
    w = wl.small(wl.EXP, dtype, B=1, NH=2, T=chunk + 37, dqk=dqk, dhv=dhv, chunk=chunk, seed=1300 + dqk, init_state=False)
    dev = gu.dev_inputs(w, wl.make_inputs(w))
    # q, k of positive mean: the normalisers of the true steps stay away from zero
    q, k = (0.25 * dev[x] + 1.0 for x in ("q", "k"))
    ip = dev["i_pre"] + 115.0
    f = tfla.mlstm_fwd(q, k, dev["v"], ip, dev["f_pre"], chunk=chunk, eps=0.0)
    assert float(f["m_out"].min()) > 104.0
    args = (q, k, dev["v"], ip, dev["f_pre"], dev["dH"], f["n_out"], f["m_out"])
    kept = tfla.mlstm_bwd(*args, chunk=chunk, eps=0.0, fwd_workspace=f["workspace"])
    again = tfla.mlstm_bwd(*args, chunk=chunk, eps=0.0)
    torch.cuda.synchronize()
    for key in ("dq", "dk", "dv", "d_i_pre", "d_f_pre", "dC0"):
        e = gu.rel_err(kept[key], again[key].double().cpu().numpy())
        assert e <= gu.TOL[dtype], (key, e)


# the larger side of the rules that the small problems above do not reach, against the fp64 oracle on the first and the last
# (batch, head): 256-wide output blocks on tensors that end inside a block; fp32 128-column blocks (512 workgroups of 64 rows
# and more: one and two LDS stages, two and four wavefronts, whole and split contractions); fp32 128 x 128 state tiles (192 of
# them and more)
@pytest.mark.parametrize("keep", [True, False])
@pytest.mark.parametrize("variant,dtype,B,NH,T,dqk,dhv,chunk", [
    (wl.EXP, wl.BF16, 2, 8, 2000, 256, 512, 256),       # 256 workgroups of dQ and dK
    (wl.SIG, wl.BF16, 1, 8, 2000, 504, 512, 256),       # 256 of every mode
    (wl.EXP, wl.BF16, 1, 4, 2000, 1000, 1024, 256),     # the same with weights from memory
    (wl.SIG, wl.F32, 2, 8, 1024, 128, 256, 64),         # H and dV: 512 workgroups of 128 columns, two stages
    (wl.EXP, wl.F32, 2, 8, 1024, 256, 128, 128),        # dQ and dK
    (wl.EXP, wl.F32, 2, 8, 1024, 256, 256, 64),         # every mode, one stage
    (wl.SIG, wl.F32, 2, 8, 1000, 256, 248, 128),        # every mode, ragged
    (wl.EXP, wl.F32, 1, 8, 1000, 512, 512, 128),        # every mode, split and ragged
    (wl.EXP, wl.F32, 4, 48, 192, 128, 128, 64),         # 192 state tiles of 128 x 128
    (wl.SIG, wl.F32, 1, 48, 150, 256, 200, 64),         # 192, ragged
])
def test_large_sides_of_the_rules(keep, variant, dtype, B, NH, T, dqk, dhv, chunk):
    w = wl.small(variant, dtype, B=B, NH=NH, T=T, dqk=dqk, dhv=dhv, chunk=chunk, seed=1400 + T + dqk)
    _check_slices(w, dCn=True, keep=keep, scan=True)


# row kernels of the layer whose wavefronts take more than one row (16384 rows and more; 65536 where four lie side by side)
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("B,NH,T,dhv", [(2, 8, 1030, 512), (3, 6, 1000, 264), (2, 8, 1100, 1024), (8, 16, 1030, 128)])
def test_layer_rows_in_rounds(dtype, B, NH, T, dhv):
    test_layer_rows(dtype, 1, B, NH, T, dhv)
