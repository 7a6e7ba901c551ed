"""The expert FFN's row tiles and work lists at the sizes where they can go
wrong: group sizes around every tile and row-block boundary, several row
tiles and bands per group, partial column tiles, a second pass on the same
dispatch, replays of captured passes, and grids of a few workgroups.

Expected values come from the oracle; the bounds are those of the other
parity tests (bf16: h, the expert rows and the output are each rounded to
bf16, 2^-9 relative, so rows are about 3e-3 off; fp8: a flipped code of h moves
a row by up to 2.5e-2)."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2606_22541_amd import inputs
from paper_2606_22541_amd import moe_stage as C
from paper_2606_22541_amd.stage import ExpertStage, bf16_bits, quantize_fp8, to_device_routing

from gpu_common import BF16_TOL, FP8_TOL, bits_to_f64, check_outputs, log, oracle_run, row_rel_l2

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))

# Rows of each local expert: around the 32-row blocks, the small tiles' limits
# (64, 160, 192), one and two large tiles (320, 640; fp8: 128, 256), a band of
# four row tiles and beyond, and empty groups between.
COUNTS = {
    "small": (1, 31, 32, 33, 0, 63, 64, 65, 95, 96),
    "medium": (97, 127, 128, 129, 159, 160, 161, 191, 192, 193),
    "large": (223, 224, 255, 256, 257, 0, 288, 289, 319, 320),
    "several_tiles": (321, 640, 641, 1281, 1600, 5, 70),
    "one_row": (0, 1, 0),
    "fp8_blocks": (15, 16, 17, 47, 48, 49, 111, 112, 113, 385),
}


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("name", sorted(COUNTS))
def test_group_sizes_at_the_tiles_edges(name, dtype):
    counts = np.asarray(COUNTS[name], np.int32)
    n = int(counts.sum())
    # d: a last column tile of half the width; f: three h tiles
    cfg = inputs.MoEConfig("sizes", d=384, f=384, E=16, e0=0, E_loc=len(counts), k=1, lengths=(n,),
                           dtype=dtype, seed=70 + n)
    log("counts %s (%s)" % (counts.tolist(), dtype))
    wts = inputs.make_weights(cfg, "cuda")
    ow = oracle.OracleWeights(wts, dtype)
    x = inputs.make_microbatches(cfg, "cuda")[0].x
    rows_x, _, _ = oracle.stage_inputs_x(bf16_bits(x), dtype)
    ref = oracle.run_grouped(cfg, ow, rows_x, counts)["y"]
    scales = None
    if dtype == "fp8":
        x, scales = quantize_fp8(x)
    y = torch.full((n, cfg.d), float("nan"), dtype=torch.bfloat16, device="cuda")
    with ExpertStage(cfg, wts, max_tokens=n) as st:
        st.expert_ffn_grouped(0, x, torch.from_numpy(counts).to("cuda"), y, row_scales=scales)
        st.sync()
    got = bits_to_f64(bf16_bits(y))
    assert np.all(np.isfinite(got))
    err = row_rel_l2(got, ref)
    assert err.max() <= (FP8_TOL if dtype == "fp8" else BF16_TOL), (int(err.argmax()), err.max())


@pytest.mark.parametrize("counts", [(193, 255, 256, 257, 288, 289, 319, 320), (200, 0, 260, 320, 193, 224, 225, 0, 310),
                                    (257, 256, 321, 255, 260, 250, 240, 230), (257, 256, 192, 255, 260, 250, 240, 230),
                                    (320,) * 8, (193,) * 8])
def test_down_product_with_row_tiles_of_its_own(counts):
    """Groups that the gate/up product splits to fill one round (f: 16 column
    tiles) and the down product (28 column tiles) takes whole; and the same
    with one group too tall, or one small, where it does not.  Run twice, bits
    compared (each call builds its row tiles and counters anew)."""
    counts = np.asarray(counts, np.int32)
    n = int(counts.sum())
    cfg = inputs.MoEConfig("own", d=7168, f=2048, E=16, e0=0, E_loc=len(counts), k=1, lengths=(n,), dtype="bf16", seed=95)
    log("counts %s" % (counts.tolist(),))
    wts = inputs.make_weights(cfg, "cuda")
    x = inputs.make_microbatches(cfg, "cuda")[0].x
    ys = [torch.full((n, cfg.d), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    with ExpertStage(cfg, wts, max_tokens=n) as st:
        for y in ys:
            st.expert_ffn_grouped(0, x, torch.from_numpy(counts).to("cuda"), y)
            st.sync()
    assert torch.equal(ys[0], ys[1])
    # every 5th row of each group (and its last) against fp32 products of the same
    # bf16 values: h and y are each rounded to bf16, as in the other bounds
    r0 = 0
    for g, c in enumerate(counts.tolist()):
        if c:
            pick = torch.tensor(sorted(set(range(0, c, 5)) | {c - 1}), device="cuda") + r0
            xr = x[pick].float()
            h = torch.nn.functional.silu(xr @ wts.w_gate[g].float().T) * (xr @ wts.w_up[g].float().T)
            ref = (h.to(torch.bfloat16).float() @ wts.w_down[g].float().T).double().cpu().numpy()
            err = row_rel_l2(ys[0][pick].double().cpu().numpy(), ref)
            assert np.all(err <= BF16_TOL), (g, c, err.max())
        r0 += c


@pytest.mark.parametrize("d,f", [(4000000, 128), (128, 4000000)])
def test_rows_so_long_that_tiles_are_lower(d, f):
    """320 rows of 4,000,000 elements pass 2^31 bytes, so the tiles of such
    rows have 256 at most: every row and column is written."""
    n = 320
    cfg = inputs.MoEConfig("long", d=d, f=f, E=2, e0=0, E_loc=1, k=2, lengths=(n // 2,), dtype="bf16", seed=99)
    log("d %d f %d" % (d, f))
    wts = inputs.make_weights(cfg, "cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(99)
    x = torch.randn((n, d), generator=g, device="cuda", dtype=torch.bfloat16)
    y = torch.full((n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    with ExpertStage(cfg, wts, max_tokens=n // 2) as st:
        st.expert_ffn_grouped(0, x, torch.tensor([n], dtype=torch.int32, device="cuda"), y)
        st.sync()
    # fp32 products of the same bf16 values, rows from every block
    pick = torch.tensor([0, 31, 32, 159, 160, 255, 256, 267, 268, 300, 319], device="cuda")
    xr = x[pick].float()
    h = torch.nn.functional.silu(xr @ wts.w_gate[0].float().T) * (xr @ wts.w_up[0].float().T)
    ref = h.to(torch.bfloat16).float() @ wts.w_down[0].float().T
    got = y[pick].float()
    assert torch.isfinite(y).all()
    err = (torch.linalg.vector_norm(got - ref, dim=1) / torch.linalg.vector_norm(ref, dim=1)).cpu().numpy()
    assert np.all(err <= BF16_TOL), err


@pytest.mark.parametrize("E,e0,E_loc,k,T", [(5, 2, 1, 3, 700), (9, 0, 3, 4, 1100), (70, 5, 33, 8, 900),
                                            (300, 40, 200, 8, 1500), (2, 0, 2, 2, 65)])
def test_placement_with_any_number_of_local_experts(E, e0, E_loc, k, T):
    """Ranks inside a 64-slot step come from ballots over the bits of the local
    index: indices of one bit, of several, and not a power of two of them."""
    rng = np.random.default_rng(E * 1000 + T)
    ids = rng.integers(-1, E, size=(T, k)).astype(np.int32)
    ids[: T // 4] = e0                                   # long runs of one expert
    ref = oracle.dispatch(ids, E, e0, E_loc)
    dev = torch.from_numpy(ids).to("cuda")
    counts = torch.full((E,), -7, dtype=torch.int32, device="cuda")
    offsets = torch.full((E_loc + 1,), -7, dtype=torch.int32, device="cuda")
    sor = torch.full((T * k,), -7, dtype=torch.int32, device="cuda")
    ros = torch.full((T * k,), -7, dtype=torch.int32, device="cuda")
    C.moe_dispatch_index_noalloc(dev, T, k, E, e0, E_loc, counts, offsets, sor, ros)
    torch.cuda.synchronize()
    n = int(ref["offsets"][-1])
    assert np.array_equal(counts.cpu().numpy(), ref["counts"])
    assert np.array_equal(offsets.cpu().numpy(), ref["offsets"])
    assert np.array_equal(sor.cpu().numpy()[:n], ref["slot_of_row"])
    assert np.array_equal(ros.cpu().numpy(), ref["row_of_slot"])


def _setup(dtype, seed):
    cfg = inputs.MoEConfig("again", d=512, f=256, E=16, e0=0, E_loc=6, k=4, lengths=(900,), dtype=dtype,
                           has_shared=True, seed=seed)
    wts = inputs.make_weights(cfg, "cuda")
    mb = inputs.make_microbatches(cfg, "cuda")[0]
    ids, w = to_device_routing(mb.ids, mb.w)
    out = torch.empty((cfg.lengths[0], cfg.d), dtype=torch.bfloat16, device="cuda")
    x, xs = quantize_fp8(mb.x) if dtype == "fp8" else (mb.x.clone(), None)
    return cfg, wts, oracle.OracleWeights(wts, dtype), mb, ids, w, out, x, xs


def _check(cfg, ow, mb, out, what):
    tol = FP8_TOL if cfg.dtype == "fp8" else BF16_TOL
    check_outputs(bf16_bits(out), oracle_run(cfg, ow, mb), tol, what)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_second_pass_on_one_dispatch(dtype):
    """moe_expert_ffn twice after one moe_dispatch, the token rows changed in
    between (fp8: the codes; their scales were gathered by the dispatch): the
    second pass computes everything again."""
    cfg, wts, ow, mb, ids, w, out, x, xs = _setup(dtype, 81)
    with ExpertStage(cfg, wts) as st:
        m = st.microbatch(x, ids, w, out, xs)
        st.dispatch(0, m)
        st.expert_ffn(0)
        st.combine(0)
        torch.cuda.synchronize()
        _check(cfg, ow, mb, out, "first pass")
        x.copy_(x.flip(0)) if dtype == "bf16" else x.zero_()
        out.fill_(float("nan"))
        st.expert_ffn(0)
        st.combine(0)
        st.sync()
    if dtype == "bf16":
        mb.x = x
        _check(cfg, ow, mb, out, "second pass")
    else:
        assert torch.all(out == 0)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("whole", [True, False])
def test_captured_pass_replays(dtype, whole):
    """A captured submit, and a captured moe_expert_ffn between an eager
    dispatch and combine, replayed with new token rows and eager work between
    the replays: every replay computes its own rows."""
    cfg, wts, ow, mb, ids, w, out, x, xs = _setup(dtype, 83)
    with ExpertStage(cfg, wts) as st:
        m = st.microbatch(x, ids, w, out, xs)
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            st.dispatch(0, m)
            st.expert_ffn(0)
            st.combine(0)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            if whole:
                st.dispatch(0, m)
            st.expert_ffn(0)
            if whole:
                st.combine(0)
        for r in range(4):
            rows = mb.x.roll(r, 0).contiguous()
            if dtype == "fp8":
                codes, scales = quantize_fp8(rows)
                x.copy_(codes)
                xs.copy_(scales)
            else:
                x.copy_(rows)
            out.fill_(float("nan"))
            torch.cuda.synchronize()
            if not whole:
                st.dispatch(0, m)
                torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            if not whole:
                st.combine(0)
                torch.cuda.synchronize()
            mb_r = inputs.MicroBatch(x=rows, ids=mb.ids, w=mb.w)
            _check(cfg, ow, mb_r, out, "replay %d" % r)
            if r == 1:                       # an eager pass between the replays
                out.fill_(float("nan"))
                st.dispatch(0, m)
                st.expert_ffn(0)
                st.combine(0)
                torch.cuda.synchronize()
                _check(cfg, ow, mb_r, out, "eager pass")
        st.sync()


@pytest.mark.parametrize("captured", ["dispatch", "submit"])
def test_second_pass_after_a_capture_on_its_slot(captured):
    """moe_expert_ffn on a dispatch whose counters are used up although the
    calls before it look as if they were not: a dispatch that was captured but
    not replayed came after the pass that used them, or a replayed submit of
    the slot did.  The token rows change in between: it computes them again."""
    cfg, wts, ow, mb, ids, w, out, x, xs = _setup("bf16", 85)
    with ExpertStage(cfg, wts) as st:
        m = st.microbatch(x, ids, w, out, xs)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        if captured == "submit":
            with torch.cuda.graph(g, stream=s):
                st.submit(m)
        with torch.cuda.stream(s):
            st.dispatch(0, m)
            if captured == "dispatch":
                st.expert_ffn(0)
                st.combine(0)
        s.synchronize()
        if captured == "dispatch":
            with torch.cuda.graph(g, stream=s):
                st.dispatch(0, m)
        else:
            with torch.cuda.stream(s):
                g.replay()
            s.synchronize()
        _check(cfg, ow, mb, out, "first pass")
        x.copy_(x.flip(0))
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            st.expert_ffn(0)
            st.combine(0)
        s.synchronize()
        st.sync()
    mb.x = x
    _check(cfg, ow, mb, out, "second pass")


def test_second_pass_with_row_tiles_of_the_down_product():
    """moe_expert_ffn twice after one moe_dispatch of groups that the down
    product takes whole and the gate/up product splits: the second pass finds
    the counters cleared, those kept per group included."""
    T = 2100                                             # about 262 rows an expert
    cfg = inputs.MoEConfig("own2", d=7168, f=2048, E=8, e0=0, E_loc=8, k=1, lengths=(T,), dtype="bf16", seed=97)
    wts = inputs.make_weights(cfg, "cuda")
    mb = inputs.make_microbatches(cfg, "cuda")[0]
    ids, w = to_device_routing(mb.ids, mb.w)
    outs = [torch.full((T, cfg.d), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    x = mb.x.clone()
    with ExpertStage(cfg, wts) as st:
        st.dispatch(0, st.microbatch(x, ids, w, outs[0]))
        view = st.view(0, rows=False)
        rows = np.diff(view["offsets"])
        assert rows.min() > 192 and rows.max() <= 320, rows
        st.expert_ffn(0)
        st.combine(0)
        torch.cuda.synchronize()
        outs[1].copy_(outs[0])
        x.copy_(x.flip(0))
        outs[0].fill_(float("nan"))
        st.expert_ffn(0)
        st.combine(0)
        torch.cuda.synchronize()
        outs[2].copy_(outs[0])
        st.sync()
    # every 7th token against fp32 products of the same bf16 values
    pick = torch.arange(0, T, 7, device="cuda")
    for rows_in, out in ((mb.x, outs[1]), (x, outs[2])):
        xr = rows_in[pick].float()
        ref = torch.zeros((len(pick), cfg.d), device="cuda")
        for e in range(cfg.E_loc):
            at = (ids[pick, 0] == e).nonzero()[:, 0]
            h = torch.nn.functional.silu(xr[at] @ wts.w_gate[e].float().T) * (xr[at] @ wts.w_up[e].float().T)
            y = (h.to(torch.bfloat16).float() @ wts.w_down[e].float().T).to(torch.bfloat16).float()
            ref[at] = y * w[pick][at]
        err = row_rel_l2(out[pick].double().cpu().numpy(), ref.double().cpu().numpy())
        assert np.all(err <= BF16_TOL), err.max()


@pytest.mark.parametrize("dtype,E_loc", [("bf16", 2), ("fp8", 4)])
def test_passes_on_several_streams_give_the_same_bits(dtype, E_loc):
    """Micro-batches of one round of items whose weights are a long stream: on
    one stream one launch runs both products, on three a launch each.  Same
    bits, with two micro-batches per slot in flight."""
    T = 700
    cfg = inputs.MoEConfig("streams", d=7168, f=2048, E=8, e0=0, E_loc=E_loc, k=2, lengths=(T,) * 6, dtype=dtype,
                           seed=101)
    wts = inputs.make_weights(cfg, "cuda")
    mbs = inputs.make_microbatches(cfg, "cuda")
    args, outs = [], []
    for mb in mbs:
        ids, w = to_device_routing(mb.ids, mb.w)
        x, xs = quantize_fp8(mb.x) if dtype == "fp8" else (mb.x, None)
        args.append((x, ids, w, xs))
    for streams in ([torch.cuda.current_stream()], [torch.cuda.Stream() for _ in range(3)]):
        log("%s on %d streams" % (dtype, len(streams)))
        out = [torch.full((T, cfg.d), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in mbs]
        with ExpertStage(cfg, wts, n_slots=3) as st:
            torch.cuda.synchronize()
            for r in range(2):                 # the second time every slot's stream is known
                for i, (x, ids, w, xs) in enumerate(args):
                    with torch.cuda.stream(streams[i % len(streams)]):
                        st.submit(st.microbatch(x, ids, w, out[i], xs))
            st.sync()
            torch.cuda.synchronize()
        outs.append(out)
    for a, b in zip(*outs):
        assert torch.isfinite(a).all()
        assert torch.equal(a, b)
    if dtype == "bf16":                        # tokens of one local expert, against fp32 products
        x, ids, w, _ = args[0]
        t = ((ids[:, 0] < E_loc) != (ids[:, 1] < E_loc)).nonzero()[::5, 0]
        j = (ids[t, 1] < E_loc).long()
        e = ids[t, j]
        ref = torch.zeros((len(t), cfg.d), device="cuda")
        for g in range(E_loc):
            at = (e == g).nonzero()[:, 0]
            xr = x[t[at]].float()
            h = torch.nn.functional.silu(xr @ wts.w_gate[g].float().T) * (xr @ wts.w_up[g].float().T)
            ref[at] = (h.to(torch.bfloat16).float() @ wts.w_down[g].float().T).to(torch.bfloat16).float()
        ref *= w[t, j][:, None]
        err = row_rel_l2(outs[1][0][t].double().cpu().numpy(), ref.double().cpu().numpy())
        assert np.all(err <= BF16_TOL), err.max()


def test_grids_of_a_few_workgroups():
    """Streams of 16 and of 32 compute units: lists of two and of four
    workgroups, so nearly every item comes from a ticket.  In a child process:
    each masked stream takes a hardware queue."""
    r = subprocess.run([sys.executable, "-u", os.path.join(HERE, "few_cus_child.py")],
                       capture_output=True, text=True, timeout=110)
    print(r.stdout[-3000:], flush=True)
    assert r.returncode == 0, r.stderr[-3000:]
    assert "FEW CUS OK" in r.stdout
