"""GPU parity: the HIP library against the fp64 CPU oracle, element by element, on seeded
inputs, through the C ABI.  Tolerances: max relative error 1e-4 (fp32) and 2e-2 (bf16), taken
per tensor as max|diff| / max|ref| and as the relative L2 error."""
import numpy as np
import pytest
import torch

from oracle import layer as O
from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import DeviceLayer, to_device, to_host
from parity import TOL, check, compare, run_both

pytestmark = pytest.mark.gpu


def _case(shape, case, random_affine=True):
    full = I.full_params(shape.with_(tp_attn=1, tp_ffn=1), case=case, random_affine=random_affine)
    params = I.shard_params(shape, full)
    x, dy = I.activations(shape, case=case)
    return params, x, dy


# fp32: the graded small configuration and ragged / sharded variants -----------------------------

def test_c1_fp32_block():
    shape, _, _ = I.WORKLOADS["C1"]
    params = I.rank_params(shape, case=1)
    x, dy = I.activations(shape, case=1)
    gpu, ref, _ = run_both(shape, params, x, dy, want_partials=True)
    compare(gpu, ref, TOL["f32"], want_partials=True)


@pytest.mark.parametrize("phase", ["both", "attn", "mlp"])
@pytest.mark.parametrize("a,f,rank", [(1, 1, 0), (3, 2, 1)])
def test_fp32_ragged_shapes_and_phases(phase, a, f, rank):
    # hidden 192 = 3 heads x 64, seq 100 (ragged against every tile), batch 3, odd FFN split
    shape = I.LayerShape(192, 3, 328, a, f, rank, 100, 3, "f32")
    params, x, dy = _case(shape, 20 + a)
    rb = (rank == 0)
    gpu, ref, _ = run_both(shape, params, x, dy, phase, rb, not rb)
    compare(gpu, ref, TOL["f32"], phase)


def test_fp32_head_dim_32_and_128():
    for heads, case in ((8, 31), (2, 32)):
        shape = I.LayerShape(256, heads, 512, 1, 1, 0, 70, 2, "f32")
        params, x, dy = _case(shape, case)
        gpu, ref, _ = run_both(shape, params, x, dy)
        compare(gpu, ref, TOL["f32"])


# bf16: tile-spanning, ragged, sharded -----------------------------------------------------------

@pytest.mark.parametrize("phase", ["both", "attn", "mlp"])
@pytest.mark.parametrize("a,f,rank,seq,batch", [(1, 1, 0, 200, 2), (2, 3, 1, 333, 1)])
def test_bf16_ragged_shapes_and_phases(phase, a, f, rank, seq, batch):
    # hidden 512 = 4 heads x 128, FFN 1536; T = 400 / 333 spans two 256-row tiles with a tail
    shape = I.LayerShape(512, 4, 1536, a, f, rank, seq, batch, "bf16")
    params, x, dy = _case(shape, 40 + a)
    rb = (rank == 0)
    gpu, ref, _ = run_both(shape, params, x, dy, phase, rb, not rb, want_partials=(phase == "both"))
    compare(gpu, ref, TOL["bf16"], phase, want_partials=(phase == "both"))


def test_bf16_multi_tile_block():
    # 3 x 3 GEMM tiles with ragged edges, 5 query tiles per head
    shape = I.LayerShape(640, 5, 1928, 1, 1, 0, 600, 1, "bf16")
    params, x, dy = _case(shape, 50)
    report = {}
    gpu, ref, _ = run_both(shape, params, x, dy)
    compare(gpu, ref, TOL["bf16"], report=report)
    print({k: f"{v[0]:.2e}" for k, v in report.items()})


def test_bf16_many_query_blocks():
    # 7 samples x 4 heads x 15 query blocks: enough blocks that attention takes its one-tile-per-step
    # kernels (smaller cases above take the variants that split the key range over two wavefronts)
    shape = I.LayerShape(512, 4, 1024, 1, 1, 0, 1800, 7, "bf16")
    params, x, dy = _case(shape, 52)
    gpu, ref, _ = run_both(shape, params, x, dy)
    compare(gpu, ref, TOL["bf16"])


@pytest.mark.parametrize("phase", ["both", "attn"])
@pytest.mark.parametrize("a,f,rank,seq,batch", [(1, 1, 0, 200, 2), (2, 3, 1, 333, 1), (1, 1, 0, 1, 3)])
def test_bf16_head_dim_64_ragged_shapes(phase, a, f, rank, seq, batch):
    # hidden 384 = 6 heads x 64: the 128-byte-row tile layout of the attention kernels
    shape = I.LayerShape(384, 6, 1536, a, f, rank, seq, batch, "bf16")
    params, x, dy = _case(shape, 70 + a)
    rb = (rank == 0)
    gpu, ref, _ = run_both(shape, params, x, dy, phase, rb, not rb, want_partials=(phase == "both"))
    compare(gpu, ref, TOL["bf16"], phase, want_partials=(phase == "both"))


def test_bf16_head_dim_64_many_and_long_blocks():
    # one-tile-per-step kernels (many (sample, head) pairs) and a longer ragged sequence with few pairs
    for hidden, heads, seq, batch, case in ((512, 8, 1300, 6, 75), (256, 4, 1999, 1, 76)):
        shape = I.LayerShape(hidden, heads, 1024, 1, 1, 0, seq, batch, "bf16")
        params, x, dy = _case(shape, case)
        gpu, ref, _ = run_both(shape, params, x, dy, "attn", want_partials=False)
        compare(gpu, ref, TOL["bf16"], "attn")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("recompute", [False, True])
def test_gelu_tanh_variant(dtype, recompute):
    # the flag must reach the forward epilogue, the backward epilogue and the recomputation
    hidden, heads = (256, 4) if dtype == "f32" else (512, 4)
    shape = I.LayerShape(hidden, heads, 1096, 1, 1, 0, 150, 2, dtype, gelu_tanh=True)
    params, x, dy = _case(shape, 95)
    gpu, ref, _ = run_both(shape, params, x, dy, "both", recompute=recompute)
    compare(gpu, ref, TOL[dtype])
    # and it must make a difference: the erf-form oracle is measurably elsewhere at fp32 resolution
    if dtype == "f32":
        ref_erf = O.layer_fwd(shape.with_(gelu_tanh=False), params, x)["y"]
        assert np.abs(ref_erf - ref["y"]).max() > 1e-5 * np.abs(ref["y"]).max()


def test_bf16_degenerate_sizes():
    # one token per sample (attention is the identity on V), and a single sample of 2 tokens
    for seq, batch, case in ((1, 5, 61), (2, 1, 62)):
        shape = I.LayerShape(256, 2, 264, 1, 1, 0, seq, batch, "bf16")
        params, x, dy = _case(shape, case)
        gpu, ref, _ = run_both(shape, params, x, dy)
        compare(gpu, ref, TOL["bf16"])


@pytest.mark.parametrize("hidden,heads", [(256, 2), (256, 4)])
def test_bf16_sequence_lengths_around_tile_edges(hidden, heads):
    # head dim 128 and 64; lengths on either side of the attention kernels' 32-row blocks, 64-key
    # steps and 128-key tiles: every count of steps from 1 to 5, odd and even numbers of query
    # blocks (the launch order pairs long and short blocks), ragged last tiles
    for seq in (31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 191, 193, 257, 320):
        shape = I.LayerShape(hidden, heads, 256, 1, 1, 0, seq, 2, "bf16")
        params, x, dy = _case(shape, 300 + seq)
        gpu, ref, _ = run_both(shape, params, x, dy, "attn", want_partials=False)
        compare(gpu, ref, TOL["bf16"], "attn")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_recompute_and_accumulate_flags(dtype):
    hidden, heads = (256, 2) if dtype == "bf16" else (128, 2)
    shape = I.LayerShape(hidden, heads, 512, 1, 1, 0, 150, 2, dtype)
    params, x, dy = _case(shape, 70)
    gpu, ref, layer = run_both(shape, params, x, dy)
    xd, dyd = to_device(x, dtype), to_device(dy, dtype)
    # recomputation reproduces the saved-activation path bit for bit
    for n in I.PARAM_NAMES:
        layer.grads[n].fill_(float("nan"))
    dx2 = layer.backward(xd, dyd, recompute=True)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(dx2), gpu["dx"])
    for n in I.PARAM_NAMES:
        assert np.array_equal(to_host(layer.grads[n]), gpu["grads"][n]), n
    # accumulation: a second backward with the flag doubles every parameter gradient
    layer.backward(xd, dyd, accumulate=True)
    torch.cuda.synchronize()
    for n in I.PARAM_NAMES:
        check("acc d" + n, to_host(layer.grads[n]), 2.0 * ref["grads"][n], TOL[dtype])


# dropout variant: masks from the counter-based generator, drawn independently on both sides ------

SEED64 = 0x1234567890ABCDEF


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("phase,recompute", [("both", False), ("both", True), ("attn", False)])
def test_dropout_variant(dtype, phase, recompute):
    # rank 1 of 2 attention ranks: the masks are those of global heads 2 and 3
    hidden, heads = (256, 4) if dtype == "f32" else (512, 4)
    shape = I.LayerShape(hidden, heads, 1096, 2, 1, 1, 150, 2, dtype, drop_attn=40, drop_hidden=30, drop_seed=SEED64)
    params, x, dy = _case(shape, 98)
    want = phase == "both" and not recompute
    gpu, ref, _ = run_both(shape, params, x, dy, phase, recompute=recompute, want_partials=want)
    compare(gpu, ref, TOL[dtype], phase, want_partials=want)
    # and the masks matter: the plain layer is measurably elsewhere
    plain = O.layer_fwd(shape.with_(drop_attn=0, drop_hidden=0), params, x, phase)
    key = "y" if phase == "both" else "p_attn"
    assert np.abs(plain[key] - ref[key]).max() > 4 * TOL[dtype] * np.abs(ref[key]).max()


@pytest.mark.parametrize("heads,hidden", [(8, 1024), (8, 512)])
def test_bf16_dropout_many_blocks_unsplit_kernels(heads, hidden):
    # enough (sample, head, query block) units that the forward and dQ kernels run unsplit;
    # several key blocks per workgroup of the dK/dV kernel; both head dimensions
    shape = I.LayerShape(hidden, heads, 256, 1, 1, 0, 1100, 6, "bf16", drop_attn=64, drop_seed=77)
    params, x, dy = _case(shape, 99)
    gpu, ref, _ = run_both(shape, params, x, dy, "attn")
    compare(gpu, ref, TOL["bf16"], "attn")


def test_bf16_dropout_keeps_few():
    # drop probability 200/256: the output is made of the few kept terms, so a misplaced mask
    # bit anywhere (either bit layout) is a large error
    shape = I.LayerShape(256, 2, 264, 1, 1, 0, 333, 2, "bf16", drop_attn=200, drop_hidden=200, drop_seed=3)
    params, x, dy = _case(shape, 100)
    gpu, ref, _ = run_both(shape, params, x, dy)
    compare(gpu, ref, TOL["bf16"])


def test_dropout_same_seed_same_result_other_seed_other_result():
    shape = I.LayerShape(256, 2, 264, 1, 1, 0, 100, 2, "bf16", drop_attn=64, drop_hidden=64, drop_seed=11)
    params, x, dy = _case(shape, 101)
    xd = to_device(x, "bf16")
    a = to_host(DeviceLayer(shape, params).forward(xd)["y"])
    b = to_host(DeviceLayer(shape, params).forward(xd)["y"])
    c = to_host(DeviceLayer(shape.with_(drop_seed=12), params).forward(xd)["y"])
    assert np.array_equal(a, b) and not np.array_equal(a, c)


def test_bf16_remainder_round_of_large_tiles():
    """Products a little over one or several rounds of 256 large tiles (here 17 x 17 = 289 for the
    FC1 / FC2 / out-proj outputs and weight gradients, 17 x 50 = 850 for the QKV weight gradient)
    are split into a large-tile launch and a small-tile launch over the remainder; 4200 rows and
    4224 columns leave quarters of the last super-tiles outside the matrix."""
    shape = I.LayerShape(4224, 33, 4104, 1, 1, 0, 1050, 4, "bf16")
    params, x, dy = _case(shape, 97)
    gpu, ref, _ = run_both(shape, params, x, dy, want_partials=True)
    compare(gpu, ref, TOL["bf16"], want_partials=True)


@pytest.mark.parametrize("phase", ["both", "attn", "mlp"])
def test_bf16_weight_gradient_output(phase):
    """GX_WGRAD_BF16: the four weight-matrix gradients arrive as bf16, each the fp32 accumulator
    rounded once; everything else is unchanged."""
    shape = I.LayerShape(512, 4, 1096, 2, 1, 1, 150, 2, "bf16")
    params, x, dy = _case(shape, 96)
    gpu, ref, _ = run_both(shape, params, x, dy, phase)
    layer = DeviceLayer(shape, params, wgrad_bf16=True)
    xd, dyd = to_device(x, "bf16"), to_device(dy, "bf16")
    layer.forward(xd, phase)
    dx = layer.backward(xd, dyd, phase)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(dx), gpu["dx"])
    mine = {"both": I.PARAM_NAMES, "attn": I.PARAM_NAMES[:6], "mlp": I.PARAM_NAMES[6:]}[phase]
    first = {}
    for n in mine:
        got = to_host(layer.grads[n])
        first[n] = got
        if n.startswith("w_"):
            assert layer.grads[n].dtype == torch.bfloat16
            assert np.array_equal(got, I.bf16_round(gpu["grads"][n])), n      # one rounding of the same sums
            check("d" + n, got, ref["grads"][n], TOL["bf16"])
        else:
            assert np.array_equal(got, gpu["grads"][n]), n
    # accumulation adds in fp32 and rounds once
    layer.backward(xd, dyd, phase, accumulate=True)
    torch.cuda.synchronize()
    for n in mine:
        got = to_host(layer.grads[n])
        if n.startswith("w_"):
            assert np.array_equal(got, I.bf16_round(first[n] + gpu["grads"][n])), n
        check("acc d" + n, got, 2.0 * ref["grads"][n], TOL["bf16"])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rank_partials_add_up_to_the_unsharded_block(dtype):
    """Simulated ranks run one after another on the GPU; their partial sums, added on the host,
    must reproduce the unsharded oracle block (outputs, input gradient, replicated-parameter
    gradients), and their column-shard gradients must tile the full gradient."""
    if dtype == "bf16":
        base = I.LayerShape(512, 4, 1024, 1, 1, 0, 96, 2, "bf16")
    else:
        base = I.LayerShape(128, 4, 256, 1, 1, 0, 50, 2, "f32")
    a, f = 2, 4
    full = I.full_params(base, case=80, random_affine=True)
    x, dy = I.activations(base, case=80)
    ref = O.layer_fwd(base, full, x)
    dx_ref, g_ref = O.layer_bwd(base, full, dy, ref["cache"])
    tol = TOL[dtype]
    sh = base.with_(tp_attn=a, tp_ffn=f)
    xd = to_device(x, dtype)
    # the harness plays the all-reduce in fp64 on the host and rounds what the next half reads
    attn_layers, p_sum = [], np.zeros_like(ref["h1"])
    for r in range(a):
        L = DeviceLayer(sh.with_(tp_rank=r), I.shard_params(sh, full, rank_attn=r, rank_ffn=0))
        p_sum += to_host(L.forward(xd, "attn", row_bias_attn=(r == 0))["p_attn"])
        attn_layers.append(L)
    h1 = x + p_sum
    check("h1", h1, ref["h1"], tol)
    h1s = I.bf16_round(h1.astype(np.float32)) if dtype == "bf16" else h1.astype(np.float32)
    h1d, dyd = to_device(h1s, dtype), to_device(dy, dtype)
    mlp_layers, m_sum = [], np.zeros_like(ref["y"])
    for r in range(f):
        L = DeviceLayer(sh.with_(tp_rank=r), I.shard_params(sh, full, rank_attn=0, rank_ffn=r))
        m_sum += to_host(L.forward(h1d, "mlp", row_bias_mlp=(r == 0))["p_mlp"])
        mlp_layers.append(L)
    check("y", h1 + m_sum, ref["y"], tol)
    dh1 = dy.astype(np.float64).copy()
    for r, L in enumerate(mlp_layers):
        dh1 += to_host(L.backward(h1d, dyd, "mlp", row_bias_mlp=(r == 0)))
    dh1s = I.bf16_round(dh1.astype(np.float32)) if dtype == "bf16" else dh1.astype(np.float32)
    dh1d = to_device(dh1s, dtype)
    dx = dh1.copy()
    for r, L in enumerate(attn_layers):
        dx += to_host(L.backward(xd, dh1d, "attn", row_bias_attn=(r == 0)))
    torch.cuda.synchronize()
    check("dx", dx, dx_ref, tol)
    G = lambda layers, n: [to_host(L.grads[n]).astype(np.float64) for L in layers]
    for n in ("ln1_g", "ln1_b", "b_o"):
        check("d" + n, sum(G(attn_layers, n)), g_ref[n], tol)
    for n in ("ln2_g", "ln2_b", "b_fc2"):
        check("d" + n, sum(G(mlp_layers, n)), g_ref[n], tol)
    check("dw_o", np.concatenate(G(attn_layers, "w_o"), axis=0), g_ref["w_o"], tol)
    check("dw_fc2", np.concatenate(G(mlp_layers, "w_fc2"), axis=0), g_ref["w_fc2"], tol)
    check("dw_fc1", np.concatenate(G(mlp_layers, "w_fc1"), axis=1), g_ref["w_fc1"], tol)
    check("db_fc1", np.concatenate(G(mlp_layers, "b_fc1")), g_ref["b_fc1"], tol)
    Hl, H = sh.hidden_local, sh.hidden
    for i in range(3):
        cat = np.concatenate([g[:, i * Hl:(i + 1) * Hl] for g in G(attn_layers, "w_qkv")], axis=1)
        check(f"dw_qkv[{i}]", cat, g_ref["w_qkv"][:, i * H:(i + 1) * H], tol)


def test_bitwise_reproducible():
    shape = I.LayerShape(512, 4, 1024, 2, 2, 0, 300, 2, "bf16")
    params, x, dy = _case(shape, 90)
    a, _, _ = run_both(shape, params, x, dy)
    b, _, _ = run_both(shape, params, x, dy)
    assert np.array_equal(a["y"], b["y"]) and np.array_equal(a["dx"], b["dx"])
    for n in I.PARAM_NAMES:
        assert np.array_equal(a["grads"][n], b["grads"][n]), n
    # the overlap switch never changes a result (this layer is small enough to stay on one stream;
    # passes that fork: test_gpu_overlap.py)
    from paper_2504_03662_amd import binding as gx
    gx.set_overlap(False)
    try:
        c, _, _ = run_both(shape, params, x, dy)
    finally:
        gx.set_overlap(True)
    assert np.array_equal(a["dx"], c["dx"])
    for n in I.PARAM_NAMES:
        assert np.array_equal(a["grads"][n], c["grads"][n]), n


@pytest.mark.parametrize("drop", [0, 48])
def test_step_replays_from_a_captured_graph(drop):
    """gx_layer_fwd / gx_layer_bwd only enqueue work, so a step can be captured into a HIP graph; every
    replay, with eager work and synchronisations in between, must reproduce the eager result bit for
    bit (a layer that stays on one stream; forks and joins: test_gpu_overlap.py)."""
    shape = I.LayerShape(512, 4, 1096, 1, 1, 0, 300, 2, "bf16", drop_attn=drop, drop_hidden=drop, drop_seed=9)
    params, x, dy = _case(shape, 102)
    layer = DeviceLayer(shape, params)
    xd, dyd = to_device(x, "bf16"), to_device(dy, "bf16")
    y, dx = layer.empty_act(), layer.empty_act()

    def step():
        layer.forward(xd, out=y)
        layer.backward(xd, dyd, out=dx)

    def snapshot():
        torch.cuda.synchronize()
        return [to_host(y).copy(), to_host(dx).copy()] + [to_host(layer.grads[n]).copy() for n in I.PARAM_NAMES]

    for _ in range(2):                       # first calls create streams, events and kernel attributes
        step()
    want = snapshot()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for _ in range(3):
        y.zero_()
        dx.zero_()
        for t in layer.grads.values():
            t.fill_(3.0)
        torch.cuda.synchronize()
        graph.replay()
        got = snapshot()
        for a, b in zip(got, want):
            assert np.array_equal(a, b)
        step()                               # eager work between replays
        torch.cuda.synchronize()


def test_launch_timing_record():
    """gx_prof_*: every launch site of one forward + backward shows up once, in launch order, with a
    positive duration, and the record is cleared by the collect."""
    from paper_2504_03662_amd import binding as gx
    shape = I.LayerShape(256, 2, 512, 1, 1, 0, 64, 2, "bf16")
    params, x, dy = _case(shape, 95)
    layer = DeviceLayer(shape, params)
    xd, dyd = to_device(x, "bf16"), to_device(dy, "bf16")
    layer.forward(xd)
    layer.backward(xd, dyd)
    gx.prof_enable(True)
    try:
        layer.forward(xd)
        fwd = gx.prof_collect()
        layer.backward(xd, dyd)
        bwd = gx.prof_collect()
        assert gx.prof_collect() == []
    finally:
        gx.prof_enable(False)
    G = gx.GX_KC_GEMM
    assert [c for c, _ in fwd] == [gx.GX_KC_LN_FWD, G + 1, gx.GX_KC_ATTN_FWD, G + 2, gx.GX_KC_LN_FWD, G + 3, G + 2]
    # column sums: the stage-1 pass over dqkv and the one finishing launch (the other bias gradients'
    # partial sums come out of the LayerNorm-backward kernel and the GELU' epilogue)
    assert sorted(c for c, _ in bwd) == sorted([gx.GX_KC_COLSUM] * 2 + [gx.GX_KC_LN_BWD] * 2 + [gx.GX_KC_ATTN_BWD]
                                               + [G + 25] * 4 + [G + 14] + [G + 10] * 3)
    assert all(t > 0 for _, t in fwd + bwd)


def test_calls_from_two_host_threads_overlap_safely():
    """Two threads that run forward + backward passes at the same time, each on its own stream and
    buffers, get bit for bit what one thread alone gets (a layer that stays on one stream; each
    thread's own side stream: test_gpu_overlap.py)."""
    import threading
    shape = I.LayerShape(512, 4, 1096, 2, 1, 0, 300, 2, "bf16")
    params, x, dy = _case(shape, 96)
    xd, dyd = to_device(x, "bf16"), to_device(dy, "bf16")

    def run(reps, out):
        layer = DeviceLayer(shape, params)
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(reps):
                y = layer.forward(xd)["y"]
                dx = layer.backward(xd, dyd)
            torch.cuda.current_stream().synchronize()
        out.append((to_host(y), to_host(dx), {n: to_host(layer.grads[n]) for n in I.PARAM_NAMES}))

    alone = []
    run(1, alone)
    torch.cuda.synchronize()
    res = [[], []]
    threads = [threading.Thread(target=run, args=(20, res[k])) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for r in res:
        y, dx, g = r[0]
        assert np.array_equal(y, alone[0][0]) and np.array_equal(dx, alone[0][1])
        for n in I.PARAM_NAMES:
            assert np.array_equal(g[n], alone[0][2][n]), n

