"""GPU parity of the whole layer (Eq. 4-5: LayerNorm, attention, MLP, skips) through the C ABI
against the fp64 oracle, element by element on the same seeded inputs.  Tolerance as for the
attention layer: max-norm relative error per tensor, 1e-5 in fp32 and 2e-2 in bf16."""
import numpy as np
import pytest

from oracle import astl_oracle
from paper_2409_06206_amd import gswa, synth
from tests import parity

pytestmark = pytest.mark.gpu

SMALL = [
    # fp32: vector and scalar channel layouts of the per-token kernels, several row passes
    dict(B=1, H=16, W=16, C=60, heads=6, groups=2, window=8, shift=4, dtype="f32", hidden=120),
    dict(B=2, H=8, W=8, C=12, heads=2, groups=1, window=4, shift=0, dtype="f32", hidden=20),
    dict(B=1, H=8, W=12, C=6, heads=2, groups=2, window=4, shift=1, dtype="f32", hidden=9),
    dict(B=1, H=8, W=8, C=68, heads=4, groups=2, window=4, shift=2, dtype="f32", hidden=100),
    dict(B=1, H=8, W=8, C=200, heads=4, groups=1, window=4, shift=2, dtype="f32", hidden=64),
    dict(B=1, H=8, W=8, C=66, heads=6, groups=3, window=4, shift=0, dtype="f32", hidden=40),
    # bf16: the benchmark's channel counts, every group setting, both window sizes
    dict(B=2, H=16, W=16, C=60, heads=6, groups=1, window=8, shift=0, dtype="bf16", hidden=120),
    dict(B=2, H=16, W=16, C=60, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=120),
    dict(B=3, H=16, W=24, C=60, heads=6, groups=3, window=8, shift=4, dtype="bf16", hidden=120),
    dict(B=1, H=16, W=16, C=60, heads=6, groups=6, window=8, shift=0, dtype="bf16", hidden=120),
    dict(B=1, H=24, W=24, C=60, heads=4, groups=2, window=12, shift=6, dtype="bf16", hidden=120, dqk=4),
    dict(B=1, H=16, W=16, C=180, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=360),
    dict(B=1, H=8, W=8, C=30, heads=3, groups=1, window=4, shift=2, dtype="bf16", hidden=50),
    dict(B=1, H=16, W=16, C=60, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=60),
    dict(B=5, H=8, W=8, C=60, heads=6, groups=2, window=8, shift=0, dtype="bf16", hidden=128),
]


def _id(c):
    return "-".join(f"{k}{v}" for k, v in c.items())


@pytest.mark.parametrize("case", SMALL, ids=_id)
def test_layer_matches_oracle(case):
    print("case", case, flush=True)
    parity.check_block(astl_oracle, **case)


@pytest.mark.parametrize("case", [SMALL[0], SMALL[7], SMALL[10]], ids=_id)
def test_init_regime(case):
    """Identity LayerNorms, small weights: the skip path dominates y, the gradients still have to match."""
    print("case", case, flush=True)
    parity.check_block(astl_oracle, regime="init", **case)


@pytest.mark.parametrize("case", [SMALL[7], SMALL[10]], ids=_id)
def test_every_path_of_the_attention_layer(case):
    print("case", case, flush=True)
    parity.check_block(astl_oracle, extra_flags=gswa.GSWA_FORCE_STAGED, **case)


@pytest.mark.parametrize("case", [SMALL[0], SMALL[7], SMALL[11]], ids=_id)
def test_inference_call_gives_the_training_output(case):
    print("case", case, flush=True)
    import torch
    _, blk = parity.check_block(astl_oracle, backward=False, **case)
    y_inf = blk.y.clone()
    blk.forward(keep=True)
    torch.cuda.synchronize()
    assert torch.equal(y_inf, blk.y)


@pytest.mark.parametrize("case", [
    SMALL[0], SMALL[7],
    # a wide layer with enough tokens for the streaming weight-gradient kernel, whose sum then writes or adds
    # straight into the gradients of the two MLP maps
    dict(B=4, H=64, W=64, C=180, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=360),
], ids=_id)
def test_accumulate_flag_adds_into_every_parameter_gradient(case):
    print("case", case, flush=True)
    import torch
    _, blk = parity.check_block(astl_oracle, **case)
    first = {k: v.clone() for k, v in blk.grads.items()}
    from paper_2409_06206_amd import astl
    c = dict(case)
    blk.desc = astl.make_desc(c["B"], c["H"], c["W"], c["C"], c["heads"], c["groups"], c["window"], c["shift"],
                              c["dtype"], c["hidden"], flags=gswa.GSWA_ACCUM_WGRAD, dqk=c.get("dqk", 0))
    blk.backward()
    torch.cuda.synchronize()
    for k, v in blk.grads.items():
        want = 2.0 * first[k]
        err = float((v - want).abs().max()) / max(float(want.abs().max()), 1e-30)
        assert err <= 1e-3, (k, err)


@pytest.mark.parametrize("name", ["astl_c2", "astl_agile", "astl_c3"])
def test_benchmark_shape_pair_against_the_oracle(name):
    """The two layers of a whole-layer workload at its full size, every output element."""
    cfg = synth.CONFIGS[name]
    for li, shift in enumerate(cfg["layers"]):
        case = dict(B=cfg["B"], H=cfg["H"], W=cfg["W"], C=cfg["C"], heads=cfg["heads"], groups=2,
                    window=cfg["window"], shift=shift, dtype=cfg["dtype"], hidden=cfg["hidden"],
                    dqk=cfg.get("dqk", 0))
        print("case", case, flush=True)
        parity.check_block(astl_oracle, seed=synth.LAYER_SEED0 + li, **case)


@pytest.mark.parametrize("case", [
    dict(B=2, H=64, W=32, C=180, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=360),
    # 4800 tokens: 37 passes of 128 and a ragged one
    dict(B=3, H=40, W=40, C=180, heads=6, groups=3, window=8, shift=0, dtype="bf16", hidden=360),
    dict(B=4, H=64, W=64, C=180, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=360),
], ids=_id)
def test_wide_layer_with_enough_tokens_for_the_streaming_weight_gradients(case):
    """C = 180, hidden 360 from 4096 tokens on (the scratch is everything behind h | dpre in the workspace):
    the MLP's four weight gradients come from ONE launch of the kernel that streams the rows once and sums
    per-workgroup partial arrays in a fixed order, straight into the gradients."""
    import torch
    print("case", case, flush=True)
    gswa.gswa_profile_enable(True)
    gswa.gswa_profile_collect()
    parity.check_block(astl_oracle, **case)
    torch.cuda.synchronize()
    names, dropped = gswa.gswa_profile_collect()
    gswa.gswa_profile_enable(False)
    assert dropped == 0
    assert names["fc_wgrad"][1] == 1 and "fill_zero" not in names, names


@pytest.mark.parametrize("groups", [1, 2])
@pytest.mark.parametrize("H,W", [(40, 104), (136, 248)])
def test_weight_gradients_of_a_last_pass_half_full(groups, H, W):
    """65 and 527 windows of 64 tokens: the weight-gradient kernels take 128 tokens a pass, the last one's second half lies
    past the last row (one group: both streaming gradients; two: the projection's); 527 also wraps the grid's rounds."""
    print("case", groups, H, W, flush=True)
    parity.check_block(astl_oracle, B=1, H=H, W=W, C=180, heads=6, groups=groups, window=8, shift=4, dtype="bf16", hidden=360)


def test_wide_layer_with_few_tokens_keeps_the_gradient_copies():
    """2048 tokens: too few rows for the streaming weight-gradient kernel (it takes 4096 and more); the layer
    takes the kernels that add into 16 gradient copies (and still the streaming MLP kernels)."""
    import torch
    case = dict(B=1, H=64, W=32, C=180, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=360)
    print("case", case, flush=True)
    gswa.gswa_profile_enable(True)
    gswa.gswa_profile_collect()
    parity.check_block(astl_oracle, **case)
    torch.cuda.synchronize()
    names, dropped = gswa.gswa_profile_collect()
    gswa.gswa_profile_enable(False)
    assert dropped == 0
    assert names["fc_wgrad"][1] == 2 and "fill_zero" in names and "mlp_bwd" in names, names


@pytest.mark.parametrize("case,kernels", [
    # hidden 400 > 384: the first map (180 -> 400) keeps its whole weight matrix in LDS and takes Eq. 4's skip and
    # LN_2 in its operand read and the GELU in its stores; the second (K = 400) runs on the chunked kernel
    (dict(B=1, H=64, W=64, C=180, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=400), ("fc1_linear", "fc2_linear")),
    # 256 channels > 192: both maps on the whole-matrix kernel with 512 threads (K = 256 and 288: more than six
    # steps of 32), LN_2 in the operand read of the first; ragged last 16-row tile (4160 tokens)
    (dict(B=1, H=80, W=52, C=256, heads=4, groups=2, window=4, shift=2, dtype="bf16", hidden=288), ("fc1_linear", "fc2_linear")),
], ids=lambda v: _id(v) if isinstance(v, dict) else "")
def test_wide_layers_beyond_the_streaming_mlp_kernels(case, kernels):
    """Wide bf16 layers that the streaming MLP kernels do not take (hidden > 384 or C > 192), with enough
    tokens (>= 4096) for the linear-map kernel that holds a whole weight matrix in LDS."""
    import torch
    print("case", case, flush=True)
    gswa.gswa_profile_enable(True)
    gswa.gswa_profile_collect()
    parity.check_block(astl_oracle, **case)
    torch.cuda.synchronize()
    names, dropped = gswa.gswa_profile_collect()
    gswa.gswa_profile_enable(False)
    assert dropped == 0
    assert all(k in names for k in kernels) and "mlp_fwd" not in names, names
    # LN_2 of the forward and of the backward's recomputation ride in the first map: only LN_1 is launched (twice)
    assert names["ln_fwd"][1] == 2, names


def test_wide_layer_backward_is_run_to_run_identical():
    """A wide bf16 layer with enough tokens for the streaming weight-gradient kernel sums every parameter
    gradient in a fixed order (partial vectors per workgroup, no atomics, no flag needed): two backward passes
    give the same bits."""
    import torch
    case = dict(B=4, H=64, W=64, C=180, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=360)
    print("case", case, flush=True)
    _, blk = parity.check_block(astl_oracle, **case)
    first = {k: v.clone() for k, v in blk.grads.items()}
    dx = blk.dx.clone()
    for _ in range(2):
        blk.backward()
        torch.cuda.synchronize()
        assert torch.equal(blk.dx, dx)
        for k, v in blk.grads.items():
            assert torch.equal(v, first[k]), k


@pytest.mark.parametrize("case", [SMALL[0], SMALL[8]], ids=_id)
def test_groups_without_the_cascade(case):
    print("case", case, flush=True)
    parity.check_block(astl_oracle, cascade=False, **case)


@pytest.mark.parametrize("eps", [1e-6, 1e-2, 0.5])
def test_eps_enters_both_layer_norms(eps):
    """A large eps changes the result visibly; both sides must take it from the descriptor."""
    case = dict(SMALL[7])
    print("case", case, "eps", eps, flush=True)
    parity.check_block(astl_oracle, eps=eps, **case)


@pytest.mark.parametrize("case", [
    SMALL[0],   # fp32, one workgroup per window
    SMALL[7],   # narrow, fused MLP kernels
    SMALL[10],  # 12x12 windows, one workgroup per window
    SMALL[11],  # wide, streaming MLP kernels
    # hidden 400: the GELU and its derivative in the linear maps of 4096 rows and more
    dict(B=1, H=64, W=64, C=180, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=400),
], ids=_id)
def test_gelu_derivative_at_subnormal_arguments(case):
    """W1 = 0: the pre-activations are b1 alone, here zero, subnormal and the smallest normal numbers of either sign, where
    GELU' is 1/2.  An argument whose derivative is lost shows as an entry of d b1 and a row of d W1 on their own scale."""
    import torch
    from paper_2409_06206_amd import runner
    c = dict(case)
    hidden, dtype = c.pop("hidden"), c.pop("dtype")
    B, H, W, C, heads, groups, window, shift = (c[k] for k in ("B", "H", "W", "C", "heads", "groups", "window", "shift"))
    dqk = c.get("dqk", 0)
    p = synth.astl_params(C, heads, groups, window, hidden, synth.LAYER_SEED0, "stress", dqk)
    least = 2.0 ** (-149 if dtype == "f32" else -133)
    args = np.array([0.0, least, 2.0 ** -129, 2.0 ** -128, 1.25 * 2.0 ** -128, 2.0 ** -126, 1e-30, -0.0, -least, -2.0 ** -129, -1e-30])
    p["w_fc1"] = np.zeros_like(p["w_fc1"])
    p["b_fc1"] = args[np.arange(hidden) % args.size].astype(np.float32)
    p = {k: synth.quantize(v, dtype) for k, v in p.items()}
    assert (p["b_fc1"][:2] == args[:2]).all()
    x, dy = (synth.quantize(a, dtype) for a in synth.activations(B, H, W, C, synth.ACT_SEED))
    blk = runner.DeviceBlock(B, H, W, C, heads, groups, window, shift, dtype, hidden, dqk=dqk)
    blk.set_params(p)
    blk.set_inputs(x, dy)
    blk.forward()
    blk.backward()
    torch.cuda.synchronize()
    got = blk.results()
    _, g = astl_oracle.backward(x, dy, p, heads=heads, groups=groups, window=window, shift=shift, dqk=dqk)
    for k in ("b_fc1", "w_fc1"):
        err = parity.rel_err(got["d" + k], g[k])
        print(k, err, flush=True)
        assert err <= parity.TOL[dtype], (k, err)


@pytest.mark.parametrize("C,heads,hidden", [(180, 6, 360), (180, 6, 400), (68, 4, 32)])
def test_layer_norm_of_a_row_whose_squares_overflow(C, heads, hidden):
    """One token of alternating +-1e20: finite, but the sum of its squared distances is not (in fp32), 1/sqrt of it is zero and
    the row of LN is beta.  In place of the token the oracle sees zeros, whose LN_1 is beta too; its output gradient is
    zero, so that the MLP half, where the two differ, adds nothing to any gradient."""
    import torch
    from paper_2409_06206_amd import runner
    B, H, W, window = 1, 8, 16, 8
    p = {k: synth.quantize(v, "bf16") for k, v in synth.astl_params(C, heads, 1, window, hidden, synth.LAYER_SEED0, "stress").items()}
    x, dy = (synth.quantize(a, "bf16") for a in synth.activations(B, H, W, C, synth.ACT_SEED))
    at = (0, 3, 5)
    rest = np.ones((B, H, W), dtype=bool)
    rest[at] = False
    x[at] = 1e20 * (1 - 2 * (np.arange(C) % 2))
    x, dy[at] = synth.quantize(x, "bf16"), 0.0
    blk = runner.DeviceBlock(B, H, W, C, heads, 1, window, 0, "bf16", hidden)
    blk.set_params(p)
    blk.set_inputs(x, dy)
    blk.forward()
    blk.backward()
    torch.cuda.synchronize()
    got = blk.results()
    plain = x.copy()
    plain[at] = 0.0
    kw = dict(heads=heads, groups=1, window=window, shift=0)
    want = {"y": astl_oracle.forward(plain, p, **kw)}
    dx, g = astl_oracle.backward(plain, dy, p, **kw)
    want.update({"dx": dx, **{"d" + k: v for k, v in g.items()}})
    assert (got["y"][at] == x[at]).all()  # (attention and MLP are far below the last bit)
    assert (got["dx"][at] == 0.0).all()
    for t in (got, want):
        t["y"], t["dx"] = t["y"][rest], t["dx"][rest]
    errs = {k: parity.rel_err(got[k], want[k]) for k in want}
    print(errs, flush=True)
    assert all(e <= parity.TOL["bf16"] for e in errs.values()), errs


def test_narrow_bf16_layers_take_the_fused_mlp_kernels():
    """The kernel timing aid names what ran: one fused launch per pass for the MLP half of a narrow
    bf16 layer, the per-step kernels otherwise (fp32, wide layers, forced)."""
    import torch
    case = dict(SMALL[7])
    print("case", case, flush=True)
    for flags, fused in ((0, True), (gswa.GSWA_FORCE_STAGED, False)):
        gswa.gswa_profile_enable(True)
        gswa.gswa_profile_collect()
        parity.check_block(astl_oracle, extra_flags=flags, **case)
        torch.cuda.synchronize()
        names, dropped = gswa.gswa_profile_collect()
        gswa.gswa_profile_enable(False)
        assert dropped == 0
        assert ("mlp_fwd" in names and "mlp_bwd" in names and "ln_fwd+mlp_reduce" in names) == fused, names
        assert ("fc1_linear" in names and "gelu_fwd" in names and "fc_wgrad" in names) == (not fused), names
        assert names["ln_fwd"][1] == (1 if fused else 4) and names["ln_bwd"][1] == (1 if fused else 2), names


@pytest.mark.parametrize("C,hidden", [(64, 120), (60, 128), (32, 64), (28, 60), (16, 24)])
def test_padding_edges_of_the_fused_mlp_tiles(C, hidden):
    """Channel and hidden widths at and next to the tile sizes of the fused MLP kernels."""
    heads = 4 if C % 4 == 0 else 2
    case = dict(B=2, H=8, W=8, C=C, heads=heads, groups=2, window=4, shift=2, dtype="bf16", hidden=hidden)
    print("case", case, flush=True)
    parity.check_block(astl_oracle, **case)


@pytest.mark.parametrize("case", [
    dict(B=1, H=4, W=4, C=256, heads=4, groups=2, window=4, shift=1, dtype="f32", hidden=16),
    dict(B=1, H=4, W=8, C=256, heads=8, groups=1, window=4, shift=0, dtype="bf16", hidden=24),
    dict(B=2, H=4, W=4, C=4, heads=2, groups=2, window=2, shift=1, dtype="bf16", hidden=4),
    dict(B=2, H=4, W=4, C=8, heads=2, groups=1, window=4, shift=2, dtype="f32", hidden=7),
    dict(B=1, H=8, W=8, C=20, heads=2, groups=2, window=4, shift=0, dtype="bf16", hidden=36),
    dict(B=1, H=5, W=5, C=68, heads=2, groups=1, window=5, shift=2, dtype="bf16", hidden=32),   # 25 rows: half a pair
    dict(B=1, H=7, W=21, C=132, heads=4, groups=1, window=7, shift=3, dtype="bf16", hidden=64), # 147
], ids=_id)
def test_extreme_widths(case):
    """The widest supported map (256 channels), the narrowest fused one, an odd hidden width."""
    print("case", case, flush=True)
    parity.check_block(astl_oracle, **case)


@pytest.mark.parametrize("C,hidden,tokens", [
    (180, 360, (1, 8, 12)),    # the benchmark's widths, 96 tokens: fewer tiles than waves of a workgroup
    (192, 384, (1, 8, 8)),     # every tile of both instantiation's largest shape full
    (132, 100, (2, 8, 12)),    # narrowest of the six-step kernel: two ragged channel steps; hidden not a multiple of 32
    (128, 256, (1, 12, 8)),    # widest of the four-step kernel, whole steps only
    (68, 32, (3, 4, 4)),       # narrowest wide layer, one stream unit, one of its three hidden steps in use
    (100, 196, (1, 20, 4)),    # the row's last four channels alone in a piece (C % 8 == 4), ragged hidden step
    (96, 384, (5, 4, 4)),
])
def test_shape_edges_of_the_streaming_mlp_forward_of_wide_layers(C, hidden, tokens):
    """Layers wider than 64 channels (up to 192, hidden up to 384) take the forward kernel that streams the
    MLP's weights through LDS: channel counts around its 32-channel steps, hidden widths around its 32-feature
    steps and 96-feature units, token counts that are not a multiple of the 16-token tiles."""
    import torch
    B, H, W = tokens
    case = dict(B=B, H=H, W=W, C=C, heads=4, groups=2, window=4, shift=1, dtype="bf16", hidden=hidden)
    print("case", case, flush=True)
    gswa.gswa_profile_enable(True)
    gswa.gswa_profile_collect()
    parity.check_block(astl_oracle, **case)
    torch.cuda.synchronize()
    names, dropped = gswa.gswa_profile_collect()
    gswa.gswa_profile_enable(False)
    assert dropped == 0
    assert "mlp_fwd" in names and "fc2_linear" not in names, names


def test_many_rounds_of_the_streaming_mlp_forward():
    """More 16-token tiles than the launch has waves (several rounds per wave, a ragged last round)."""
    case = dict(B=9, H=64, W=64, C=180, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=360)
    print("case", case, flush=True)
    parity.check_block(astl_oracle, backward=False, **case)


def test_ragged_token_count_in_the_fused_mlp_kernels():
    """Token counts that are not a multiple of the 16-token tiles or of the 128-token rounds."""
    for B, H, W in ((1, 4, 12), (3, 4, 4), (7, 8, 4)):
        case = dict(B=B, H=H, W=W, C=60, heads=6, groups=2, window=4, shift=1, dtype="bf16", hidden=120)
        print("case", case, flush=True)
        parity.check_block(astl_oracle, **case)


def test_graph_replays_of_a_layer_pair_match_the_eager_result():
    """A step of two chained whole layers captured into a HIP graph: every replay, with eager work
    and synchronisation in between, gives the eager outputs (the attention layer's fused path sums
    in a fixed order; the LayerNorm gradients go through atomics, hence a tolerance there)."""
    import torch
    from paper_2409_06206_amd import runner
    cfg = dict(B=2, H=16, W=16, C=60, heads=6, groups=2, window=8, dtype="bf16", hidden=120)
    x, dy = synth.activations(cfg["B"], cfg["H"], cfg["W"], cfg["C"], 1)
    blocks = []
    for li, shift in enumerate((0, 4)):
        blk = runner.DeviceBlock(cfg["B"], cfg["H"], cfg["W"], cfg["C"], cfg["heads"], cfg["groups"], cfg["window"],
                                 shift, cfg["dtype"], cfg["hidden"])
        blk.set_params(synth.astl_params(cfg["C"], cfg["heads"], cfg["groups"], cfg["window"], cfg["hidden"],
                                         200 + li, "stress"))
        blocks.append(blk)
    blocks[0].set_inputs(x)
    blocks[1].dy = runner.to_device(dy, cfg["dtype"])
    blocks[1].x, blocks[0].dy = blocks[0].y, blocks[1].dx

    def step():
        for b in blocks:
            b.forward()
        for b in reversed(blocks):
            b.backward()

    def snapshot():
        torch.cuda.synchronize()
        out = {}
        for i, b in enumerate(blocks):
            out.update({f"{i}.{k}": v.copy() for k, v in b.results().items()})
        return out

    print("eager step", flush=True)
    step()
    want = snapshot()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    print("capture", flush=True)
    with torch.cuda.graph(graph, stream=side):
        step()
    for rep in range(4):
        # eager work of the program's own between the replays: the outputs are overwritten
        for b in blocks:
            b.y.zero_()
            b.dx.zero_()
            for g in b.grads.values():
                g.fill_(7.0)
        torch.cuda.synchronize()
        print("replay", rep, flush=True)
        graph.replay()
        got = snapshot()
        for k, w in want.items():
            exact = k.endswith(".y") or k.endswith(".dx")
            if exact:
                assert np.array_equal(got[k], w), (rep, k)
            else:
                assert parity.rel_err(got[k], w) <= 1e-4, (rep, k, parity.rel_err(got[k], w))


STACKS = [
    dict(B=1, H=16, W=16, C=60, heads=6, groups=2, window=8, shift=4, dtype="f32", hidden=120, n_layers=3),
    dict(B=2, H=16, W=16, C=60, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=120, n_layers=5),
    dict(B=1, H=24, W=24, C=60, heads=4, groups=2, window=12, shift=6, dtype="bf16", hidden=120, n_layers=4, dqk=4),
    # wide layers: the streaming MLP kernels (the forward one hands LN_1 to the next layer), 4096 tokens
    dict(B=1, H=64, W=64, C=180, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=360, n_layers=3),
]


@pytest.mark.parametrize("every", [0, 1, 2, 3, 9])
@pytest.mark.parametrize("case", STACKS, ids=_id)
def test_stack_matches_oracle_with_and_without_checkpointing(case, every):
    """A sequence of layers with alternating shift; recomputed blocks give the same gradients."""
    import torch
    from paper_2409_06206_amd import runner
    c = dict(case)
    print("case", c, "checkpoint_every", every, flush=True)
    dtype, L, dqk = c["dtype"], c["n_layers"], c.get("dqk", 0)
    ps = [synth.astl_params(c["C"], c["heads"], c["groups"], c["window"], c["hidden"], 300 + l, "stress", dqk)
          for l in range(L)]
    ps = [{k: synth.quantize(v, dtype) for k, v in p.items()} for p in ps]
    x, dy = (synth.quantize(a, dtype) for a in synth.activations(c["B"], c["H"], c["W"], c["C"], 2))
    # a tensor handed from one layer to the next is a tensor of the layer's element type on both sides
    # ("bf16 activations with fp32 accumulation"); inside a layer the oracle stays in fp64
    kw = dict(heads=c["heads"], groups=c["groups"], window=c["window"], shift=c["shift"], dqk=dqk,
              store=None if dtype == "f32" else (lambda a: synth.quantize(a, dtype)))
    want = {"y": astl_oracle.stack_forward(x, ps, **kw)}
    dx, grads = astl_oracle.stack_backward(x, dy, ps, **kw)
    want["dx"] = dx
    for l, g in enumerate(grads):
        want.update({f"{l}.d{k}": v for k, v in g.items()})
    st = runner.DeviceStack(c["B"], c["H"], c["W"], c["C"], c["heads"], c["groups"], c["window"], c["shift"], dtype,
                            c["hidden"], L, every, dqk=dqk)
    st.set_params(ps)
    st.set_inputs(x, dy)
    st.forward()
    st.backward()
    torch.cuda.synchronize()
    got = st.results()
    tol = parity.TOL[dtype]
    errs = {k: parity.rel_err(got[k], w) for k, w in want.items()}
    bad = {k: e for k, e in errs.items() if not e <= tol}
    assert not bad, (bad, max(errs.values()))
    # inference call: same output, nothing saved
    y_train = st.y.clone()
    st.y.zero_()
    st.forward(keep=False)
    torch.cuda.synchronize()
    assert torch.equal(st.y, y_train)


TILED = [
    # (case, band sizes in window rows): bands that divide the map and bands that do not, one band per
    # image, one window row per band; shift 0 in every layer; odd shift; three images
    (dict(B=1, H=48, W=16, C=60, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=120, n_layers=4),
     (1, 2, 4, 5, 6, 9)),
    (dict(B=3, H=32, W=24, C=60, heads=6, groups=3, window=8, shift=3, dtype="bf16", hidden=120, n_layers=3),
     (1, 3)),
    (dict(B=2, H=40, W=16, C=180, heads=6, groups=2, window=8, shift=4, dtype="bf16", hidden=360, n_layers=3),
     (2, 3)),
    (dict(B=1, H=24, W=8, C=60, heads=6, groups=2, window=8, shift=0, dtype="bf16", hidden=120, n_layers=2),
     (1, 2)),
    (dict(B=2, H=20, W=12, C=12, heads=2, groups=1, window=4, shift=1, dtype="f32", hidden=20, n_layers=3),
     (1, 2, 4)),
    (dict(B=1, H=48, W=24, C=60, heads=4, groups=2, window=12, shift=6, dtype="bf16", hidden=120, n_layers=2,
          dqk=4), (1, 3)),
]


@pytest.mark.parametrize("case,bands", TILED, ids=lambda v: _id(v) if isinstance(v, dict) else str(v))
def test_band_by_band_inference_is_the_whole_map_inference(case, bands):
    """Bands of window rows through every layer: the oracle's output within tolerance, and the very bits of
    the call that takes each image as one band (a window's arithmetic does not depend on the band it is in)."""
    import torch
    from paper_2409_06206_amd import runner
    c = dict(case)
    print("case", c, flush=True)
    dtype, L, dqk = c["dtype"], c["n_layers"], c.get("dqk", 0)
    ps = [synth.astl_params(c["C"], c["heads"], c["groups"], c["window"], c["hidden"], 500 + l, "stress", dqk)
          for l in range(L)]
    ps = [{k: synth.quantize(v, dtype) for k, v in p.items()} for p in ps]
    x = synth.quantize(synth.activations(c["B"], c["H"], c["W"], c["C"], 1)[0], dtype)
    kw = dict(heads=c["heads"], groups=c["groups"], window=c["window"], shift=c["shift"], dqk=dqk,
              store=None if dtype == "f32" else (lambda a: synth.quantize(a, dtype)))
    want = astl_oracle.stack_forward(x, ps, **kw)
    st = runner.DeviceStack(c["B"], c["H"], c["W"], c["C"], c["heads"], c["groups"], c["window"], c["shift"], dtype,
                            c["hidden"], L, 0, dqk=dqk)
    st.set_params(ps)
    st.set_inputs(x)
    x_before = st.x.clone()
    # one band per image: every layer is one plain call of the whole-layer forward per image
    st.forward_tiled(c["H"])
    torch.cuda.synchronize()
    whole = st.y.clone()
    assert parity.rel_err(runner.to_host(whole), want) <= parity.TOL[dtype]
    for nb in bands:
        print("band_windows", nb, flush=True)
        st.y.fill_(float("nan"))
        st.forward_tiled(nb)
        torch.cuda.synchronize()
        assert torch.equal(st.y, whole), nb
        assert torch.equal(st.x, x_before)
    # the whole-map call hands LayerNorm_1 from layer to layer inside its MLP kernel where it can, which
    # sums a row in another order: equal up to the rounding of the stored activations
    st.forward(keep=False)
    torch.cuda.synchronize()
    assert parity.rel_err(runner.to_host(st.y), runner.to_host(whole)) <= (1e-6 if dtype == "f32" else 2e-2)


@pytest.mark.parametrize("groups,hidden,shift", [(1, 120, 4), (2, 128, 3), (3, 68, 4), (6, 120, 7)])
def test_narrow_layers_of_a_sequence_in_one_launch(groups, hidden, shift):
    """Narrow layers of a sequence: one launch a layer and one each for all weights of both halves; the same bits for an
    image alone, first of a batch, band by band (in place) and with the state kept."""
    import torch
    from paper_2409_06206_amd import runner
    B, H, W, L = 41, 40, 48, 3
    ps = [{k: synth.quantize(v, "bf16") for k, v in synth.astl_params(60, 6, groups, 8, hidden, 500 + l, "stress").items()}
          for l in range(L)]
    x, dy = (synth.quantize(a, "bf16") for a in synth.activations(B, H, W, 60, 1))

    def stack(n, every=0):
        st = runner.DeviceStack(n, H, W, 60, 6, groups, 8, shift, "bf16", hidden, L, every)
        st.set_params(ps)
        st.set_inputs(x[:n], dy[:n])
        return st
    one, many = stack(1), stack(B)
    with parity.launched() as names:
        one.forward(keep=False)
    assert names == {"pack_fwd", "mlp_pack", "layer_fwd"}, names
    alone = one.y.clone()
    kw = dict(heads=6, groups=groups, window=8, shift=shift, store=lambda a: synth.quantize(a, "bf16"))
    assert parity.rel_err(runner.to_host(alone), astl_oracle.stack_forward(x[:1], ps, **kw)) <= parity.TOL["bf16"]
    many.forward(keep=False)
    torch.cuda.synchronize()
    assert torch.equal(many.y[:1], alone)
    for nb in (1, 2, 5):
        one.y.fill_(float("nan"))
        one.forward_tiled(nb)
        torch.cuda.synchronize()
        assert torch.equal(one.y, alone), nb
    grads = []
    for every in (0, 2):
        st = stack(1, every)
        st.forward(keep=True)
        st.backward()
        torch.cuda.synchronize()
        assert torch.equal(st.y, alone)
        grads.append(st.dx.clone())
    assert torch.equal(*grads)


@pytest.mark.parametrize("groups", [1, 2, 3, 6])
def test_narrow_layers_of_a_sequence_in_several_rounds(groups):
    """More windows than the workgroups of the one-launch layer hold at once (four each, one workgroup per compute unit):
    every image of the batch, those of the second and third round among them, has the bits it has alone, in
    inference and with the state kept, and so has its gradient."""
    import torch
    from paper_2409_06206_amd import runner
    H, W, L, hidden = 40, 48, 3, 120
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    B = 8 * cus // 30 + 2  # images of 30 windows
    ps = [{k: synth.quantize(v, "bf16") for k, v in synth.astl_params(60, 6, groups, 8, hidden, 500 + l, "stress").items()}
          for l in range(L)]
    x, dy = (synth.quantize(a, "bf16") for a in synth.activations(B, H, W, 60, 1))

    def stack(n):
        st = runner.DeviceStack(n, H, W, 60, 6, groups, 8, 4, "bf16", hidden, L)
        st.set_params(ps)
        return st
    many, one = stack(B), stack(1)
    many.set_inputs(x, dy)
    many.forward(keep=False)
    y = many.y.clone()
    many.y.fill_(float("nan"))
    many.forward(keep=True)
    many.backward()
    torch.cuda.synchronize()
    for i in range(B):
        one.set_inputs(x[i:i + 1], dy[i:i + 1])
        one.forward(keep=True)
        one.backward()
        torch.cuda.synchronize()
        assert torch.equal(y[i], one.y[0]) and torch.equal(many.y[i], one.y[0]), i
        assert torch.equal(many.dx[i], one.dx[0]), i


@pytest.mark.parametrize("C,groups,window,images", [(180, 2, 8, 8), (180, 1, 16, 8), (60, 2, 8, 24)])
def test_band_by_band_inference_of_more_than_2_31_elements(C, groups, window, images):
    """Bands are small whatever the input: a batch of 2^31 elements and more gives every image the bits it has alone
    (the kernels that serve a whole map of that size are others, and read the weights repacked in another order)."""
    import torch
    from paper_2409_06206_amd import runner
    H, W, L = 1008, 1504, 2
    assert images * H * W * C >= 1 << 31
    print("case", C, groups, window, images, flush=True)
    ps = [{k: synth.quantize(v, "bf16") for k, v in synth.astl_params(C, 6, groups, window, 2 * C, 500 + l, "stress").items()}
          for l in range(L)]
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(1)
    x = torch.randn((images, H, W, C), generator=gen, device="cuda:0", dtype=torch.bfloat16)

    def stack(n):
        st = runner.DeviceStack(n, H, W, C, 6, groups, window, window // 2, "bf16", 2 * C, L, band_windows=16, inference_only=True)
        st.set_params(ps)
        st.ws.fill_(255)  # (NaN where nothing is written)
        return st
    many, one = stack(images), stack(1)
    many.x = x
    many.forward(keep=False)
    for i in range(images):
        one.x = x[i:i + 1]
        one.forward(keep=False)
        torch.cuda.synchronize()
        finite, same = bool(torch.isfinite(one.y).all()), torch.equal(many.y[i], one.y[0])
        assert finite and same, i


@pytest.mark.parametrize("C,W", [(180, 93200), (60, 279616)])
def test_bands_on_both_sides_of_2_31_elements(C, W):
    """Bands of 16 window rows just below 2^31 elements and, in the shifted layer, of 17 rows above: other kernels
    serve them, and neither kind's scratch may lie over the weights the other repacked.  Against bands of four
    rows, at the tolerance of two organisations of the same layers."""
    import torch
    from paper_2409_06206_amd import runner
    H, L = 264, 3
    assert 16 * 8 * W * C < 1 << 31 <= 17 * 8 * W * C
    print("case", C, W, flush=True)
    ps = [{k: synth.quantize(v, "bf16") for k, v in synth.astl_params(C, 6, 2, 8, 2 * C, 500 + l, "stress").items()}
          for l in range(L)]
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(1)
    st = runner.DeviceStack(1, H, W, C, 6, 2, 8, 4, "bf16", 2 * C, L, band_windows=16, inference_only=True)
    st.set_params(ps)
    st.x = torch.randn((1, H, W, C), generator=gen, device="cuda:0", dtype=torch.bfloat16)
    st.ws.fill_(255)  # (NaN where nothing is written)
    st.forward(keep=False)
    got = st.y.clone()
    st.forward_tiled(4)
    torch.cuda.synchronize()
    for r in range(0, H, 8):
        a, b = got[0, r:r + 8].float(), st.y[0, r:r + 8].float()
        err = float((a - b).abs().max() / b.abs().max())
        assert err <= 2e-2, (r, err)


@pytest.mark.parametrize("groups,window,shift", [(1, 8, 4), (2, 8, 3), (3, 16, 8)])
def test_wide_layers_take_ln1_in_the_attention_kernel(groups, window, shift):
    """Wide layers with the streaming MLP kernels: no launch of LN_1, so that a sequence gives the bits of the banded
    call and of single layer calls, kept state or not."""
    import torch
    from paper_2409_06206_amd import runner
    B, H, W, L, hidden = 2, 3 * window, 5 * window, 3, 360
    ps = [{k: synth.quantize(v, "bf16") for k, v in synth.astl_params(180, 6, groups, window, hidden, 500 + l, "stress").items()}
          for l in range(L)]
    x, dy = (synth.quantize(a, "bf16") for a in synth.activations(B, H, W, 180, 1))
    st = runner.DeviceStack(B, H, W, 180, 6, groups, window, shift, "bf16", hidden, L, 0)
    st.set_params(ps)
    st.set_inputs(x)
    with parity.launched() as names:
        st.forward(keep=False)
    assert "mlp_fwd" in names and "ln_fwd" not in names, names
    whole = st.y.clone()
    for run in (lambda: st.forward_tiled(1), lambda: st.forward(keep=True)):
        st.y.fill_(float("nan"))
        run()
        torch.cuda.synchronize()
        assert torch.equal(st.y, whole)
    kw = dict(heads=6, groups=groups, window=window, shift=shift, store=lambda a: synth.quantize(a, "bf16"))
    assert parity.rel_err(runner.to_host(whole), astl_oracle.stack_forward(x, ps, **kw)) <= parity.TOL["bf16"]


def test_inference_sequence_at_the_benchmark_size():
    """astl_infer_stack6 as bench.py runs it (six whole layers, one 512x512 map, C = 180, hidden 360, in one
    call): every output element against the oracle's loop over the layers, and the band-by-band form on the
    same map against both."""
    import torch
    from paper_2409_06206_amd import runner
    cfg = synth.CONFIGS["astl_infer_stack6"]
    L, groups, dtype = cfg["stack"], cfg["groups"][0], cfg["dtype"]
    print("case", cfg, flush=True)
    ps = [synth.astl_params(cfg["C"], cfg["heads"], groups, cfg["window"], cfg["hidden"], 700 + l, "stress")
          for l in range(L)]
    ps = [{k: synth.quantize(v, dtype) for k, v in p.items()} for p in ps]
    x, _ = synth.activations(cfg["B"], cfg["H"], cfg["W"], cfg["C"], synth.ACT_SEED + 9)
    x = synth.quantize(x, dtype)
    want = astl_oracle.stack_forward(x, ps, heads=cfg["heads"], groups=groups, window=cfg["window"],
                                     shift=cfg["stack_shift"], store=lambda a: synth.quantize(a, dtype))
    st = runner.DeviceStack(cfg["B"], cfg["H"], cfg["W"], cfg["C"], cfg["heads"], groups, cfg["window"],
                            cfg["stack_shift"], dtype, cfg["hidden"], L, 0, inference_only=True)
    st.set_params(ps)
    st.set_inputs(x)
    st.forward(keep=False)
    torch.cuda.synchronize()
    whole = runner.to_host(st.y)
    assert parity.rel_err(whole, want) <= parity.TOL[dtype]
    st.y.fill_(float("nan"))
    st.forward_tiled(16)
    torch.cuda.synchronize()
    banded = runner.to_host(st.y)
    assert parity.rel_err(banded, want) <= parity.TOL[dtype]
    assert parity.rel_err(banded, whole) <= parity.TOL[dtype]


def _random_layers(n, seed):
    """Seeded random whole-layer shapes that satisfy the divisibility rules: any window, head count,
    head width, hidden width, narrow or plain queries and keys."""
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        M = int(rng.choice([2, 3, 4, 5, 6, 8]))
        heads = int(rng.choice([1, 2, 3, 4, 6]))
        groups = int(rng.choice([g for g in (1, 2, 3, 4, 6) if heads % g == 0]))
        d = int(rng.integers(1, 11))
        if heads * d > 256:
            continue
        B, nh, nw = int(rng.integers(1, 3)), int(rng.integers(1, 4)), int(rng.integers(1, 4))
        case = dict(B=B, H=nh * M, W=nw * M, C=heads * d, heads=heads, groups=groups, window=M,
                    shift=int(rng.integers(0, M)), hidden=int(rng.integers(1, 140)),
                    dqk=int(rng.choice([0, 0, 1, 3, 4])))
        # A LayerNorm over very few channels is ill-conditioned with a tiny eps: 1/sqrt(var + eps)
        # reaches eps^-1/2 = 316 when a token's channels nearly coincide, and every rounding of the
        # normalised value is amplified by that factor in both arithmetics.  Such layers get an eps
        # that conditions them (eps is a parameter of the layer): 1/sqrt(var + eps) <= 10.
        if heads * d < 6:
            case["eps"] = 1e-2
        out.append(case)
    return out


@pytest.mark.parametrize("case", _random_layers(14, 31), ids=_id)
def test_random_layers_fp32(case):
    print("case", case, flush=True)
    parity.check_block(astl_oracle, dtype="f32", **case)


@pytest.mark.parametrize("case", _random_layers(10, 32), ids=_id)
def test_random_layers_bf16(case):
    print("case", case, flush=True)
    parity.check_block(astl_oracle, dtype="bf16", **case)


@pytest.mark.parametrize("groups,shape,shift,cascade", [
    (1, (1, 24, 16), 0, True), (2, (4, 64, 72), 4, True), (3, (2, 8, 24), 5, True), (6, (1, 16, 8), 3, True),
    (3, (1, 16, 16), 4, False),
])
def test_fp32_whole_layers_one_workgroup_per_window(groups, shape, shift, cascade):
    """A whole fp32 layer of 60 channels, hidden 120, is one launch per direction: every group count, with and without
    the cascade, more windows (288) than vectors of parameter gradients (256)."""
    B, H, W = shape
    case = dict(B=B, H=H, W=W, C=60, heads=6, groups=groups, window=8, shift=shift, dtype="f32", hidden=120)
    print("case", case, flush=True)
    with parity.launched() as names:
        parity.check_block(astl_oracle, cascade=cascade, **case)
    assert names == {"layer_fwd", "layer_bwd", "reduce_partials"}


@pytest.mark.parametrize("heads,groups,dqk,shape,shift", [
    (4, 1, 4, (1, 24, 36), 6), (4, 4, 4, (2, 12, 24), 5), (4, 1, 8, (1, 36, 12), 6), (4, 2, 8, (1, 24, 24), 0),
    (4, 4, 8, (1, 12, 12), 7), (6, 1, 4, (1, 24, 24), 6), (6, 2, 4, (1, 24, 12), 3), (6, 3, 4, (17, 48, 48), 6),
    (6, 6, 4, (1, 24, 24), 6),
])
def test_12x12_window_layers_one_workgroup_per_window(heads, groups, dqk, shape, shift):
    """Whole bf16 layers with 12x12 windows and narrow q / k are one launch per direction: every organisation of the
    heads, one window, windows cut by the shift in both directions, more windows (272) than vectors of parameter
    gradients (256)."""
    B, H, W = shape
    case = dict(B=B, H=H, W=W, C=60, heads=heads, groups=groups, window=12, shift=shift, dtype="bf16", hidden=120, dqk=dqk)
    print("case", case, flush=True)
    with parity.launched() as names:
        parity.check_block(astl_oracle, **case)
    assert names == {"layer_fwd", "layer_bwd", "reduce_partials"}


@pytest.mark.parametrize("case,copies", [
    (dict(H=16, W=24, heads=6, groups=1, window=8, shift=4, dtype="bf16"), 90),
    (dict(H=16, W=24, heads=6, groups=2, window=8, shift=3, dtype="bf16"), 90),
    (dict(H=24, W=16, heads=6, groups=3, window=8, shift=4, dtype="bf16"), 90),
    (dict(H=24, W=36, heads=4, groups=2, window=12, shift=6, dtype="bf16", dqk=4), 90),
    (dict(H=24, W=16, heads=6, groups=2, window=8, shift=4, dtype="f32"), 90),
], ids=lambda v: _id(v) if isinstance(v, dict) else str(v))
def test_an_image_gives_the_same_bits_alone_and_in_a_batch(case, copies):
    """Every (image, window) is computed on its own, by kernels that are chosen without a look at the number of
    images: the output and the input gradient of an image through a sequence of layers have the same bits whether the
    call holds that image alone (6 windows) or with 89 others (540)."""
    import torch
    from paper_2409_06206_amd import runner
    c = dict(C=60, hidden=120, n_layers=2, **case)
    print("case", c, flush=True)
    ps = [synth.astl_params(60, c["heads"], c["groups"], c["window"], 120, 300 + l, "stress", c.get("dqk", 0)) for l in range(2)]
    ps = [{k: synth.quantize(v, c["dtype"]) for k, v in p.items()} for p in ps]
    x, dy = synth.activations(copies, c["H"], c["W"], 60, 2)
    got = []
    for B in (1, copies):
        st = runner.DeviceStack(B, checkpoint_every=1, **c)
        st.set_params(ps)
        st.set_inputs(x[:B], dy[:B])
        st.forward(keep=False)
        torch.cuda.synchronize()
        y = st.y[:1].clone()
        st.forward()
        st.backward()
        torch.cuda.synchronize()
        got.append((y, st.y[:1].clone(), st.dx[:1].clone()))
    for name, alone, batch in zip(("inference y", "y", "dx"), *got):
        assert torch.equal(alone, batch), name


def test_gradient_at_the_second_layer_norm_stays_in_fp32():
    """A whole layer with 12x12 windows whose numbers up to d LN_2 are all exact: dy = 1, GELU' = 1 (b_fc1 = 16), and W1, W2
    so that every entry of the gradient at LN_2's output is 1 + 15/4096, which bf16 rounds to 1.  Its sum over the
    tokens is d ln2_b: fp32 keeps it to 208 additions of 2^-24 (1.3e-5) and GELU' in fp32, one rounding to bf16 costs
    3.7e-3."""
    from paper_2409_06206_amd import runner
    import torch
    C, hidden = 60, 120
    p = synth.astl_params(C, 4, 2, 12, hidden, 300, "stress", 4)
    eye = np.eye(C, dtype=np.float32)
    p["w_fc1"] = np.concatenate([eye, eye * (15.0 / 4096.0)])
    p["w_fc2"] = np.concatenate([eye, eye], axis=1)
    p["b_fc1"] = np.full(hidden, 16.0, dtype=np.float32)
    p["ln2_w"], p["ln2_b"] = np.ones(C, dtype=np.float32), np.zeros(C, dtype=np.float32)
    p = {k: synth.quantize(v, "bf16") for k, v in p.items()}
    blk = runner.DeviceBlock(1, 12, 12, C, 4, 2, 12, 6, "bf16", hidden, dqk=4)
    blk.set_params(p)
    x, _ = synth.activations(1, 12, 12, C, 3)
    blk.set_inputs(synth.quantize(x, "bf16"), np.ones((1, 12, 12, C), dtype=np.float32))
    print("forward, backward", flush=True)
    blk.forward()
    blk.backward()
    torch.cuda.synchronize()
    want = np.full(C, 144.0 * (1.0 + 15.0 / 4096.0))
    assert parity.rel_err(blk.results()["dln2_b"], want) <= 2e-5


def test_fp32_channel_means_are_rounded_once():
    """A whole fp32 layer on a map of 959 and 961: every token's mean is 960 and its variance 1, both exact, as long as the
    sum is divided by 60 and not multiplied by the rounded 1/60 (5.2e-8 too much: 960.00006).  d ln1_w, the sum over the
    tokens of a gradient times the normalised map, would be off by 6e-5."""
    from paper_2409_06206_amd import runner
    import torch
    C = 60
    p = synth.astl_params(C, 6, 2, 8, 120, 300, "stress")
    p["ln1_w"], p["ln1_b"] = np.ones(C, dtype=np.float32), np.zeros(C, dtype=np.float32)
    p["w_fc2"][:] = 0.0   # (nothing comes back through LN_2, whose input near 960 has an fp32 rounding of its own)
    x = np.broadcast_to(np.where(np.arange(C) % 2 == 0, 961.0, 959.0), (1, 16, 16, C)).astype(np.float32)
    _, dy = synth.activations(1, 16, 16, C, 3)
    blk = runner.DeviceBlock(1, 16, 16, C, 6, 2, 8, 4, "f32", 120)
    blk.set_params(p)
    blk.set_inputs(x, dy)
    blk.forward()
    blk.backward()
    torch.cuda.synchronize()
    _, grads = astl_oracle.backward(x, dy, p, heads=6, groups=2, window=8, shift=4)
    assert parity.rel_err(blk.results()["dln1_w"], grads["ln1_w"]) <= parity.TOL["f32"]
