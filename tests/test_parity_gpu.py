"""GPU parity: the HIP library against the CPU oracle, element by element, through the C ABI."""
import numpy as np
import pytest

from paper_2409_06206_amd import synth
from tests import parity

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)


# B, H, W, C, heads, groups, window, shift, dtype, regime
SMALL = [
    (1, 16, 16, 60, 6, 2, 8, 4, "f32", "init"),      # the fp32 parity configuration
    (1, 16, 16, 60, 6, 2, 8, 4, "f32", "stress"),
    (2, 16, 24, 60, 6, 1, 8, 0, "f32", "stress"),
    (2, 24, 16, 60, 6, 3, 8, 3, "f32", "stress"),
    (1, 16, 16, 60, 6, 6, 8, 7, "f32", "stress"),
    (3, 8, 16, 12, 6, 2, 4, 1, "f32", "stress"),     # ragged: 12 channels, 16-token windows
    (1, 8, 8, 6, 3, 3, 8, 5, "f32", "stress"),       # one window per image
    (1, 7, 14, 6, 2, 1, 7, 3, "f32", "stress"),      # odd window side
    (1, 16, 16, 180, 6, 1, 8, 4, "f32", "stress"),
    (1, 16, 16, 180, 6, 3, 8, 4, "f32", "stress"),
    (1, 32, 32, 180, 6, 2, 16, 8, "f32", "stress"),  # 256-token windows
    (2, 16, 16, 60, 6, 1, 8, 0, "bf16", "init"),
    (2, 16, 16, 60, 6, 2, 8, 4, "bf16", "init"),
    (2, 16, 16, 60, 6, 2, 8, 4, "bf16", "stress"),
    (2, 24, 16, 60, 6, 3, 8, 4, "bf16", "stress"),
    (1, 16, 16, 60, 6, 6, 8, 4, "bf16", "stress"),
    (1, 16, 24, 180, 6, 1, 8, 4, "bf16", "stress"),
    (1, 16, 16, 180, 6, 2, 8, 0, "bf16", "stress"),
    (1, 16, 16, 180, 6, 3, 8, 4, "bf16", "init"),
    (1, 32, 32, 180, 6, 2, 16, 8, "bf16", "stress"),
]


@pytest.mark.parametrize("B,H,W,C,heads,groups,window,shift,dtype,regime", SMALL)
def test_small_shapes_forward_backward(oracle, B, H, W, C, heads, groups, window, shift, dtype, regime):
    _say("case", B, H, W, C, heads, groups, window, shift, dtype, regime)
    errs, _ = parity.check_case(oracle, B, H, W, C, heads, groups, window, shift, dtype,
                                seed=synth.LAYER_SEED0 + 3, regime=regime)
    _say("  errors", {k: f"{v:.2e}" for k, v in errs.items()})


@pytest.mark.parametrize("groups,shift", [(1, 0), (2, 4), (3, 5), (6, 4)])
def test_forced_staged_path_bf16(oracle, groups, shift):
    """The one-kernel-per-step path stays correct where a fused kernel would normally run."""
    from paper_2409_06206_amd import gswa
    parity.check_case(oracle, 2, 16, 24, 60, 6, groups, 8, shift, "bf16", regime="stress",
                      extra_flags=gswa.GSWA_FORCE_STAGED)


def test_forced_staged_path_wide_layer(oracle):
    from paper_2409_06206_amd import gswa
    parity.check_case(oracle, 1, 16, 24, 180, 6, 3, 8, 4, "bf16", regime="stress",
                      extra_flags=gswa.GSWA_FORCE_STAGED)


@pytest.mark.parametrize("C,heads", [(96, 6), (140, 5), (180, 6), (192, 6)])
def test_forced_staged_path_one_group_many_tokens(oracle, C, heads):
    """One group and at least 4096 tokens: the backward recomputes q|k|v (3C output columns: two or three column
    blocks of the kernel that streams the weights through LDS, the last one ragged or full) and, from 132 channels
    on, takes the input gradient on the same kernel."""
    from paper_2409_06206_amd import gswa
    parity.check_case(oracle, 1, 64, 72, C, heads, 1, 8, 4, "bf16", regime="stress",
                      extra_flags=gswa.GSWA_FORCE_STAGED)


@pytest.mark.parametrize("groups,rows,cols,launches", [(2, 8, 113, 3), (2, 5, 181, 2), (3, 23, 59, 4), (3, 14, 97, 3)])
def test_last_sums_of_a_wide_backward_in_two_launches_and_in_one(oracle, groups, rows, cols, launches):
    """180 channels: with 904 windows and two groups, 1357 and three, the projection's partial vectors (256 compute units) do
    not fit the part of the scratch that is free by then; with 905 and 1358 they just do, while the other sums still have
    to be taken (with three groups the vectors of q|k|v are summed one entry a load, the projection's four); here all are added."""
    from paper_2409_06206_amd import gswa, runner
    H, W = 8 * rows, 8 * cols
    x, dy, p = parity.make_inputs(1, H, W, 180, 6, groups, 8, "bf16", synth.LAYER_SEED0 + 3, "stress")
    layer = runner.DeviceLayer(1, H, W, 180, 6, groups, 8, 4, "bf16", gswa.GSWA_ACCUM_WGRAD)
    layer.set_params(p)
    layer.set_inputs(x, dy)
    for g in layer.grads.values():
        g.fill_(0.5)
    layer.forward()
    with parity.launch_counts() as counts:
        layer.backward()
    assert counts["reduce_partials"] == launches, counts
    got = layer.results()
    want = parity.oracle_results(oracle, x, dy, p, 6, groups, 8, 4)
    for k in parity.GRAD_NAMES:
        assert parity.rel_err(got[k] - (0.5 if k != "dx" else 0.0), want[k]) <= parity.TOL["bf16"], k


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("B,H,W,window,direct", [(1, 64, 120, 8, False), (1, 88, 88, 8, True), (3, 56, 72, 8, True),
                                                 (1, 12, 636, 12, False), (1, 72, 108, 12, True), (2, 72, 72, 12, True)])
def test_one_group_of_a_wide_layer_sums_its_gradients_directly(oracle, B, H, W, window, direct, accumulate):
    """180 channels, one group.  From 7723 tokens on the scratch (q|k|v of all tokens) holds 16 partial vectors of both weight
    gradients: one launch sums them and the windows' bias-table gradients, written or added, and nothing is cleared; below,
    two sums add onto cleared copies that a third collects.  7680 and 7744 tokens in 8x8 windows, 7632 and 7776 in 12x12
    ones, and more; 7744 and 12096 are no whole number of passes of 128.  Twice the same call: the same bits."""
    from paper_2409_06206_amd import gswa, runner
    x, dy, p = parity.make_inputs(B, H, W, 180, 6, 1, window, "bf16", synth.LAYER_SEED0 + 2, "stress")
    layer = runner.DeviceLayer(B, H, W, 180, 6, 1, window, 4, "bf16", gswa.GSWA_ACCUM_WGRAD if accumulate else 0)
    layer.set_params(p)
    layer.set_inputs(x, dy)
    start = 0.5 if accumulate else 0.0
    layer.forward()
    runs = []
    for _ in range(2):
        for g in layer.grads.values():
            g.fill_(0.5)
        with parity.launch_counts() as counts:
            layer.backward()
        assert (counts.get("fill_zero", 0), counts["reduce_partials"]) == ((0, 1) if direct else (1, 3)), counts
        runs.append({k: v.copy() for k, v in layer.results().items()})
    want = parity.oracle_results(oracle, x, dy, p, 6, 1, window, 4)
    for k in parity.GRAD_NAMES:
        assert (runs[0][k] == runs[1][k]).all(), k
        got = runs[0][k] - (start if k != "dx" else 0.0)
        assert parity.rel_err(got, want[k]) <= parity.TOL["bf16"], k


@pytest.mark.parametrize("groups", [2, 3])
def test_no_cascade_flag_wide_layer(oracle, groups):
    """Wide fused path (C=180) with Eq. 8 switched off: no cascade input, no cascade gradient."""
    parity.check_case(oracle, 1, 16, 16, 180, 6, groups, 8, 4, "bf16", regime="stress", cascade=False)


@pytest.mark.parametrize("groups", [2, 3])
def test_accumulate_flag_on_wide_fused_path(oracle, groups):
    """Every partial-sum launch of the wide backward (per group, table, projection) adds into its output."""
    import torch
    from paper_2409_06206_amd import gswa, runner
    x, dy, p = parity.make_inputs(2, 16, 24, 180, 6, groups, 8, "bf16", synth.LAYER_SEED0 + 1, "stress")
    layer = runner.DeviceLayer(2, 16, 24, 180, 6, groups, 8, 4, "bf16", gswa.GSWA_ACCUM_WGRAD)
    layer.set_params(p)
    layer.set_inputs(x, dy)
    for g in layer.grads.values():
        g.fill_(0.5)
    layer.forward()
    layer.backward()
    layer.backward()
    torch.cuda.synchronize()
    got = layer.results()
    want = parity.oracle_results(oracle, x, dy, p, 6, groups, 8, 4)
    for k in parity.GRAD_NAMES[1:]:
        assert parity.rel_err(got[k] - 0.5, 2.0 * want[k]) <= parity.TOL["bf16"], k


@pytest.mark.parametrize("C,heads,dqk,window", [
    (180, 6, 0, 8),   # 30 channels: the last four of a head's two tiles half full
    (36, 2, 0, 8),    # 18: one pair behind a whole tile
    (64, 2, 0, 8),    # 32: no remainder
    (34, 2, 0, 8),    # 17: heads that begin between two dwords
    (60, 2, 18, 12),  # 30 and 18, 12x12 windows
    (60, 2, 5, 8),    # 30, and five channels of q and k
])
def test_attention_adjoint_by_pairs_of_channels(oracle, C, heads, dqk, window):
    """The attention adjoint of the one-kernel-per-step path takes the channels of a head in pairs where heads and rows
    begin on a dword, one by one where they do not."""
    from paper_2409_06206_amd import gswa
    print("case", C, heads, dqk, window, flush=True)
    parity.check_case(oracle, 2, 2 * window, 3 * window, C, heads, 1, window, 3, "bf16", regime="stress", dqk=dqk,
                      extra_flags=gswa.GSWA_FORCE_STAGED)


@pytest.mark.parametrize("groups", [1, 2, 3])
@pytest.mark.parametrize("B,H,W,window,shift", [
    (1, 8, 8, 8, 4),         # one window: three of four window slots of the workgroup empty
    (3, 24, 328, 8, 3),      # 369 windows, odd shift: the second slot partly filled
    (1, 328, 216, 8, 0),     # 1107 windows: a second round of a few slots
    (1, 16, 16, 16, 8),
    (1, 304, 224, 16, 5),    # 266 windows: a second round of a few workgroups
])
def test_wide_forward_in_one_launch(oracle, B, H, W, window, shift, groups):
    """The forward of a wide layer: one launch besides the packing for both window sizes; training and inference
    give the same bits."""
    x, dy, p = parity.make_inputs(B, H, W, 180, 6, groups, window, "bf16", synth.LAYER_SEED0 + 3, "stress")
    want = parity.oracle_results(oracle, x, dy, p, 6, groups, window, shift, backward=False)["y"]
    with parity.launched() as names:
        got, _ = parity.gpu_results(x, dy, p, 6, groups, window, shift, "bf16", backward=False)
    assert names == {"pack_fwd", "fused_fwd"}
    assert parity.rel_err(got["y"], want) <= parity.TOL["bf16"]
    assert all(e <= parity.TOL["bf16"] for e in parity.border_errs({"y": got["y"]}, {"y": want}, window, shift).values())
    from paper_2409_06206_amd import runner
    import torch
    layer = runner.DeviceLayer(B, H, W, 180, 6, groups, window, shift, "bf16")
    layer.set_params(p)
    layer.set_inputs(x, dy)
    layer.forward(keep=True)
    torch.cuda.synchronize()
    assert np.array_equal(layer.results()["y"], got["y"])


@pytest.mark.parametrize("groups", [1, 2, 3])
def test_wide_forward_gives_an_image_the_same_bits_alone_and_in_a_batch(groups):
    """Up to two windows a compute unit four waves take a window, beyond two."""
    import torch
    from paper_2409_06206_amd import runner
    x, dy, p = parity.make_inputs(18, 40, 48, 180, 6, groups, 8, "bf16", synth.LAYER_SEED0 + 6, "stress")  # 540 windows
    y = []
    for n in (18, 1):
        layer = runner.DeviceLayer(n, 40, 48, 180, 6, groups, 8, 4, "bf16")
        layer.set_params(p)
        layer.set_inputs(x[:n], dy[:n])
        layer.forward(keep=False)
        torch.cuda.synchronize()
        y.append(layer.results()["y"][:1])
    assert np.array_equal(*y)


@pytest.mark.parametrize("groups", [1, 2, 3])
@pytest.mark.parametrize("window,shift", [(8, 4), (8, 0), (16, 8), (16, 3)])
def test_wide_forward_of_2_31_elements_and_more(window, shift, groups):
    """The one-launch forward of wide layers addresses fewer than 2^31 elements; larger inputs take one launch per head
    chunk and one of the projection.  Every image against itself alone, which the one-launch kernel computes, at the
    tolerance of two organisations of the same layer; with and without the group outputs kept."""
    import torch
    from paper_2409_06206_amd import gswa, runner
    B, H, W, C = 8, 1008, 1504, 180
    assert (B - 1) * H * W * C < 1 << 31 <= B * H * W * C
    print("case", window, shift, groups, flush=True)
    _, _, p = parity.make_inputs(1, window, window, C, 6, groups, window, "bf16", synth.LAYER_SEED0 + 7, "stress")
    one = runner.DeviceLayer(1, H, W, C, 6, groups, window, shift, "bf16")
    one.set_params(p)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(1)
    x = torch.randn((B, H, W, C), generator=gen, device="cuda:0", dtype=torch.bfloat16)
    desc = gswa.make_desc(B, H, W, C, 6, groups, window, shift, "bf16")
    saved_bytes, fwd_bytes, _ = gswa.gswa_query_bytes(desc)
    ws = torch.full((fwd_bytes + saved_bytes,), 255, dtype=torch.uint8, device="cuda:0")  # (NaN where nothing is written)
    args = [one.params[k] for k in ("w_qkv", "b_qkv", "w_proj", "b_proj", "table")]
    y = []
    for saved in (None, torch.empty(saved_bytes, dtype=torch.uint8, device="cuda:0")):
        y.append(torch.full_like(x, float("nan")))
        with parity.launched() as names:
            gswa.gswa_forward(desc, x, *args, y[-1], saved, ws)
        assert names == {"pack_fwd", "fused_attn_fwd", "proj_gemm"}
    assert torch.equal(*y)
    for i in range(B):
        one.x = x[i:i + 1]
        with parity.launched() as names:
            one.forward(keep=False)
        assert names == {"pack_fwd", "fused_fwd"}
        want, top = one.y[0], float(one.y.abs().max())
        for r in range(0, H, 16):
            err = float((y[0][i, r:r + 16].float() - want[r:r + 16].float()).abs().max()) / top
            assert err <= parity.TOL["bf16"], (i, r, err)


@pytest.mark.parametrize("shift", [4, 3])
def test_wide_backward_of_2_31_elements_and_more(shift):
    """Two groups: one kernel takes the backward of inputs of any size.  Every image's input gradient against the image alone,
    and the parameter gradients against the sum over the images, at the tolerance of two organisations of the same layer (the
    forward of such inputs is another one, so the group outputs that both passes of the backward start from are rounded
    differently)."""
    import torch
    from paper_2409_06206_amd import gswa, runner
    B, H, W, C = 8, 1008, 1504, 180
    assert (B - 1) * H * W * C < 1 << 31 <= B * H * W * C
    _say("case", shift)
    _, _, p = parity.make_inputs(1, 8, 8, C, 6, 2, 8, "bf16", synth.LAYER_SEED0 + 7, "stress")
    one = runner.DeviceLayer(1, H, W, C, 6, 2, 8, shift, "bf16", gswa.GSWA_ACCUM_WGRAD)
    one.set_params(p)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(2)
    x, dy = (torch.randn((B, H, W, C), generator=gen, device="cuda:0", dtype=torch.bfloat16) for _ in range(2))
    desc = gswa.make_desc(B, H, W, C, 6, 2, 8, shift, "bf16")
    saved_bytes, fwd_bytes, bwd_bytes = gswa.gswa_query_bytes(desc)
    ws = torch.full((max(fwd_bytes, bwd_bytes),), 255, dtype=torch.uint8, device="cuda:0")  # (NaN where nothing is written)
    saved = torch.full((saved_bytes,), 255, dtype=torch.uint8, device="cuda:0")
    y, dx = torch.empty_like(x), torch.full_like(x, float("nan"))
    names = ("w_qkv", "b_qkv", "w_proj", "b_proj", "table")
    args = [one.params[k] for k in names]
    grads = [torch.full_like(one.grads[k], float("nan")) for k in names]
    gswa.gswa_forward(desc, x, *args, y, saved, ws)
    with parity.launch_counts() as counts:
        gswa.gswa_backward(desc, x, dy, *args, saved, dx, *grads, ws)
    assert counts["wide_attn_bwd"] == 2 and "fused_bwd" not in counts, counts
    for g in one.grads.values():
        g.zero_()
    for i in range(B):
        one.x, one.dy = x[i:i + 1], dy[i:i + 1]
        one.forward()
        one.backward()
        top = float(one.dx.abs().max())
        for r in range(0, H, 16):
            err = float((dx[i, r:r + 16].float() - one.dx[0, r:r + 16].float()).abs().max()) / top
            assert err <= parity.TOL["bf16"], (i, r, err)
    for k, g in zip(names, grads):
        assert parity.rel_err(runner.to_host(g), runner.to_host(one.grads[k])) <= parity.TOL["bf16"], k


@pytest.mark.parametrize("groups", [1, 2, 3, 6])
@pytest.mark.parametrize("shift", [0, 3])
def test_narrow_forward_in_four_waves_and_in_one(oracle, groups, shift):
    """Up to four windows a compute unit a window is taken by four waves that exchange K and V, beyond by one: the
    same bits (and the kept group outputs: the gradients of the same rows agree with the oracle in both)."""
    import torch
    from paper_2409_06206_amd import runner
    x, dy, p = parity.make_inputs(41, 40, 48, 60, 6, groups, 8, "bf16", synth.LAYER_SEED0 + 5, "stress")  # 1230 windows

    def run(n, keep):
        layer = runner.DeviceLayer(n, 40, 48, 60, 6, groups, 8, shift, "bf16")
        layer.set_params(p)
        layer.set_inputs(x[:n], dy[:n])
        layer.forward(keep=keep)
        if keep:
            layer.backward()
        torch.cuda.synchronize()
        return layer.results()
    whole, alone, kept = run(41, True), run(1, False), run(1, True)
    assert np.array_equal(whole["y"][:1], alone["y"]) and np.array_equal(alone["y"], kept["y"])
    assert np.array_equal(whole["dx"][:1], kept["dx"])
    want = parity.oracle_results(oracle, x[:1], dy[:1], p, 6, groups, 8, shift)
    for k, w in want.items():
        assert parity.rel_err(kept[k], w) <= parity.TOL["bf16"], k


@pytest.mark.parametrize("groups", [2, 6])
def test_kernel_timing_aid_reports_the_launched_kernels(groups):
    """gswa_profile_*: per-kernel HIP-event totals for one forward + backward, the launches of a kernel added up (the backward
    of six groups is two launches with a sum behind each)."""
    import torch
    from paper_2409_06206_amd import gswa, runner
    x, dy, p = parity.make_inputs(2, 16, 16, 60, 6, groups, 8, "bf16", synth.LAYER_SEED0, "init")
    layer = runner.DeviceLayer(2, 16, 16, 60, 6, groups, 8, 4, "bf16")
    layer.set_params(p)
    layer.set_inputs(x, dy)
    gswa.gswa_profile_enable(True)
    try:
        gswa.gswa_profile_collect()
        layer.forward()
        layer.backward()
        res, dropped = gswa.gswa_profile_collect()
    finally:
        gswa.gswa_profile_enable(False)
    torch.cuda.synchronize()
    assert dropped == 0
    assert res["fused_fwd"][1] == 1 and res["fused_bwd"][1] == res["reduce_partials"][1] >= 1  # one sum per launch
    if groups == 6:
        assert res["fused_bwd"][1] == 2
    assert all(ms > 0 for ms, _ in res.values())
    layer.forward()
    assert gswa.gswa_profile_collect()[0] == {}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_no_cascade_flag(oracle, dtype):
    parity.check_case(oracle, 1, 16, 16, 60, 6, 3, 8, 4, dtype, regime="stress", cascade=False)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_inference_mode_matches_training_forward(oracle, dtype):
    x, dy, p = parity.make_inputs(2, 16, 16, 60, 6, 2, 8, dtype, synth.LAYER_SEED0, "stress")
    a, _ = parity.gpu_results(x, dy, p, 6, 2, 8, 4, dtype, backward=True)
    b, _ = parity.gpu_results(x, dy, p, 6, 2, 8, 4, dtype, backward=False)
    assert np.array_equal(a["y"], b["y"])


def test_accumulate_flag_adds_into_parameter_gradients(oracle):
    import torch
    from paper_2409_06206_amd import gswa, runner
    x, dy, p = parity.make_inputs(1, 16, 16, 60, 6, 2, 8, "f32", synth.LAYER_SEED0, "stress")
    layer = runner.DeviceLayer(1, 16, 16, 60, 6, 2, 8, 4, "f32", gswa.GSWA_ACCUM_WGRAD)
    layer.set_params(p)
    layer.set_inputs(x, dy)
    for g in layer.grads.values():
        g.fill_(1.0)
    layer.forward()
    layer.backward()
    layer.backward()
    torch.cuda.synchronize()
    got = layer.results()
    want = parity.oracle_results(oracle, x, dy, p, 6, 2, 8, 4)
    for k in parity.GRAD_NAMES[1:]:
        assert parity.rel_err(got[k], 2.0 * want[k] + 1.0) <= 1e-5, k
    assert parity.rel_err(got["dx"], want["dx"]) <= 1e-5


def test_accumulate_flag_on_fused_path(oracle):
    import torch
    from paper_2409_06206_amd import gswa, runner
    x, dy, p = parity.make_inputs(2, 16, 16, 60, 6, 3, 8, "bf16", synth.LAYER_SEED0, "stress")
    layer = runner.DeviceLayer(2, 16, 16, 60, 6, 3, 8, 4, "bf16", gswa.GSWA_ACCUM_WGRAD)
    layer.set_params(p)
    layer.set_inputs(x, dy)
    for g in layer.grads.values():
        g.fill_(0.5)
    layer.forward()
    layer.backward()
    layer.backward()
    torch.cuda.synchronize()
    got = layer.results()
    want = parity.oracle_results(oracle, x, dy, p, 6, 3, 8, 4)
    for k in parity.GRAD_NAMES[1:]:
        assert parity.rel_err(got[k] - 0.5, 2.0 * want[k]) <= parity.TOL["bf16"], k


def test_accumulate_flag_with_narrow_query_key(oracle):
    """12 x 12 windows, narrow q/k (gradient copies summed at the end): two backward calls add twice."""
    import torch
    from paper_2409_06206_amd import gswa, runner
    shape = (2, 24, 24, 60, 4, 2, 12)
    x, dy, p = parity.make_inputs(*shape, "bf16", synth.LAYER_SEED0, "stress", dqk=4)
    layer = runner.DeviceLayer(*shape, 6, "bf16", gswa.GSWA_ACCUM_WGRAD, dqk=4)
    layer.set_params(p)
    layer.set_inputs(x, dy)
    for g in layer.grads.values():
        g.fill_(0.25)
    layer.forward()
    layer.backward()
    layer.backward()
    torch.cuda.synchronize()
    got = layer.results()
    want = parity.oracle_results(oracle, x, dy, p, 4, 2, 12, 6, dqk=4)
    for k in parity.GRAD_NAMES[1:]:
        assert parity.rel_err(got[k] - 0.25, 2.0 * want[k]) <= parity.TOL["bf16"], k
    assert parity.rel_err(got["dx"], want["dx"]) <= parity.TOL["bf16"]


def test_fused_path_gradients_are_run_to_run_identical():
    """The fused backward sums per-workgroup partials in a fixed order: no atomics on outputs."""
    import torch
    from paper_2409_06206_amd import runner
    x, dy, p = parity.make_inputs(4, 32, 32, 60, 6, 2, 8, "bf16", synth.LAYER_SEED0, "stress")
    layer = runner.DeviceLayer(4, 32, 32, 60, 6, 2, 8, 4, "bf16")
    layer.set_params(p)
    layer.set_inputs(x, dy)
    runs = []
    for _ in range(3):
        layer.forward()
        layer.backward()
        torch.cuda.synchronize()
        runs.append({k: v.copy() for k, v in layer.results().items()})
    for r in runs[1:]:
        for k in r:
            assert np.array_equal(r[k], runs[0][k]), k


def test_repeated_calls_reuse_buffers(oracle):
    """Two different inputs through the same buffers: the second result owes nothing to the first."""
    import torch
    from paper_2409_06206_amd import runner
    x1, dy1, p = parity.make_inputs(1, 16, 16, 60, 6, 2, 8, "bf16", synth.LAYER_SEED0, "stress")
    x2, dy2, _ = parity.make_inputs(1, 16, 16, 60, 6, 2, 8, "bf16", synth.LAYER_SEED0 + 9, "stress")
    layer = runner.DeviceLayer(1, 16, 16, 60, 6, 2, 8, 4, "bf16")
    layer.set_params(p)
    for x, dy in ((x1, dy1), (x2, dy2)):
        layer.set_inputs(x, dy)
        layer.forward()
        layer.backward()
        torch.cuda.synchronize()
        got = layer.results()
        want = parity.oracle_results(oracle, x, dy, p, 6, 2, 8, 4)
        for k in want:
            assert parity.rel_err(got[k], want[k]) <= parity.TOL["bf16"], k


FULL = [
    # name, groups, layer index: full benchmark shapes, every element compared
    ("c2", 1, 0), ("c2", 2, 1), ("c2", 3, 0), ("c2", 6, 1),
    ("c3", 1, 1), ("c3", 2, 0), ("c3", 3, 1),
    ("c4", 2, 1), ("c4", 3, 1),
    ("agile_h4_qk16", 2, 1), ("agile_h4_qk32", 4, 0), ("agile_h6_qk24", 2, 1), ("agile_h6_qk24", 3, 0),
]


@pytest.mark.parametrize("name,groups,layer", FULL)
def test_full_size_layers(oracle, name, groups, layer):
    cfg = synth.CONFIGS[name]
    _say("full", name, "G", groups, "layer", layer)
    errs, _ = parity.check_case(oracle, cfg["B"], cfg["H"], cfg["W"], cfg["C"], cfg["heads"], groups,
                                cfg["window"], cfg["layers"][layer], cfg["dtype"],
                                seed=synth.LAYER_SEED0 + layer, dqk=cfg.get("dqk", 0))
    _say("  errors", {k: f"{v:.2e}" for k, v in errs.items()})


# The benchmark's initialisation (weights of standard deviation 0.02) gives nearly uniform
# probabilities, which would hide a wrong mask, bias index or exponential: the wide layers are
# therefore also run at full size with scores of order 1-5 (`stress`), shifted.
FULL_STRESS = [("c2", 2, 1), ("c3", 1, 1), ("c3", 2, 1), ("c3", 3, 1), ("c4", 2, 1), ("c4", 3, 1)]


@pytest.mark.parametrize("name,groups,layer", FULL_STRESS)
def test_full_size_layers_peaky_softmax(oracle, name, groups, layer):
    cfg = synth.CONFIGS[name]
    assert cfg["layers"][layer] > 0
    _say("full, stress", name, "G", groups, "layer", layer)
    errs, _ = parity.check_case(oracle, cfg["B"], cfg["H"], cfg["W"], cfg["C"], cfg["heads"], groups,
                                cfg["window"], cfg["layers"][layer], cfg["dtype"],
                                seed=synth.LAYER_SEED0 + 40 + layer, regime="stress")
    _say("  errors", {k: f"{v:.2e}" for k, v in errs.items()})


@pytest.mark.parametrize("groups", [2, 3])
def test_more_windows_than_wavefronts(oracle, groups):
    """48 x (9 x 5) = 2160 windows: more than the 2048 wavefronts a forward launch has on 256
    compute units, so some waves take a second window; odd window counts per image, shifted."""
    _say("many windows", groups)
    errs, _ = parity.check_case(oracle, 48, 72, 40, 60, 6, groups, 8, 4, "bf16",
                                seed=synth.LAYER_SEED0 + 3, regime="stress")
    _say("  errors", {k: f"{v:.2e}" for k, v in errs.items()})


@pytest.mark.parametrize("groups", [1, 2, 3])
@pytest.mark.parametrize("B,H,W,shift,cascade", [
    (1, 8, 40, 0, True),    # 5 windows: one a workgroup, the pipeline of groups filled and drained at once
    (1, 24, 16, 7, True),   # windows cut by the shift in both directions
    (7, 56, 48, 4, True),   # 294: a second window for some of 256 workgroups
    (4, 24, 104, 3, False), # 156, no cascade
    (11, 72, 64, 1, True),  # 792: three or four windows a workgroup
    (3, 8, 8, 0, True),     # images of one window
    (1, 16, 8, 5, True),    # of two, both cut by the shift in both directions
    (2, 16, 16, 4, True),   # of four
])
def test_narrow_backward_with_a_wave_per_head(oracle, B, H, W, shift, cascade, groups):
    """One to three groups of a narrow layer, images of any size: the whole backward is one launch and one sum, and the same bits
    twice."""
    _say("wave per head", B, H, W, shift, cascade, groups)
    with parity.launch_counts() as counts:
        errs, layer = parity.check_case(oracle, B, H, W, 60, 6, groups, 8, shift, "bf16", seed=synth.LAYER_SEED0 + 4,
                                        regime="stress", cascade=cascade)
    assert counts["fused_bwd"] == 1 and counts["reduce_partials"] == 1
    first = layer.results()
    layer.backward()
    again = layer.results()
    assert all(np.array_equal(first[k], again[k]) for k in first)
    _say("  errors", {k: f"{v:.2e}" for k, v in errs.items()})


@pytest.mark.parametrize("B,H,W,shift,cascade,accumulate", [
    (1, 8, 8, 0, True, False),     # one window
    (1, 24, 40, 7, True, True),    # 15, cut by an odd shift in both directions, added
    (7, 56, 48, 4, True, False),   # 294: a second window for some of 256 workgroups
    (4, 24, 104, 3, False, True),  # 156, no cascade
    (13, 72, 64, 1, True, False),  # 936: three or four a workgroup, the last three sums in one launch
])
def test_wide_backward_with_a_wave_per_head(oracle, B, H, W, shift, cascade, accumulate):
    """Two groups of a wide layer: one launch a group, any shift, and the same bits twice (added onto 0.5 where asked)."""
    from paper_2409_06206_amd import gswa, runner
    _say("wide, wave per head", B, H, W, shift, cascade, accumulate)
    flags = (gswa.GSWA_ACCUM_WGRAD if accumulate else 0) | (0 if cascade else gswa.GSWA_NO_CASCADE)
    x, dy, p = parity.make_inputs(B, H, W, 180, 6, 2, 8, "bf16", synth.LAYER_SEED0 + 4, "stress")
    layer = runner.DeviceLayer(B, H, W, 180, 6, 2, 8, shift, "bf16", flags)
    layer.set_params(p)
    layer.set_inputs(x, dy)
    layer.forward()
    start, runs = 0.5 if accumulate else 0.0, []
    for _ in range(2):
        for g in layer.grads.values():
            g.fill_(0.5)
        with parity.launch_counts() as counts:
            layer.backward()
        assert counts["wide_attn_bwd"] == 2 and "wide_qkv_grad" not in counts and "fused_bwd" not in counts, counts
        runs.append({k: v.copy() for k, v in layer.results().items()})
    want = parity.oracle_results(oracle, x, dy, p, 6, 2, 8, shift, cascade=cascade)
    for k in parity.GRAD_NAMES:
        assert parity.rel_err(runs[0][k] - (start if k != "dx" else 0.0), want[k]) <= parity.TOL["bf16"], k
        assert np.array_equal(runs[0][k], runs[1][k]), k


@pytest.mark.parametrize("groups", [2, 3])
def test_wide_layers_more_windows_than_wavefronts(oracle, groups):
    """27 x (9 x 5) = 1215 windows of a wide layer.  Two groups: four or five windows for each of 256 workgroups of a backward
    launch.  Three groups: more than the 1024 wavefronts of a backward launch
    on 256 compute units (a ragged second round), an odd number of windows (the kernel that takes
    them in pairs is left with one), odd window counts per image, shifted."""
    _say("many windows, wide", groups)
    errs, _ = parity.check_case(oracle, 27, 72, 40, 180, 6, groups, 8, 4, "bf16",
                                seed=synth.LAYER_SEED0 + 5, regime="stress")
    _say("  errors", {k: f"{v:.2e}" for k, v in errs.items()})


@pytest.mark.parametrize("shift", [2, 3, 6])
def test_wide_layers_other_shifts(oracle, shift):
    """Shifts other than half a window: even ones split the last window column's rows at a
    16-byte boundary, odd ones do not."""
    parity.check_case(oracle, 1, 24, 16, 180, 6, 2, 8, shift, "bf16", regime="stress")


@pytest.mark.parametrize("B,H,W,shift", [(1, 8, 8, 0), (1, 24, 16, 3), (5, 56, 64, 7)])
def test_three_groups_of_a_wide_layer_odd_shifts(oracle, B, H, W, shift):
    """Three groups: an odd shift takes a launch of whole groups a head pair, any other the streamed backward; one window, six,
    and more than one a workgroup."""
    with parity.launch_counts() as counts:
        parity.check_case(oracle, B, H, W, 180, 6, 3, 8, shift, "bf16", regime="stress")
    assert (counts.get("fused_bwd", 0), counts.get("wide_attn_bwd", 0)) == ((3, 0) if shift % 2 else (0, 3)), counts


@pytest.mark.parametrize("regime", ["init", "stress"])
@pytest.mark.parametrize("name", ["c5_m8", "c5_m16"])
def test_large_image_inference(oracle, name, regime):
    cfg = synth.CONFIGS[name]
    _say("full", name, regime)
    errs, _ = parity.check_case(oracle, cfg["B"], cfg["H"], cfg["W"], cfg["C"], cfg["heads"],
                                cfg["groups"][0], cfg["window"], cfg["layers"][0], cfg["dtype"],
                                backward=False, regime=regime)
    _say("  errors", {k: f"{v:.2e}" for k, v in errs.items()})


def _random_shapes(n, seed):
    """Seeded random layer shapes that satisfy the divisibility rules (staged path territory)."""
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        M = int(rng.choice([2, 3, 4, 5, 6, 8]))
        heads = int(rng.choice([1, 2, 3, 4, 6]))
        groups = int(rng.choice([g for g in (1, 2, 3, 4, 6) if heads % g == 0]))
        d = int(rng.integers(1, 9))
        B, nh, nw = int(rng.integers(1, 3)), int(rng.integers(1, 4)), int(rng.integers(1, 4))
        s = int(rng.integers(0, M))
        out.append((B, nh * M, nw * M, heads * d, heads, groups, M, s))
    return out


AGILE_SMALL = [
    # B, H, W, C, heads, groups, window, shift, dqk, dtype, regime   (Sec. "Parameter Allocation")
    (2, 24, 24, 60, 4, 2, 12, 6, 4, "f32", "stress"),
    (1, 24, 36, 60, 4, 2, 12, 0, 8, "f32", "init"),
    (2, 24, 24, 60, 6, 2, 12, 6, 4, "bf16", "stress"),
    (1, 36, 24, 60, 6, 3, 12, 5, 16, "bf16", "stress"),
    (3, 16, 24, 60, 6, 2, 8, 4, 4, "bf16", "stress"),     # narrow q/k on 8 x 8 windows
    (2, 16, 16, 60, 6, 1, 8, 4, 16, "bf16", "init"),      # q/k wider than v
    (1, 24, 24, 180, 6, 2, 12, 6, 8, "bf16", "stress"),
    (1, 16, 16, 12, 6, 6, 4, 1, 1, "f32", "stress"),
    (2, 24, 24, 60, 4, 2, 12, 6, 20, "bf16", "stress"),   # q/k of 17..32 channels: two 16-channel tiles
    (1, 24, 24, 180, 6, 3, 12, 7, 32, "bf16", "stress"),
    (2, 16, 16, 42, 6, 2, 8, 3, 5, "bf16", "stress"),     # head width 7, 21 channels per group (odd row strides)
    (1, 24, 24, 18, 6, 2, 12, 6, 3, "bf16", "stress"),    # head width 3
    (2, 24, 24, 60, 6, 1, 12, 6, 4, "bf16", "stress"),    # one group: two q/k tiles, four v tiles, two K steps
    (1, 24, 36, 60, 6, 3, 12, 5, 4, "bf16", "stress"),
    (1, 24, 24, 60, 6, 6, 12, 6, 8, "bf16", "stress"),    # one head per group
    (2, 16, 16, 60, 4, 1, 8, 4, 8, "bf16", "stress"),
    (1, 24, 24, 36, 6, 3, 12, 6, 6, "bf16", "init"),      # q/k as wide as v, spelled out
]


@pytest.mark.parametrize("B,H,W,C,heads,groups,window,shift,dqk,dtype,regime", AGILE_SMALL)
def test_narrow_query_key_and_window_12(oracle, B, H, W, C, heads, groups, window, shift, dqk, dtype, regime):
    """q and k of dqk channels per head, 12 x 12 windows: forward and every gradient."""
    parity.check_case(oracle, B, H, W, C, heads, groups, window, shift, dtype, regime=regime, dqk=dqk)
    parity.check_case(oracle, B, H, W, C, heads, groups, window, shift, dtype, regime=regime, dqk=dqk,
               cascade=False, seed=synth.LAYER_SEED0 + 3)


@pytest.mark.parametrize("heads,dqk,kernel", [(4, 4, "window_attn_fwd"), (6, 0, "window_fwd")])
def test_window_forward_inference_and_staged_forward_agree(oracle, heads, dqk, kernel):
    """12 x 12 windows: the one-launch forward (of the kernels for both passes, and of the one for the forward alone)
    without a saved buffer gives the bits of the training forward, and the one-kernel-per-step forward the same result
    within the tolerance."""
    from paper_2409_06206_amd import gswa
    shape = (2, 24, 24, 60, heads, 2, 12)
    x, dy, p = parity.make_inputs(*shape, "bf16", synth.LAYER_SEED0, "stress", dqk=dqk)
    a, _ = parity.gpu_results(x, dy, p, heads, 2, 12, 6, "bf16", backward=True, dqk=dqk)
    with parity.launched() as names:
        b, _ = parity.gpu_results(x, dy, p, heads, 2, 12, 6, "bf16", backward=False, dqk=dqk)
    assert names == {kernel}
    c, _ = parity.gpu_results(x, dy, p, heads, 2, 12, 6, "bf16", backward=False, dqk=dqk,
                              extra_flags=gswa.GSWA_FORCE_STAGED)
    assert np.array_equal(a["y"], b["y"])
    assert parity.rel_err(c["y"], a["y"].astype(np.float64)) <= parity.TOL["bf16"]


def test_spelled_out_query_key_width_takes_the_same_path(oracle):
    """dqk = C / heads is the plain layer: same kernels, same bits."""
    x, dy, p = parity.make_inputs(2, 16, 16, 60, 6, 2, 8, "bf16", synth.LAYER_SEED0, "stress")
    a, _ = parity.gpu_results(x, dy, p, 6, 2, 8, 4, "bf16")
    b, _ = parity.gpu_results(x, dy, p, 6, 2, 8, 4, "bf16", dqk=10)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("shape", _random_shapes(16, 2024))
def test_random_shapes_fp32(oracle, shape):
    B, H, W, C, heads, groups, M, s = shape
    _say("random", shape)
    parity.check_case(oracle, B, H, W, C, heads, groups, M, s, "f32", seed=synth.LAYER_SEED0 + 7,
                      regime="stress")


@pytest.mark.parametrize("shape", _random_shapes(6, 77))
def test_random_shapes_bf16(oracle, shape):
    B, H, W, C, heads, groups, M, s = shape
    _say("random bf16", shape)
    # tiny layers (a few windows, head width down to 1): see check_case on `conditioned`
    errs, _ = parity.check_case(oracle, B, H, W, C, heads, groups, M, s, "bf16", seed=synth.LAYER_SEED0 + 8,
                                regime="stress", conditioned=True)
    _say("  errors", {k: f"{v:.2e}" for k, v in errs.items()})


@pytest.mark.parametrize("dtype,shape,flags", [
    ("f32", (4, 32, 32, 60, 6, 2, 8, 4), 0),                 # one workgroup per window
    ("f32", (4, 32, 32, 60, 6, 2, 8, 4), "staged"),          # one-kernel-per-step path, vector ALUs
    ("f32", (2, 32, 48, 180, 6, 3, 16, 8), 0),               # 256-token windows: strips of queries
    ("bf16", (4, 32, 32, 60, 6, 2, 8, 4), "staged"),         # the same path on the matrix cores
    ("bf16", (2, 48, 48, 60, 4, 2, 12, 6), 0),               # 12 x 12 windows, narrow q/k: one workgroup per window
    ("bf16", (2, 48, 48, 60, 4, 2, 12, 6), "staged"),        # the same, one-kernel-per-step backward
])
def test_reproducible_mode_gives_the_same_bits_every_run(oracle, dtype, shape, flags):
    """GSWA_DETERMINISTIC: no gradient depends on the order in which workgroups finish."""
    import torch
    from paper_2409_06206_amd import gswa, runner
    B, H, W, C, heads, groups, window, shift = shape
    dqk = 4 if window == 12 else 0
    fl = gswa.GSWA_DETERMINISTIC | (gswa.GSWA_FORCE_STAGED if flags == "staged" else 0)
    x, dy, p = parity.make_inputs(B, H, W, C, heads, groups, window, dtype, synth.LAYER_SEED0 + 5, "stress", dqk)
    layer = runner.DeviceLayer(B, H, W, C, heads, groups, window, shift, dtype, fl, dqk=dqk)
    layer.set_params(p)
    layer.set_inputs(x, dy)
    runs = []
    for _ in range(3):
        layer.ws.fill_(0x5a)          # whatever an earlier call left in the scratch must not matter
        layer.forward()
        layer.backward()
        torch.cuda.synchronize()
        runs.append({k: v.copy() for k, v in layer.results().items()})
    for r in runs[1:]:
        for k in r:
            assert np.array_equal(r[k], runs[0][k]), k
    want = parity.oracle_results(oracle, x, dy, p, heads, groups, window, shift, dqk=dqk)
    for k in want:
        assert parity.rel_err(runs[0][k], want[k]) <= parity.TOL[dtype], k


def test_training_forward_on_the_fused_path_needs_no_scratch(oracle):
    """Where gswa_query_bytes reports 0 bytes of forward scratch, ws may be NULL."""
    import torch
    from paper_2409_06206_amd import gswa, runner
    x, dy, p = parity.make_inputs(2, 16, 16, 60, 6, 2, 8, "bf16", synth.LAYER_SEED0, "stress")
    layer = runner.DeviceLayer(2, 16, 16, 60, 6, 2, 8, 4, "bf16")
    assert layer.fwd_ws_bytes == 0
    layer.set_params(p)
    layer.set_inputs(x, dy)
    layer.forward()
    torch.cuda.synchronize()
    y_ref = layer.y.clone()
    layer.y.zero_()
    q = layer.params
    gswa.gswa_forward(layer.desc, layer.x, q["w_qkv"], q["b_qkv"], q["w_proj"], q["b_proj"], q["table"],
                      layer.y, layer.saved, None)
    torch.cuda.synchronize()
    assert torch.equal(layer.y, y_ref)
    with pytest.raises(gswa.GswaError):   # inference keeps its state in the scratch: NULL is an error there
        gswa.gswa_forward(layer.desc, layer.x, q["w_qkv"], q["b_qkv"], q["w_proj"], q["b_proj"], q["table"],
                          layer.y, None, None)


@pytest.mark.parametrize("groups,shape,shift", [
    (1, (4, 64, 72), 3),      # 288 windows: more than the 256 vectors of parameter gradients, so some workgroups take two
    (2, (4, 64, 72), 4),
    (3, (1, 8, 8), 5),        # one window, cut by the shift in both directions
    (6, (33, 8, 64), 7),      # 264 windows of one window row
])
def test_fp32_layers_one_workgroup_per_window(oracle, groups, shape, shift):
    """fp32 layers of 60 channels and 8x8 windows run one workgroup per window: every group count, workgroups with
    one and with two windows, windows cut by the shift in every way."""
    with parity.launched() as names:
        parity.check_case(oracle, *shape, 60, 6, groups, 8, shift, "f32", regime="stress")
    assert names == {"window_attn_fwd", "window_bwd", "reduce_partials"}


@pytest.mark.parametrize("heads,groups,dqk,shape,shift", [
    (4, 1, 4, (1, 24, 36), 6), (4, 1, 8, (1, 12, 12), 3), (4, 2, 8, (1, 24, 24), 0), (4, 4, 4, (2, 12, 24), 5),
    (6, 1, 4, (1, 24, 24), 6), (6, 6, 4, (29, 36, 36), 6),
])
def test_12x12_windows_one_workgroup_per_window(oracle, heads, groups, dqk, shape, shift):
    """bf16 attention layers with 12x12 windows: the organisations of the heads that no other test runs."""
    with parity.launched() as names:
        parity.check_case(oracle, *shape, 60, heads, groups, 12, shift, "bf16", regime="stress", dqk=dqk)
    assert names == {"window_attn_fwd", "window_bwd", "reduce_partials"}


@pytest.mark.parametrize("heads,groups,dqk", [(4, 1, 4), (4, 2, 8), (6, 3, 4)])
def test_shift_mask_of_12x12_windows_is_minus_100(oracle, heads, groups, dqk):
    """One 12x12 window cut in half by the shift, no queries or keys, a bias of 100 between tokens six and more rows
    apart: they lie on both sides of the cut, so bias and mask cancel, and any other mask (-99.8 is what -100 log2(e)
    becomes in bf16) gives them other weights than the tokens of the query's own side."""
    B, H, W, C, window, shift = 1, 12, 12, 60, 12, 6
    x, dy, p = parity.make_inputs(B, H, W, C, heads, groups, window, "bf16", synth.LAYER_SEED0, "stress", dqk)
    hg = heads // groups
    p["w_qkv"][:, :2 * hg * dqk], p["b_qkv"][:, :2 * hg * dqk] = 0.0, 0.0
    rows = np.arange((2 * window - 1) ** 2) // (2 * window - 1) - (window - 1)
    p["table"][:] = np.where(np.abs(rows) >= 6, 100.0, 0.0)[:, None]
    x += np.where(np.arange(H) < 6, 1.0, -1.0)[None, :, None, None]
    x = synth.quantize(x, "bf16")
    want = parity.oracle_results(oracle, x, dy, p, heads, groups, window, shift, dqk=dqk)
    got, _ = parity.gpu_results(x, dy, p, heads, groups, window, shift, "bf16", dqk=dqk)
    errs = {k: parity.rel_err(got[k], want[k]) for k in ("y", "dx")}
    assert max(errs.values()) <= parity.TOL["bf16"], errs


@pytest.mark.parametrize("dqk", [4, 8])
def test_cascade_of_odd_groups_is_added_in_fp32(oracle, dqk):
    """12x12 windows, four groups of 15 channels, no queries or keys: group 0 puts out delta = 15/4096 everywhere, group 1
    holds +1 and -1 by turns and its values are sums of a pair, so they are 2 delta; with x + O_0 rounded to bf16 on the
    way they would be 2^-8, half as much.  What is left are the roundings of v, of the group's output and of y, 2^-9 each."""
    C, groups, window, Cg = 60, 4, 12, 15
    p = {k: np.zeros(s, dtype=np.float32) for k, s in synth.param_shapes(C, 4, groups, window, dqk).items()}
    p["w_qkv"][0, 2 * dqk:] = np.eye(Cg)
    for i in range(14):
        p["w_qkv"][1, 2 * dqk + i, [i - i % 2, i - i % 2 + 1]] = 1.0
    p["w_proj"][:] = np.eye(C)
    x = np.zeros((1, 24, 24, C), dtype=np.float32)
    x[..., :Cg] = 15.0 / 4096.0
    x[..., Cg:2 * Cg - 1] = np.where(np.arange(14) % 2 == 0, 1.0, -1.0)
    want = oracle.forward(x, p["w_qkv"], p["b_qkv"], p["w_proj"], p["b_proj"], p["table"], heads=4, groups=groups,
                          window=window, shift=6, dqk=dqk)[..., Cg:2 * Cg]
    got, _ = parity.gpu_results(x, None, p, 4, groups, window, 6, "bf16", backward=False, dqk=dqk)
    assert abs(want.max() - 30.0 / 4096.0) <= 1e-9
    assert parity.rel_err(got["y"][..., Cg:2 * Cg], want) <= 3 * parity.U_BF16


@pytest.mark.parametrize("groups", [2, 3])
def test_fp32_on_the_matrix_cores_is_as_exact_as_on_the_vector_alus(oracle, groups):
    """fp32 layers of 60 channels: the error of y, dx and the bias-table gradient against fp64, as a geometric mean over
    eight layers, beside that of the one-kernel-per-step path.  Both are a few 2^-24 of roundings; the mean of a path
    moves by about 2 % from one set of layers to another, and 7 % is what is allowed.  (A sum of exponentials in the order
    of the keys, scores scaled before their product or probabilities from a rounded logarithm cost 10 to 16 %.)"""
    from paper_2409_06206_amd import gswa
    rel = lambda got, want: float(np.linalg.norm(np.asarray(got, dtype=np.float64) - want) / np.linalg.norm(want))
    logs = {0: [], gswa.GSWA_FORCE_STAGED: []}
    for seed in range(8):
        x, dy, p = parity.make_inputs(2, 16, 24, 60, 6, groups, 8, "f32", synth.LAYER_SEED0 + 20 + seed, "stress")
        want = parity.oracle_results(oracle, x, dy, p, 6, groups, 8, 4)
        for flags, rows in logs.items():
            got, _ = parity.gpu_results(x, dy, p, 6, groups, 8, 4, "f32", extra_flags=flags)
            rows.append([np.log(rel(got[k], want[k])) for k in ("y", "dx", "dtable")])
    ratio = np.exp(np.mean(logs[0], axis=0) - np.mean(logs[gswa.GSWA_FORCE_STAGED], axis=0))
    print("error of y, dx, dtable against the one-kernel-per-step path's:", ratio, flush=True)
    assert ratio.max() <= 1.07, ratio
