"""GPU parity of spec_tv_loss_fwd_bwd against the float64 oracle (through
the C ABI): loss, per-step overlap and the gradient w.r.t. the draft logits
for every loss mode, ragged vocabularies, forward-only calls and the
full-size training workload (sampled positions plus a loss identity)."""

import ctypes

import numpy as np
import pytest
import torch

import oracle
from oracle.tv import chain_factors
from paper_2606_12370_amd import binding
from paper_2606_12370_amd import workloads as W
from tests.parity import TOL, compare_tv, device_inputs, host_logits

pytestmark = pytest.mark.gpu
MODES = {"e2e": 0, "prod": 1, "per_step": 2}


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    binding.load_library()
    yield
    torch.cuda.synchronize()


def run_case(d, mode, T=1.0, scale=1.0, want_grad=True):
    tgt, drf = device_inputs(d)
    loss, ov, grad = binding.tv_loss_fwd_bwd(tgt, drf, T, mode, scale, want_grad=want_grad)
    torch.cuda.synchronize()
    ref = oracle.tv_ref(W.to_float64(d["target"], d["dtype"]), W.to_float64(d["draft"], d["dtype"]),
                        float(np.float32(T)), MODES[mode], float(np.float32(scale)), want_grad=True)
    return loss, ov, grad, ref


@pytest.mark.parametrize("mode", ["e2e", "prod", "per_step"])
@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("T", [1.0, 0.7])
def test_small_all_modes(mode, dtype, T):
    d = W.tv_inputs_numpy(4, 3, 5000, dtype, 3)
    loss, ov, grad, ref = run_case(d, mode, T, scale=0.5)
    print(mode, dtype, T, compare_tv(loss, ov, grad, ref, dtype))


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("N,K,V", [(3, 1, 1), (2, 2, 7), (3, 3, 1023), (2, 8, 8197), (5, 2, 20480 + 3)])
def test_ragged(dtype, N, K, V):
    d = W.tv_inputs_numpy(N, K, V, dtype, 11 + V)
    loss, ov, grad, ref = run_case(d, "e2e", 1.0, 1.0)
    print(dtype, N, K, V, compare_tv(loss, ov, grad, ref, dtype))


def test_forward_only_and_q_equals_p():
    d = W.tv_inputs_numpy(6, 3, 30000, W.BF16, 4)
    loss, ov, grad, ref = run_case(d, "e2e", 1.0, 1.0, want_grad=False)
    assert grad is None
    compare_tv(loss, ov, None, ref, W.BF16)
    d = W.tv_inputs_numpy(3, 2, 30000, W.F32, 5, q_equals_p=True)
    loss, ov, grad, ref = run_case(d, "prod")
    assert torch.allclose(ov, torch.ones_like(ov), atol=1e-5)
    # q = p is a stationary point: only rounding residue remains
    assert float(grad.abs().max()) < 1e-6


def test_determinism():
    d = W.tv_inputs_numpy(8, 3, 40000, W.BF16, 6)
    tgt, drf = device_inputs(d)
    a = binding.tv_loss_fwd_bwd(tgt, drf, 0.9, "e2e", 0.25)
    b = binding.tv_loss_fwd_bwd(tgt, drf, 0.9, "e2e", 0.25)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.fixture(scope="module")
def training_inputs():
    cfg = W.CONFIGS["tv_bf16_n16384_k3_v151936"]
    d = W.tv_inputs_torch(cfg["N"], cfg["K"], cfg["V"], cfg["dtype"], cfg["seed"])
    yield cfg, d
    del d
    torch.cuda.empty_cache()


@pytest.mark.parametrize("mode,scale", [("prod", 1.0), ("e2e", 1.0 / 16384), ("per_step", 0.5)])
def test_training_workload_sampled_positions(training_inputs, mode, scale):
    """N=16384 positions x 3 steps x V=151936 (bf16) in each loss mode: the
    paper's multi-step loss (Eq. e2e_tv) with a mean over positions, the
    product-of-overlaps loss and the per-step loss.  Sampled positions
    (their overlaps and every gradient element of their 3 x 151936 draft
    logits) against the oracle; the total loss against the loss recomputed in
    float64 from the kernel's own per-step overlaps."""
    cfg, d = training_inputs
    loss, ov, grad = binding.tv_loss_fwd_bwd(d["target"], d["draft"], 1.0, mode, scale)
    torch.cuda.synchronize()
    rng = np.random.default_rng(cfg["seed"] + len(mode))
    pos = np.sort(rng.choice(cfg["N"], size=4, replace=False))
    pi = torch.as_tensor(pos, device="cuda")
    sc = float(np.float32(scale))
    ref = oracle.tv_ref(host_logits(d["target"][pi], W.BF16), host_logits(d["draft"][pi], W.BF16), 1.0,
                        MODES[mode], sc)
    rep = compare_tv(loss, ov, grad, ref, W.BF16, positions=pos, loss_exact=False)
    _, L = chain_factors(ov.cpu().numpy().astype(np.float64), MODES[mode])
    lg = float(loss.cpu().numpy()[0])
    assert abs(lg - sc * L.sum()) <= TOL[W.BF16] * abs(sc * L.sum())
    print("training workload", mode, rep, "loss", lg)


@pytest.mark.parametrize("mode", ["e2e", "prod", "per_step"])
@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
def test_masked_vocabulary(mode, dtype):
    """The same 5 % of positions and the last 37 tokens are -inf in both the
    target and the draft row (p = q = 0): they add nothing to the overlaps
    and get a zero gradient."""
    N, K, V = 3, 3, 5000
    d = W.tv_inputs_numpy(N, K, V, dtype, 71)
    rng = np.random.default_rng(72)
    mask = rng.random((N, K, V)) < 0.05
    mask[..., V - 37:] = True
    neg = W.f32_to_bf16_bits(np.array([-np.inf], np.float32))[0] if dtype == W.BF16 else np.float32(-np.inf)
    for key in ("target", "draft"):
        arr = d[key].copy()
        arr[mask] = neg
        d[key] = arr
    loss, ov, grad, ref = run_case(d, mode, 0.9, scale=0.5)
    assert np.all(np.isfinite(ref["grad"]))
    assert np.all(grad.cpu().numpy()[mask] == 0.0)
    print(mode, dtype, compare_tv(loss, ov, grad, ref, dtype))


@pytest.mark.parametrize("mode", ["e2e", "per_step"])
@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
def test_target_masked_tokens(mode, dtype):
    """Tokens the target masks (-inf) but the draft does not: p = 0 < q, so
    they add nothing to the overlap and their gradient is -g S q / T."""
    N, K, V = 3, 3, 5000
    d = W.tv_inputs_numpy(N, K, V, dtype, 91)
    mask = np.random.default_rng(92).random((N, K, V)) < 0.05
    neg = W.f32_to_bf16_bits(np.array([-np.inf], np.float32))[0] if dtype == W.BF16 else np.float32(-np.inf)
    arr = d["target"].copy()
    arr[mask] = neg
    d["target"] = arr
    loss, ov, grad, ref = run_case(d, mode, 0.9, scale=0.5)
    assert np.all(np.isfinite(ref["grad"]))
    print(mode, dtype, compare_tv(loss, ov, grad, ref, dtype))


@pytest.mark.parametrize("mode", ["e2e", "prod", "per_step"])
@pytest.mark.parametrize("N,K,V,dtype", [
    (3, 2, 4, W.BF16),            # one vector per row
    (5, 3, 2048, W.BF16),         # one whole tile of a slice
    (5, 3, 2052, W.BF16),         # a second tile of one vector
    (2, 8, 38 * 2048, W.BF16),    # the most tiles one slice holds
    (2, 8, 38 * 2048 + 4, W.BF16),
    (300, 1, 16 * 2048 - 8, W.BF16),   # more positions than groups: several per group, the last round partial
    (70, 4, 80 * 1024 + 12, W.BF16),   # the same with slices exchanging records
    (2, 3, 19 * 2048 + 4, W.F32),
    (5, 3, 2049, W.BF16),         # rows at odd addresses, a last vector of one, two and three elements
    (5, 3, 38 * 2048 + 2, W.BF16),
    (4, 2, 2048 + 7, W.F32),
    (4, 2, 19 * 2048 + 2, W.F32),
    (3, 2, 5, W.F32),             # one vector and one element
    (2, 8, 262144, W.F32),        # more slices than a position may take: the two-read passes
])
def test_single_read_edges(N, K, V, dtype, mode):
    """The gradient call at the edges of the single-read pass's tiles, slices
    and position groups, rows at any alignment among them, and just beyond the
    slices it takes, against the oracle (a few positions of the long calls),
    and twice the same bits."""
    g = np.random.default_rng(V + K)
    d = W.tv_inputs_numpy(N, K, V, dtype, 900 + K, noise=g.uniform(0.05, 2.0, N))
    tgt, drf = device_inputs(d)
    a = binding.tv_loss_fwd_bwd(tgt, drf, 0.8, mode, 0.5)
    b = binding.tv_loss_fwd_bwd(tgt, drf, 0.8, mode, 0.5)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    pos = np.unique(np.linspace(0, N - 1, min(N, 6)).astype(int))
    ref = oracle.tv_ref(W.to_float64(d["target"][pos], dtype), W.to_float64(d["draft"][pos], dtype),
                        float(np.float32(0.8)), MODES[mode], 0.5, want_grad=True)
    ref["scale"] = 0.5
    compare_tv(a[0], a[1], a[2], ref, dtype, positions=pos, loss_exact=len(pos) == N)
    # the total loss from the call's own overlaps
    al = a[1].cpu().numpy().astype(np.float64)
    total = 0.5 * chain_factors(al, MODES[mode])[1].sum()
    assert abs(float(a[0]) - total) <= 1e-5 * abs(total) + 1e-6 * N * K


@pytest.mark.parametrize("mode", ["e2e", "prod", "per_step"])
@pytest.mark.parametrize("N,K,V,dtype", [
    (1500, 3, 4097, W.BF16),      # so many positions of short rows that the passes that read twice take them
    (2000, 2, 1023, W.F32),
    (4096, 1, 16384, W.BF16),
    (70, 3, 4097, W.BF16),        # short rows of few positions: the single-read pass
    (500, 3, 32000, W.BF16),      # many positions of longer rows: the single-read pass
])
def test_short_rows(N, K, V, dtype, mode):
    """Either side of the rule that sends calls of many positions over short
    rows to the passes that read twice: sampled positions against the oracle."""
    d = W.tv_inputs_torch(N, K, V, dtype, 31, chunk=64)
    loss, ov, grad = binding.tv_loss_fwd_bwd(d["target"], d["draft"], 0.8, mode, 0.5)
    torch.cuda.synchronize()
    pos = np.unique(np.linspace(0, N - 1, 6).astype(int))
    pi = torch.as_tensor(pos, device="cuda")
    ref = oracle.tv_ref(host_logits(d["target"][pi], dtype), host_logits(d["draft"][pi], dtype),
                        float(np.float32(0.8)), MODES[mode], 0.5, want_grad=True)
    ref["scale"] = 0.5
    compare_tv(loss, ov, grad, ref, dtype, positions=pos, loss_exact=False)
    total = 0.5 * chain_factors(ov.cpu().numpy().astype(np.float64), MODES[mode])[1].sum()
    assert abs(float(loss) - total) <= 1e-5 * abs(total) + 1e-6 * N * K


@pytest.mark.parametrize("mode", ["e2e", "prod", "per_step"])
@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("V,first,count,masked", [
    (2048, 0, 4, False), (2052, 2048, 4, False),    # every logit one thread holds
    (40000, 0, 10240, False),                       # every logit of its first tiles
    (40000, 123, 1, True), (200000, 199999, 1, True),   # one NaN in a row masked but for a few tokens
])
@pytest.mark.parametrize("which", ["target", "draft"])
def test_single_read_nan_anywhere(which, V, first, count, masked, dtype, mode):
    """NaN logits wherever they stand, also where a thread holds nothing else:
    NaN in the position's loss, in the step's overlap and all of its gradient."""
    N, K = 3, 2
    d = W.tv_inputs_numpy(N, K, V, W.F32, 8)
    if masked:
        for x in (d["target"], d["draft"]):
            x[1, 0, : V - V // 4] = -np.inf
            if first >= V - V // 4:
                x[1, 0, V // 2:] = -np.inf
                x[1, 0, : 3000] = 0.5
    d[which][1, 0, first:first + count] = np.nan
    cast = torch.bfloat16 if dtype == W.BF16 else torch.float32
    tgt, drf = (torch.from_numpy(d[n]).cuda().to(cast) for n in ("target", "draft"))
    loss, ov, grad = binding.tv_loss_fwd_bwd(tgt, drf, 1.0, mode, 1.0)
    torch.cuda.synchronize()
    assert torch.isnan(loss).all() and torch.isnan(ov[1, 0]) and torch.isnan(grad[1, 0]).all()
    assert torch.isfinite(ov[0]).all() and torch.isfinite(ov[2]).all() and torch.isfinite(ov[1, 1])
    assert torch.isfinite(grad[0]).all() and torch.isfinite(grad[2]).all()
    assert torch.isnan(grad[1, 1]).all() if mode != "per_step" else torch.isfinite(grad[1, 1]).all()


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("which", ["target", "draft"])
@pytest.mark.parametrize("dtype,V", [(W.F32, 262144), (W.BF16, 5000), (W.BF16, 600001)])
def test_two_read_data_errors(dtype, V, which, bad):
    """The passes that read the logits twice (forward-only calls, and gradient
    calls whose positions span too many slices): a NaN or infinite logit of
    either row makes the loss, the step's overlap and all of its gradient NaN."""
    N, K = 2, 8
    d = W.tv_inputs_numpy(N, K, V, W.F32, 9)
    d[which][1, 0, V // 3] = bad
    cast = torch.bfloat16 if dtype == W.BF16 else torch.float32
    tgt, drf = (torch.from_numpy(d[n]).cuda().to(cast) for n in ("target", "draft"))
    for mode in ("e2e", "per_step"):
        for want_grad in (False, True):
            loss, ov, grad = binding.tv_loss_fwd_bwd(tgt, drf, 1.0, mode, 1.0, want_grad=want_grad)
            torch.cuda.synchronize()
            assert torch.isnan(loss).all() and torch.isnan(ov[1, 0]), (mode, want_grad)
            assert torch.isfinite(ov[0]).all() and torch.isfinite(ov[1, 1:]).all()
            if want_grad:
                assert torch.isnan(grad[1, 0]).all() and torch.isfinite(grad[0]).all(), mode
                assert mode == "e2e" or torch.isfinite(grad[1, 1:]).all()


def test_single_read_data_errors():
    """NaN or infinite logits make that position's loss and gradient NaN."""
    for bad in (np.nan, np.inf):
        d = W.tv_inputs_numpy(3, 2, 4096, W.F32, 8)
        d["target"][1, 0, 77] = bad
        tgt, drf = device_inputs(d)
        loss, ov, grad = binding.tv_loss_fwd_bwd(tgt, drf, 1.0, "e2e", 1.0)
        torch.cuda.synchronize()
        assert torch.isnan(loss).all() and torch.isnan(ov[1, 0]) and torch.isnan(grad[1]).all()
        assert torch.isfinite(grad[0]).all() and torch.isfinite(grad[2]).all() and torch.isfinite(ov[0]).all()


def test_single_read_graph_replays():
    """A captured gradient call gives the eager results on every replay (the
    launches reset their own counters and records), with eager calls and other
    inputs in between."""
    N, K, V = 70, 2, 90000
    d = [W.tv_inputs_numpy(N, K, V, W.BF16, 40 + i) for i in range(2)]
    dev = [device_inputs(x) for x in d]
    eager = [binding.tv_loss_fwd_bwd(t, q, 1.0, "e2e", 0.5) for t, q in dev]
    tgt, drf = dev[0][0].clone(), dev[0][1].clone()
    ws = torch.empty(binding.tv_workspace_size(N, K, V), dtype=torch.uint8, device="cuda")
    grad = torch.empty((N, K, V), device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        loss, ov, _ = binding.tv_loss_fwd_bwd(tgt, drf, 1.0, "e2e", 0.5, ws=ws, grad_out=grad)
    for i in (0, 1, 0, 0, 1):
        tgt.copy_(dev[i][0])
        drf.copy_(dev[i][1])
        grad.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for got, want in zip((loss, ov, grad), eager[i]):
            assert torch.equal(got, want)
        binding.tv_loss_fwd_bwd(*dev[1 - i], 1.0, "e2e", 0.5)


def test_single_read_two_streams():
    """Calls on two streams at once, each with its own workspace: whichever
    workgroups the device holds, every group finishes, with the same bits."""
    N, K, V = 400, 3, 100000
    d = W.tv_inputs_torch(N, K, V, W.BF16, 51, chunk=64)
    want = binding.tv_loss_fwd_bwd(d["target"], d["draft"], 1.0, "prod", 1.0)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    ws = [torch.empty(binding.tv_workspace_size(N, K, V), dtype=torch.uint8, device="cuda") for _ in streams]
    outs = [[], []]
    for _ in range(3):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                outs[i].append(binding.tv_loss_fwd_bwd(d["target"], d["draft"], 1.0, "prod", 1.0, ws=ws[i]))
    torch.cuda.synchronize()
    for o in outs[0] + outs[1]:
        for got, ref in zip(o, want):
            assert torch.equal(got, ref)


@pytest.mark.parametrize("N,K,V,dtype", [
    (70, 3, 100000, W.BF16),      # slices that exchange statistics
    (300, 2, 30001, W.BF16),      # one slice a row, several positions a group
    (40, 1, 8000, W.BF16),        # a group of one workgroup
    (60, 3, 60001, W.F32),
    (5, 8, 4 * 19 * 2048, W.F32),
])
@pytest.mark.parametrize("waits", [
    (0, 0, 0, 1 << 20, 0xFFFFFFFF),   # every group but the first gives up
    (0, 0, 0, 1 << 20, 1),            # every other group
    (0, 0, 0, 1 << 20, 0),            # groups that are not complete at the first look
    (1, 3, 1, 1 << 20, 0xFFFFFFFE),   # after a few looks: pairs of groups but the first
    (0, 1 << 18, 256, 0, 0),          # complete groups whose records do not come: the loss is NaN
])
def test_single_read_groups_that_give_up(waits, N, K, V, dtype):
    """Position groups that cannot wait for their workgroups (the waits' polls
    are cut short, and whole groups never count as complete): the finish
    launch computes their positions, the bits of the undisturbed call.  The
    second call reuses the first one's workspace."""
    d = W.tv_inputs_torch(N, K, V, dtype, 77, chunk=64)
    tgt, drf = d["target"], d["draft"]
    want = binding.tv_loss_fwd_bwd(tgt, drf, 0.9, "e2e", 0.5)
    lib = binding.load_library()
    call = lib.spec_internal_tv_loss_waits
    call.argtypes = binding.TV_ARGTYPES + [ctypes.POINTER(ctypes.c_uint)]
    ws = torch.empty(binding.tv_workspace_size(N, K, V, tgt.dtype), dtype=torch.uint8, device="cuda")
    loss = torch.empty(1, device="cuda")
    ov = torch.empty((N, K), device="cuda")
    grad = torch.empty((N, K, V), device="cuda")
    w = (ctypes.c_uint * 5)(*waits)
    for _ in range(2):
        for x in (loss, ov, grad):
            x.fill_(7.0)
        st = call(tgt.data_ptr(), tgt.stride(0), tgt.stride(1), drf.data_ptr(), drf.stride(0), drf.stride(1),
                  binding.SPEC_BF16 if dtype == W.BF16 else binding.SPEC_F32, N, K, V, 0.9, 0, 0.5, loss.data_ptr(),
                  ov.data_ptr(), grad.data_ptr(), ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream, w)
        torch.cuda.synchronize()
        assert st == 0
        if waits[3] == 0:
            assert torch.isnan(loss).all()
            continue
        for got, ref in zip((loss, ov, grad), want):
            assert torch.equal(got, ref)


def test_single_read_sums_of_a_dominant_token():
    """Equal rows of one dominant token, first in its thread's sum, over a flat
    tail whose terms t = 1.19e-8 are below half a unit in the last place of its
    share, in calls of so many positions that a thread sums 152 elements.  The
    overlap is 1; float32 sums of at most 64 elements lose at most 63 t =
    7.5e-7 of it, less the 37 t that the normaliser's sums of 38 lose, plus the
    rounding of the result (one sum of 152 is 1.35e-6 off)."""
    N, V = 256, 38 * 2048
    z = torch.zeros((N, 1, V), dtype=torch.bfloat16, device="cuda")
    z[:, :, 0] = 18.25
    loss, ov, grad = binding.tv_loss_fwd_bwd(z, z, 1.0, "per_step", 1.0)
    torch.cuda.synchronize()
    err = float((ov.double() - 1.0).abs().max())
    assert err < 9e-7, err
