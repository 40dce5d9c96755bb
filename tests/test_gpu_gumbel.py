"""GPU parity of spec_verify_gumbel and spec_sample_gumbel against the
float64 oracle (App. G.2, Alg. rs_gumbel), through the C ABI."""

import numpy as np
import pytest
import torch
from scipy import stats

import oracle
from oracle.gumbel import sample_gumbel_ref, verify_gumbel_ref
from paper_2606_12370_amd import binding
from paper_2606_12370_amd import workloads as W
from tests.parity import compare_sample_gumbel, compare_verify_gumbel, device_inputs, host_logits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    binding.load_library()
    yield
    torch.cuda.synchronize()


def run_case(d, seed=0, offset=0, T=None, want_overlap=True):
    tgt, drf = device_inputs(d)
    ids = torch.from_numpy(d["ids"]).cuda()
    if T is None:
        Tg, Tr = torch.from_numpy(d["temperature"]).cuda(), d["temperature"].astype(np.float64)
    else:
        Tg, Tr = float(T), float(np.float32(T))
    out = binding.verify(tgt, drf, ids, Tg, seed, offset, want_debug=True, want_overlap=want_overlap, gumbel=True)
    torch.cuda.synchronize()
    ref = verify_gumbel_ref(W.to_float64(d["target"], d["dtype"]), W.to_float64(d["draft"], d["dtype"]), d["ids"],
                            Tr, seed, offset)
    return out, ref


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("B,K,V", [(4, 1, 1024), (6, 3, 20000), (3, 2, 2049), (5, 1, 1023), (4, 4, 7), (3, 1, 1),
                                   (2, 8, 9000), (3, 3, 65536 + 24), (2, 2, 256 * 8192 + 8195)])
def test_verify_gumbel_ragged(dtype, B, K, V):
    d = W.verify_inputs_numpy(B, K, V, dtype, "rollout_t", 500 + B + K + V)
    out, ref = run_case(d, seed=19, offset=4)
    print(dtype, B, K, V, compare_verify_gumbel(out, ref, dtype))


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
def test_verify_gumbel_without_overlap(dtype):
    d = W.verify_inputs_numpy(24, 3, 50000, dtype, "rollout_t", 78)
    full, ref = run_case(d, seed=6, offset=1)
    lean, _ = run_case(d, seed=6, offset=1, want_overlap=False)
    assert "overlap" not in lean
    for k in lean:
        assert torch.equal(full[k], lean[k]), k
    compare_verify_gumbel(lean, ref, dtype)


def test_verify_gumbel_chi_square_and_tempered_bonus():
    cfg = W.CONFIGS["exact_f32_b65536_k1_v8"]
    d = W.verify_inputs_numpy(cfg["B"], 1, 8, W.F32, "exact", cfg["seed"], shared_target=True)
    out, ref = run_case(d, seed=321)
    print("shared", compare_verify_gumbel(out, ref, W.F32))
    p, _ = oracle.softmax_t(d["target"][0, 0].astype(np.float64), 1.0)
    counts = np.bincount(out["emitted"][:, 0].cpu().numpy(), minlength=8)
    pval = stats.chisquare(counts, p * counts.sum()).pvalue
    print("first token chi-square p-value", pval)
    assert pval > 1e-3
    d = W.verify_inputs_numpy(cfg["B"], 1, 8, W.F32, "exact", cfg["seed"] + 1, shared_target=True, q_equals_p=True)
    out, ref = run_case(d, seed=5, T=0.6)
    compare_verify_gumbel(out, ref, W.F32)
    assert bool((out["accept_len"] == 1).all())
    p1, _ = oracle.softmax_t(d["target"][0, 1].astype(np.float64), float(np.float32(0.6)))
    counts = np.bincount(out["emitted"][:, 1].cpu().numpy(), minlength=8)
    pval = stats.chisquare(counts, p1 * counts.sum()).pvalue
    print("bonus chi-square p-value", pval)
    assert pval > 1e-3


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
def test_verify_gumbel_row_errors(dtype):
    d = W.verify_inputs_numpy(8, 2, 3000, dtype, "rollout", 10)
    tgt = W.to_float64(d["target"], dtype).astype(np.float32)
    drf = W.to_float64(d["draft"], dtype).astype(np.float32)
    tgt[0, 1, 3] = np.nan
    drf[1, 0, 0] = np.inf
    tgt[2, 2, :] = -np.inf
    d["ids"][3, 1] = 3000
    d["temperature"][4] = 0.0
    tgt[5, 0, :100] = -np.inf
    d["ids"][6, 0] = -1
    d["target"] = W.f32_to_bf16_bits(tgt) if dtype == W.BF16 else tgt
    d["draft"] = W.f32_to_bf16_bits(drf) if dtype == W.BF16 else drf
    out, ref = run_case(d)
    assert list(ref["row_error"]) == [True, True, True, True, True, False, True, False]
    compare_verify_gumbel(out, ref, dtype)


def test_verify_gumbel_benchmark_batch_sampled_rows():
    cfg = W.CONFIGS["verify_bf16_b256_k3_v151936"]
    d = W.verify_inputs_torch(cfg["B"], cfg["K"], cfg["V"], cfg["dtype"], cfg["gen"], cfg["seed"])
    out = binding.verify(d["target"], d["draft"], d["ids"], d["temperature"], 3, 0, want_debug=True, gumbel=True)
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(4).choice(cfg["B"], size=24, replace=False))
    ri = torch.as_tensor(rows, device="cuda")
    ref = verify_gumbel_ref(host_logits(d["target"][ri], W.BF16), host_logits(d["draft"][ri], W.BF16),
                            d["ids"][ri].cpu().numpy(), d["temperature"][ri].cpu().numpy().astype(np.float64), 3, 0,
                            rows=rows)
    print(compare_verify_gumbel(out, ref, W.BF16, rows=rows))


# ----------------------------------------------------------------------------
# Gumbel-max draft sampler

def _store(x32, dtype):
    return W.f32_to_bf16_bits(x32) if dtype == W.BF16 else np.ascontiguousarray(x32, np.float32)


def _dev(arr, dtype):
    if dtype == W.BF16:
        return torch.from_numpy(np.ascontiguousarray(arr).view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(arr)).cuda()


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("R,V", [(40, 1024), (9, 20000), (17, 2049), (5, 7), (4, 1), (6, 65536 + 24),
                                 (2, 256 * 8192 + 8195)])
def test_sample_gumbel_ragged(dtype, R, V):
    rng = np.random.default_rng(R * 7 + V)
    z = _store((rng.standard_normal((R, V)) * rng.uniform(1, 8, size=(R, 1))).astype(np.float32), dtype)
    T = rng.uniform(0.6, 1.2, size=R).astype(np.float32)
    T[::4] = 0.0
    out = binding.sample_gumbel(_dev(z, dtype), torch.from_numpy(T).cuda(), 41, 2)
    torch.cuda.synchronize()
    ref = sample_gumbel_ref(W.to_float64(z, dtype), T.astype(np.float64), 41, 2)
    print(dtype, R, V, compare_sample_gumbel(out["tokens"], ref))


def test_sample_gumbel_chi_square_errors_and_strides():
    B, V = 65536, 8
    z = np.broadcast_to(np.linspace(-2, 1.5, V).astype(np.float32), (B, V)).copy()
    z[:, 4] = -np.inf
    out = binding.sample_gumbel(torch.from_numpy(z).cuda(), 0.8, 7)
    torch.cuda.synchronize()
    ref = sample_gumbel_ref(z.astype(np.float64), float(np.float32(0.8)), 7)
    compare_sample_gumbel(out["tokens"], ref)
    counts = np.bincount(out["tokens"].cpu().numpy(), minlength=V)
    p = np.exp(z[0].astype(np.float64) / np.float64(np.float32(0.8)))
    pval = stats.chisquare(counts[p > 0], (p / p.sum() * B)[p > 0]).pvalue
    print("chi-square p-value", pval)
    assert pval > 1e-3 and counts[4] == 0
    zz = np.zeros((6, 40000), np.float32)
    zz[0, [5, 20000, 39999]] = 3.0
    zz[1, 100] = np.nan
    zz[2, :] = -np.inf
    zz[3, 7] = np.inf
    T = np.array([0, 1, 1, 1, -1, 0.5], np.float32)
    out = binding.sample_gumbel(torch.from_numpy(zz).cuda(), torch.from_numpy(T).cuda(), 3)
    torch.cuda.synchronize()
    tok = out["tokens"].cpu().numpy()
    assert list(tok[:5]) == [5, -1, -1, -1, -1] and tok[5] >= 0
    ref = sample_gumbel_ref(zz.astype(np.float64), T.astype(np.float64), 3)
    compare_sample_gumbel(out["tokens"], ref)
    R, V2 = 11, 3001
    x = (np.random.default_rng(5).standard_normal((R, V2)) * 3).astype(np.float32)
    big = torch.zeros((R, V2 + 5), dtype=torch.float32, device="cuda")
    big[:, 1:V2 + 1] = torch.from_numpy(x).cuda()
    out = binding.sample_gumbel(big[:, 1:V2 + 1], 1.1, 8)
    torch.cuda.synchronize()
    compare_sample_gumbel(out["tokens"], sample_gumbel_ref(x.astype(np.float64), float(np.float32(1.1)), 8))


def test_sample_gumbel_benchmark_draft_rows():
    cfg = W.CONFIGS["verify_bf16_b256_k3_v151936"]
    d = W.verify_inputs_torch(cfg["B"], cfg["K"], cfg["V"], cfg["dtype"], cfg["gen"], cfg["seed"])
    flat = d["draft"].reshape(-1, cfg["V"])
    T = d["temperature"].repeat_interleave(cfg["K"]).contiguous()
    out = binding.sample_gumbel(flat, T, 9, 4)
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(3).choice(flat.shape[0], size=32, replace=False))
    ri = torch.as_tensor(rows, device="cuda")
    ref = sample_gumbel_ref(host_logits(flat[ri], W.BF16), T[ri].cpu().numpy().astype(np.float64), 9, 4, rows=rows)
    print(compare_sample_gumbel(out["tokens"], ref, rows=rows))


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("V", [5, 8, 2047, 2048, 2056, 16384 + 8, 50001])
def test_sampler_scan_bounds(V, dtype):
    """Rows whose elements mostly need no variate (one or a few logits far
    above the rest, at either end of the row), rows where every element does,
    masked rows, equal logits and large scales, at the edges of the scan's
    blocks and parts: the tokens of the oracle, which draws every variate."""
    R = 24
    rng = np.random.default_rng(V)
    z = rng.standard_normal((R, V)).astype(np.float32)
    z[0:4] *= 8.0
    z[4, V - 1] = 30.0
    z[5, 0] = 30.0
    z[6, V // 2] = 18.0
    z[7, :] = 1.5                                  # all equal
    z[8, : V // 2] = -np.inf                       # masked halves
    z[9, V // 2:] = -np.inf
    z[10, 1:] = -np.inf                            # one token left
    z[11] *= 1000.0
    z[12] = z[12] * 0.01 + 300.0
    z[13] = z[13] * 0.01 - 300.0
    z[14, V - 1] = np.nan
    z[15, V // 3] = np.inf
    z[16, :] = -np.inf
    T = np.ones(R, np.float32)
    T[17] = 0.05
    T[18] = 20.0
    T[19] = 0.0
    d = W.f32_to_bf16_bits(z) if dtype == W.BF16 else z
    lg = torch.from_numpy(d.view(np.int16)).cuda().view(torch.bfloat16) if dtype == W.BF16 else torch.from_numpy(d).cuda()
    pad = torch.zeros((R, V + 9), dtype=lg.dtype, device="cuda")
    pad[:, 1:V + 1] = lg
    out = binding.sample_gumbel(lg, torch.from_numpy(T).cuda(), seed=11, offset=3)["tokens"]
    odd = binding.sample_gumbel(pad[:, 1:V + 1], torch.from_numpy(T).cuda(), seed=11, offset=3)["tokens"]
    torch.cuda.synchronize()
    ref = sample_gumbel_ref(W.to_float64(d, dtype), T.astype(np.float64), 11, 3)
    compare_sample_gumbel(out, ref)
    assert torch.equal(out, odd)


@pytest.mark.parametrize("V", [9, 2 * 2048, 2 * 2048 + 3, 40000])
def test_verify_scan_parts_without_residual_mass(V):
    """Rejected steps whose residual has mass in one half of the row only (the
    draft holds nearly all of its mass in the other), so that the parts of
    the other half fall back to p_n and must not win."""
    B, K = 32, 2
    rng = np.random.default_rng(V + 1)
    tgt = rng.standard_normal((B, K + 1, V)).astype(np.float32) * 3
    drf = tgt[:, :K].copy()
    half = V // 2
    drf[: B // 2, :, half:] += 20.0
    drf[B // 2:, :, :half] += 20.0
    ids = rng.integers(0, half, (B, K)).astype(np.int32)
    ids[: B // 2] += V - half
    T = np.ones(B, np.float32)
    out = binding.verify(torch.from_numpy(tgt).cuda(), torch.from_numpy(drf).cuda(), torch.from_numpy(ids).cuda(),
                         torch.from_numpy(T).cuda(), seed=4, offset=1, gumbel=True)
    torch.cuda.synchronize()
    ref = verify_gumbel_ref(tgt.astype(np.float64), drf.astype(np.float64), ids, T.astype(np.float64), 4, 1)
    assert (ref["accept_len"] < K).sum() >= B // 4  # rejections to look at
    print(compare_verify_gumbel(out, ref, W.F32))


@pytest.mark.parametrize("R,V", [(96, 4 * 16384), (97, 4 * 16384), (384, 4100), (3, 16384 + 1)])
def test_sampler_parts_rule(R, V):
    """Either side of the calls whose rows are scanned in half chunks, and rows
    with fewer tiles than such parts: the tokens of the oracle."""
    g = torch.Generator(device="cuda")
    g.manual_seed(R + V)
    z = torch.randn((R, V), device="cuda", generator=g) * torch.linspace(0.5, 8.0, R, device="cuda")[:, None]
    out = binding.sample_gumbel(z, 0.9, seed=5, offset=7)["tokens"]
    torch.cuda.synchronize()
    rows = np.unique(np.linspace(0, R - 1, 12).astype(int))
    ref = sample_gumbel_ref(z[torch.as_tensor(rows, device="cuda")].cpu().numpy().astype(np.float64),
                            np.full(len(rows), float(np.float32(0.9))), 5, 7, rows=rows)
    compare_sample_gumbel(out, ref, rows=rows)


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("V", [5, 2049, 40000])
def test_sampler_overflowing_scale(V, dtype):
    """Finite logits whose z / T overflows float32 (a token forced with the
    largest finite value; a tiny temperature) are no data error: the row's
    token is that of the oracle.  NaN and +inf logits stay one at any T."""
    R = 12
    top = float(np.finfo(np.float32).max) if dtype == W.F32 else float(np.float32(2.0 ** 128 - 2.0 ** 120))
    rng = np.random.default_rng(V)
    z = -np.abs(rng.standard_normal((R, V))).astype(np.float32) - 1.0
    T = np.ones(R, np.float32)
    z[0, V - 1] = top
    z[1, 0] = top
    z[2, V // 2], T[2] = top, 0.25
    z[3, V // 2], T[3] = top, 20.0                 # no overflow
    z[4, V // 3], T[4] = 300.0, 1e-37              # ordinary logits, a tiny temperature
    z[5, V // 3], T[5] = 300.0, 1e-37
    z[5, V - 1] = np.nan
    z[6, V // 3], T[6] = 300.0, 1e-37
    z[6, 0] = np.inf
    z[7, V - 1], z[7, 1] = top, np.nan
    z[8, V - 1], z[8, 1] = top, np.inf
    z[9, V - 1], z[9, : V // 2] = top, -np.inf
    z[10, : V - 1], z[10, V - 1] = -np.inf, top
    d = W.f32_to_bf16_bits(z) if dtype == W.BF16 else z
    lg = torch.from_numpy(d.view(np.int16)).cuda().view(torch.bfloat16) if dtype == W.BF16 else torch.from_numpy(d).cuda()
    out = binding.sample_gumbel(lg, torch.from_numpy(T).cuda(), seed=21, offset=2)["tokens"]
    torch.cuda.synchronize()
    ref = sample_gumbel_ref(W.to_float64(d, dtype), T.astype(np.float64), 21, 2)
    assert ref["token"][0] == V - 1 and ref["token"][1] == 0 and (ref["token"][5:9] == -1).all()
    compare_sample_gumbel(out, ref)


@pytest.mark.parametrize("B,V,top", [(1024, 262144, 0.99), (2048, 262144, 0.995), (1024, 1 << 21, 0.9)])
def test_overlap_of_the_emitting_step_long_parts(B, V, top):
    """Calls of so many rows that one workgroup scans a whole row: the
    overlap of the rejected step, one dominant token over a flat tail whose
    terms are about half a unit in the last place of the dominant one's share.
    Bound: the row statistics and the overlap each sum 64 elements a lane in
    float32, 63 * 2^-24 = 3.8e-6 at worst, the probabilities' rounding adds
    2e-7.  One float32 sum over the row's 1024 and more elements per thread is
    1.8e-5 and more off.
    The rows of the batch share one row's storage (stride 0)."""
    p = np.full(V, (1.0 - top) / (V - 1))
    p[0] = top
    q = 0.5 * p
    q[7] += 0.5
    z = torch.from_numpy(np.log(np.stack([p, p, q])).astype(np.float32)).cuda()
    tgt = z[:2].unsqueeze(0).expand(B, 2, V)
    drf = z[2:].unsqueeze(0).expand(B, 1, V)
    ids = torch.full((B, 1), 7, dtype=torch.int32, device="cuda")
    out = binding.verify(tgt, drf, ids, 1.0, seed=3, offset=1, gumbel=True)
    torch.cuda.synchronize()
    s = torch.softmax(z.double(), -1)
    want = float(torch.minimum(s[0], s[2]).sum())
    ov = out["overlap"].double()[:, 0]
    rejected = out["accept_len"] == 0
    assert int(rejected.sum()) > B // 2
    err = float((ov[rejected] - want).abs().max()) / want
    assert err < 8e-6, err
