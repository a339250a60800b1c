"""GPU parity: the HIP path through the C ABI against the binary64 oracle, on
the same seeded inputs.  KV append is compared byte for byte over the whole
pools; attention within max-abs 1e-2 / rel-L2 2e-3 (bf16 KV) and 3e-2 / 1e-2
(fp8 KV), element by element over whole outputs: every step of the
Llama-3-8B-shaped run, and the full-size summarization (uncapped and capped)
and fp8 stress batches at several steps, in the launch configuration the
benchmark times; plus properties that hold at any size."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from tests import _dense as dn
from tests import _gpu as G

pytestmark = pytest.mark.gpu

bl = pytest.importorskip("paper_2510_15330_amd")
from paper_2510_15330_amd import workloads as wl  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    bl.library()
    yield
    torch.cuda.synchronize()


def dev_case(case, kv="bf16"):
    """Device tensors of a tests._dense.random_case."""
    if kv == "bf16":
        kp = torch.from_numpy(case["k_pages"].view(np.int16)).view(torch.bfloat16)
        vp = torch.from_numpy(case["v_pages"].view(np.int16)).view(torch.bfloat16)
    else:
        kp = torch.from_numpy(case["k_pages"])
        vp = torch.from_numpy(case["v_pages"])
    d = dict(
        q=torch.from_numpy(case["q_bits"].view(np.int16)).view(torch.bfloat16).cuda(),
        k=kp.cuda(), v=vp.cuda(),
        bt=torch.from_numpy(case["block_table"]).cuda(),
        sl=torch.from_numpy(case["seq_lens"]).cuda(),
        ks=None if case["k_scale"] is None else torch.from_numpy(case["k_scale"]).cuda(),
        vs=None if case["v_scale"] is None else torch.from_numpy(case["v_scale"]).cuda(),
    )
    B, H_q, D = case["q_bits"].shape
    d["out"] = torch.full((B, H_q, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    return d


def run_case(d, scale, **kw):
    bl.decode_attention(d["q"], d["k"], d["v"], d["bt"], d["sl"], scale, d["out"],
                        k_scale=d["ks"], v_scale=d["vs"], **kw)
    torch.cuda.synchronize()
    return G.out_f64(d["out"])


def oracle_case(case, scale, kv="bf16"):
    return oracle.decode_attention(case["q_bits"], case["k_pages"], case["v_pages"], case["block_table"],
                                   case["seq_lens"], scale, G.kv_code(kv), case["k_scale"], case["v_scale"])


# ------------------------------------------------------------ tiny config ---

@pytest.mark.parametrize("reading", ["after", "before"])
def test_tiny_append_bitexact_and_attention(reading):
    w = G.to_device(wl.build("tiny", seed=0, tiny_reading=reading))
    # oracle side: host copies of the initial state
    kp, vp = G.bits16(w.k_pages), G.bits16(w.v_pages)
    sl = w.seq_lens.cpu().numpy().astype(np.int32)
    oracle.kv_append(G.bits16(w.k_new[0]), G.bits16(w.v_new[0]), kp, vp, w.block_table.cpu().numpy(), sl)
    out = torch.full((w.B, w.H_q, w.D), float("nan"), dtype=torch.bfloat16, device="cuda")
    print(f"tiny reading={reading} lens0={list(w.lens0)}", flush=True)
    G.gpu_step(w, 0, out)
    torch.cuda.synchronize()
    assert bl.device_errors() == 0
    assert np.array_equal(w.seq_lens.cpu().numpy(), sl)
    assert np.array_equal(G.bits16(w.k_pages), kp)
    assert np.array_equal(G.bits16(w.v_pages), vp)
    ref = oracle.decode_attention(G.bits16(w.q[0]), kp, vp, w.block_table.cpu().numpy(), sl, w.scale)
    G.assert_close(G.out_f64(out), ref, "bf16", f"tiny/{reading}")
    if reading == "after":
        # the length-1 request returns its only V row exactly
        v_row = ref[0]
        assert np.array_equal(G.out_f64(out)[0], v_row)


@pytest.mark.parametrize("depth", [1, 2])
@pytest.mark.parametrize("pps", [1, 2])
@pytest.mark.parametrize("waves", [1, 2, 3, 7, 64, 5000])
def test_tiny_wave_counts(waves, pps, depth):
    """Different wave counts cut the requests at different pages (the 16+17+
    200-token batch has 32 (page, head) units, so 64 and 5000 waves leave
    most waves without work); every cut must merge back to the oracle."""
    w = G.to_device(wl.build("tiny", seed=1))
    out = torch.full((w.B, w.H_q, w.D), float("nan"), dtype=torch.bfloat16, device="cuda")
    G.gpu_step(w, 0, out, max_waves=waves, pages_per_step=pps, pipeline_depth=depth)
    torch.cuda.synchronize()
    ref = G.oracle_full(w, 0)
    G.assert_close(G.out_f64(out), ref, "bf16", f"waves={waves} pages/step={pps}")


# ------------------------------------------------------ llama3-8b config ---

def test_llama3_8b_steps():
    w = G.to_device(wl.build("llama3_8b", seed=0))
    kp, vp = G.bits16(w.k_pages), G.bits16(w.v_pages)
    sl = w.seq_lens.cpu().numpy().astype(np.int32)
    bt = w.block_table.cpu().numpy()
    out = torch.empty((w.B, w.H_q, w.D), dtype=torch.bfloat16, device="cuda")
    for step in range(w.steps):
        # every step: the whole output against the oracle on the host pools,
        # which the oracle's own append advances in lockstep
        G.gpu_step(w, step, out)
        oracle.kv_append(G.bits16(w.k_new[step]), G.bits16(w.v_new[step]), kp, vp, bt, sl)
        torch.cuda.synchronize()
        ref = oracle.decode_attention(G.bits16(w.q[step]), kp, vp, bt, sl, w.scale)
        G.assert_close(G.out_f64(out), ref, "bf16", f"llama3_8b step {step}")
    torch.cuda.synchronize()
    assert bl.device_errors() == 0
    assert np.array_equal(w.seq_lens.cpu().numpy(), sl)
    assert np.array_equal(G.bits16(w.k_pages), kp), "K pool differs after 100 appends"
    assert np.array_equal(G.bits16(w.v_pages), vp), "V pool differs after 100 appends"


# ------------------------------------------------- full-size, whole batch ---

@pytest.mark.parametrize("name", ["summarization", "summarization_capped", "stress_fp8"])
def test_full_size_whole_batch(name):
    """The full-size batches, stepped as the benchmark steps them (append +
    attention, default launch configuration): every output element against
    the oracle over the whole pools, at the first, middle and last of the
    summarization batches' 50 steps and at both steps of a two-step fp8
    stress run."""
    steps = wl.CONFIGS[name]["steps"] if name.startswith("summarization") else 2
    check = {0, steps // 2, steps - 1}
    w = wl.build(name, seed=0, device="cuda", steps=steps)
    out = torch.full((w.B, w.H_q, w.D), float("nan"), dtype=torch.bfloat16, device="cuda")
    L0 = w.seq_lens.cpu().numpy().copy()
    print(f"{name}: B={w.B} pages={w.num_pages} mean L={w.lens0.mean():.0f} steps={steps}", flush=True)
    for step in range(steps):
        G.gpu_step(w, step, out)
        if step in check:
            torch.cuda.synchronize()
            assert bl.device_errors() == 0
            got = G.out_f64(out)
            ref = G.oracle_full(w, step)
            G.assert_close(got, ref, w.kv, f"{name} step {step}, all {w.B} requests")
    torch.cuda.synchronize()
    assert np.array_equal(w.seq_lens.cpu().numpy(), L0 + steps)


# ------------------------------------------------------------ invariants ---

def test_page_permutation_and_determinism_bitexact():
    rng = np.random.default_rng(21)
    lens = [300, 17, 1000, 64]
    case = dn.random_case(rng, 4, 32, 8, 128, lens)
    d = dev_case(case)
    a = run_case(d, 0.088, max_waves=5)
    b = run_case(d, 0.088, max_waves=5)
    assert np.array_equal(a, b), "run-to-run differs"
    perm = rng.permutation(case["num_pages"]).astype(np.int32)
    kp = np.empty_like(case["k_pages"])
    vp = np.empty_like(case["v_pages"])
    kp[perm] = case["k_pages"]
    vp[perm] = case["v_pages"]
    bt = case["block_table"].copy()
    bt[bt >= 0] = perm[bt[bt >= 0]]
    d2 = dev_case(dict(case, k_pages=kp, v_pages=vp, block_table=bt))
    c = run_case(d2, 0.088, max_waves=5)
    assert np.array_equal(a, c), "page permutation changed the output"
    # With one wave and the same pages per step (the library's default
    # depends on the table's size), no request is cut, so a request alone
    # equals the same request inside the batch bit for bit; with many waves
    # the cuts depend on the batch and the results agree within rounding.
    single = run_case(d, 0.088, max_waves=1, pages_per_step=2)
    for bi in range(4):
        sub = dict(case, q_bits=case["q_bits"][bi:bi + 1], block_table=case["block_table"][bi:bi + 1],
                   seq_lens=case["seq_lens"][bi:bi + 1])
        one = run_case(dev_case(sub), 0.088, max_waves=1, pages_per_step=2)
        assert np.array_equal(one[0], single[bi]), f"batch independence b={bi}"
    ref = oracle_case(case, 0.088)
    G.assert_close(a, ref, "bf16", "invariant case, 5 waves")
    G.assert_close(single, ref, "bf16", "invariant case, 1 wave")


def test_closed_forms_exact():
    rng = np.random.default_rng(22)
    lens = [1, 40, 700]
    case = dn.random_case(rng, 3, 8, 2, 128, lens)
    # constant V rows (per head) and a ones column in V dim 3
    cv = torch.from_numpy(rng.standard_normal((3, 2, 128)).astype(np.float32)).to(torch.bfloat16)
    cv = cv.view(torch.int16).numpy().view(np.uint16)
    one = np.uint16(0x3F80)
    for b in range(3):
        case["dense_v"][b][:] = cv[b][None]
        case["dense_v"][b][:, :, 3] = one
    kp, vp = dn.write_pools(case["dense_k"], case["dense_v"], lens, case["page_lists"], case["num_pages"],
                            2, 128, 8, np.uint16(0x7FC0))
    case.update(k_pages=kp, v_pages=vp)
    for waves, pps in ((1, 1), (8, 1), (0, 1), (1, 2), (8, 2), (0, 2)):
        got = run_case(dev_case(case), 0.088, max_waves=waves, pages_per_step=pps)
        for b in range(3):
            for h in range(8):
                ref = dn.bits_to_f64_bf16(cv[b][h // 4]).copy()
                ref[3] = 1.0
                assert np.array_equal(got[b, h], ref), f"constant V not exact b={b} h={h} waves={waves}"


@pytest.mark.parametrize("B,Hq,Hkv,D,lens,kv", [
    (3, 8, 8, 64, [5, 16, 33], "bf16"),          # G = 1
    (2, 16, 1, 128, [100, 1], "bf16"),           # G = 16
    (4, 4, 2, 64, [0, 1, 0, 47], "bf16"),        # empty requests
    (1, 32, 8, 128, [4096], "bf16"),             # B = 1, long
    (3, 64, 8, 128, [1, 129, 2000], "fp8"),      # fp8, G = 8
    (2, 8, 2, 64, [31, 320], "fp8"),             # fp8, D = 64
])
def test_edge_shapes(B, Hq, Hkv, D, lens, kv):
    rng = np.random.default_rng(sum(lens) + D)
    case = dn.random_case(rng, B, Hq, Hkv, D, lens, kv)
    scale = float(np.float32(1.0 / np.sqrt(D)))
    ref = oracle_case(case, scale, kv)
    for waves in (0, 1, 5, 13):
        for pps in ((1, 2, 4) if kv == "fp8" else (1, 2)):
            for depth in (1, 2):
                got = run_case(dev_case(case, kv), scale, max_waves=waves, pages_per_step=pps, pipeline_depth=depth)
                G.assert_close(got, ref, kv, f"edge {B},{Hq},{Hkv},{D},{lens},{kv} waves={waves} "
                                             f"pages/step={pps} depth={depth}")
        for b, L in enumerate(lens):
            if L == 0:
                assert np.all(got[b] == 0.0)


@pytest.mark.parametrize("kv", ["bf16", "fp8"])
def test_negative_zero_and_sharp_scales(kv):
    # the softmax scale is any finite number: negative (the scores' order
    # reverses), zero (uniform weights: the mean of the visible values) and
    # four times the usual 1/sqrt(D) (peaked weights).  Much sharper weights
    # make each output one value row, whose own bf16 rounding (half an ulp of
    # values up to ~11 in the fp8 case) alone reaches the max-abs bound.
    B, Hq, Hkv, D, lens = 3, 16, 2, 128, [1, 77, 900]
    rng = np.random.default_rng(4242)
    case = dn.random_case(rng, B, Hq, Hkv, D, lens, kv)
    s0 = float(np.float32(1.0 / np.sqrt(D)))
    for scale in (-s0, 0.0, 4 * s0):
        ref = oracle_case(case, scale, kv)
        for waves in (0, 7):
            got = run_case(dev_case(case, kv), scale, max_waves=waves)
            G.assert_close(got, ref, kv, f"scale {scale} {kv} waves={waves}")


def _sweep_lengths(rng, B):
    """Lengths that land on and next to page (16) and four-page (64) step
    boundaries, plus empty and one-token requests and arbitrary ones."""
    out = []
    for _ in range(B):
        kind = rng.integers(0, 6)
        k = int(rng.integers(1, 12))
        if kind == 0:
            out.append(int(rng.choice([0, 1])))
        elif kind == 1:
            out.append(16 * k + int(rng.integers(-1, 2)))
        elif kind == 2:
            out.append(64 * k + int(rng.integers(-1, 2)))
        else:
            out.append(int(rng.integers(1, 700)))
    return out


@pytest.mark.parametrize("seed", range(24))
def test_random_shapes_and_splits(seed):
    # seeded sweep over shapes, length mixes and wave caps: the planner deals
    # steps of 1, 2 or 4 pages, so cuts fall on step boundaries of requests
    # whose lengths sit on either side of page and step edges
    rng = np.random.default_rng(9000 + seed)
    kv = "fp8" if seed % 3 == 2 else "bf16"
    D = 64 if seed % 2 else 128
    H_kv = int(rng.choice([1, 2, 4, 8]))
    Gq = int(rng.choice([1, 2, 3, 4, 6, 8, 16]))
    B = int(rng.integers(1, 25))
    lens = _sweep_lengths(rng, B)
    case = dn.random_case(rng, B, Gq * H_kv, H_kv, D, lens, kv)
    if kv == "fp8":
        # codes are N(0, 40^2); scales near 1/40 give unit-scale values as in
        # the workloads.  The absolute bound is one for unit-scale data: above
        # |out| = 7.68 the bf16 rounding of the output alone (half an ulp,
        # 2^-9 |out|) would exceed 3e-2.
        case["k_scale"] = (rng.uniform(0.5, 1.5, size=(B, H_kv)) / 40.0).astype(np.float32)
        case["v_scale"] = (rng.uniform(0.5, 1.5, size=(B, H_kv)) / 40.0).astype(np.float32)
    scale = float(np.float32(1.0 / np.sqrt(D)))
    ref = oracle_case(case, scale, kv)
    for _ in range(3):
        waves = int(rng.choice([0, 1, 2, 3, 5, 8, 17, 33, 100]))
        pps = int(rng.choice([1, 2, 4] if kv == "fp8" else [1, 2]))
        depth = int(rng.choice([1, 2]))
        got = run_case(dev_case(case, kv), scale, max_waves=waves, pages_per_step=pps, pipeline_depth=depth)
        G.assert_close(got, ref, kv, f"sweep seed={seed} B={B} G={Gq} H_kv={H_kv} D={D} {kv} lens={lens} "
                                     f"waves={waves} pages/step={pps} depth={depth}")
        for b, L in enumerate(lens):
            if L == 0:
                assert np.all(got[b] == 0.0)


@pytest.mark.parametrize("kv,pps,depth", [("bf16", 2, 2), ("fp8", 4, 1)])
def test_long_shares_with_weighted_split(kv, pps, depth):
    # shares of 384 pages or more a wave take the even/odd-XCD weights (one
    # workgroup per CU at depth 2, two at depth 1), also with wave counts
    # that do not fill a period of eight
    rng = np.random.default_rng(8192)
    case = dn.random_case(rng, 2, 32, 8, 128, [8192, 3000], kv)
    if kv == "fp8":   # unit-sized values, where the absolute bound holds
        case["k_scale"] = (rng.uniform(0.5, 1.5, size=(2, 8)) / 40.0).astype(np.float32)
        case["v_scale"] = (rng.uniform(0.5, 1.5, size=(2, 8)) / 40.0).astype(np.float32)
    scale = float(np.float32(1.0 / np.sqrt(128)))
    ref = oracle_case(case, scale, kv)
    for waves in (1, 3, 5, 7, 9):
        got = run_case(dev_case(case, kv), scale, max_waves=waves, pages_per_step=pps, pipeline_depth=depth)
        G.assert_close(got, ref, kv, f"long shares waves={waves}")


@pytest.mark.parametrize("B,Hq,Hkv,D,lens,kv", [
    (1, 16, 1, 128, [3000], "bf16"),             # pieces of 8 slices, two waves a slice, several batches
    (2, 7, 1, 128, [2500, 9], "bf16"),           # pieces of 3.5 slices
    (3, 2, 1, 64, [300, 1, 700], "bf16"),        # a piece of half a slice; fewer units than waves
    (1, 8, 1, 128, [20000], "fp8"),
    (24, 64, 4, 128, [100 + 37 * i for i in range(24)], "bf16"),   # pieces of over 256 float4s: from 2 a cut on
    (24, 36, 4, 128, [100 + 37 * i for i in range(24)], "fp8"),
])
def test_requests_cut_over_many_waves(B, Hq, Hkv, D, lens, kv):
    # few (request, head)s, each cut over 8 waves' ranges or more: the merge
    # that deals a cut's pieces over the waves of a workgroup
    rng = np.random.default_rng(sum(lens))
    case = dn.random_case(rng, B, Hq, Hkv, D, lens, kv)
    scale = float(np.float32(1.0 / np.sqrt(D)))
    ref = oracle_case(case, scale, kv)
    for waves in (0, 700, 130, 17):
        got = run_case(dev_case(case, kv), scale, max_waves=waves)
        G.assert_close(got, ref, kv, f"many waves {B},{Hq},{Hkv},{D},{lens},{kv} waves={waves}")
    d = dev_case(case, kv)
    d["bt"][0, 3] = case["num_pages"] + 7        # one poisoned piece among the others
    bl.device_errors()
    got = run_case(d, scale)
    assert bl.device_errors() & 4
    assert np.all(np.isnan(got[0]))
    if B > 1:
        G.assert_close(got[1:], ref[1:], kv, "other requests")


def test_shares_left_empty_by_extreme_weights():
    # weight 511 : 1 over shares of 400 pages: some odd workgroups' waves get
    # no unit, and the merge skips their pieces
    rng = np.random.default_rng(77)
    case = dn.random_case(rng, 2, 32, 8, 128, [8192, 3008], "bf16")
    scale = float(np.float32(1.0 / np.sqrt(128)))
    got = run_case(dev_case(case), scale, max_waves=14, xcd_skew=255, pages_per_step=2)
    G.assert_close(got, oracle_case(case, scale), "bf16", "weights 511 : 1")


@pytest.mark.parametrize("Hq,D,edge", [(2, 64, 96), (18, 64, 126), (32, 64, 224), (8, 128, 3584), (18, 128, 3584)])
def test_fp8_workgroups_on_both_sides_of_the_rule(Hq, D, edge):
    # one workgroup a CU or two, by the table's pages a wave: the same results
    # within the bound on both sides of the line, and with empty columns
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    B, Hkv = 8, 2
    rng = np.random.default_rng(Hq + D)
    case = dn.random_case(rng, B, Hq, Hkv, D, [1, 0, 17, 900, 64, 2000, 333, 16], "fp8")
    # values below 8: from there on the output's own rounding to bf16 (2^-9 of
    # it, 0.031 at the value of one token) is over the bound on the largest error
    case["v_scale"] = (rng.uniform(0.5, 1.5, size=(B, Hkv)) * (5 / 448)).astype(np.float32)
    scale = float(np.float32(1.0 / np.sqrt(D)))
    ref = oracle_case(case, scale, "fp8")
    for width in (edge * 4 * cus // (B * Hkv) - 1, edge * 4 * cus // (B * Hkv)):
        d = dev_case(case, "fp8")
        d["bt"] = torch.nn.functional.pad(d["bt"], (0, width - d["bt"].shape[1]), value=-1)
        got = run_case(d, scale)
        assert bl.device_errors() == 0
        G.assert_close(got, ref, "fp8", f"D={D} G={Hq // Hkv} width={width}")


def test_nan_and_inf_shares_as_uncut():
    # keys of whole shares that are NaN in KV head 0, and over bf16 pools
    # score -inf in KV head 1: every cut gives what one wave gives (a NaN row
    # is NaN, a weight of -inf is 0 as the oracle has it), through both merges
    for B, lens in ((1, [6000]), (24, [6000] * 24)):
        for kv in ("bf16", "fp8"):
            rng = np.random.default_rng(B)
            case = dn.random_case(rng, B, 4, 2, 128, lens, kv)
            scale = float(np.float32(1.0 / np.sqrt(128)))
            d = dev_case(case, kv)
            d["q"][:, 2:, 0] = 1.0
            case["q_bits"] = G.bits16(d["q"])
            pages = torch.cat([d["bt"][:, lo:hi].reshape(-1) for lo, hi in ((0, 60), (128, 256))]).long()
            if kv == "fp8":
                d["k"][pages, 0] = 0x7F
            else:
                d["k"][pages, 0] = float("nan")
                d["k"][pages, 1, 0, :, 0] = -float("inf")
            case["k_pages"] = G.host_codes(d["k"], kv)
            ref = oracle_case(case, scale, kv)
            for waves in (1, 0, 37, 300):
                got = run_case(d, scale, max_waves=waves)
                assert np.isnan(got[:, :2]).all(), (B, kv, waves)
                G.assert_close(got[:, 2:], ref[:, 2:], kv, f"-inf shares B={B} {kv} waves={waves}")


@pytest.mark.parametrize("B,kv", [(2500, "bf16"), (8192, "fp8")])
def test_large_batches_of_short_requests(B, kv):
    # more than 1024 requests: every attention wave reads the lengths in
    # several batches of 1024 to find its share
    rng = np.random.default_rng(B)
    lens = rng.integers(0, 60, size=B)
    lens[rng.random(B) < 0.2] = 0
    case = dn.random_case(rng, B, 8, 2, 64, [int(x) for x in lens], kv)
    if kv == "fp8":
        case["k_scale"] = (rng.uniform(0.5, 1.5, size=(B, 2)) / 40.0).astype(np.float32)
        case["v_scale"] = (rng.uniform(0.5, 1.5, size=(B, 2)) / 40.0).astype(np.float32)
    scale = 0.125
    ref = oracle_case(case, scale, kv)
    for waves, pps in ((0, 0), (1, 1), (37, 2), (3000, 0)):
        got = run_case(dev_case(case, kv), scale, max_waves=waves, pages_per_step=pps)
        G.assert_close(got, ref, kv, f"B={B} {kv} waves={waves} pages/step={pps}")
        assert np.all(got[lens == 0] == 0.0)


@pytest.mark.parametrize("B", [63, 64, 65, 511, 512, 513, 1025])
def test_batches_at_the_planner_row_edges(B):
    # the planner holds 64 requests a row and 8 rows at a time
    rng = np.random.default_rng(B)
    lens = rng.integers(0, 50, size=B)
    lens[[0, B // 2, B - 1]] = [0, 0, 33]
    case = dn.random_case(rng, B, 4, 2, 64, [int(x) for x in lens], "bf16")
    ref = oracle_case(case, 0.125)
    for waves in (0, 3, 1000):
        got = run_case(dev_case(case), 0.125, max_waves=waves)
        G.assert_close(got, ref, "bf16", f"B={B} waves={waves}")
        assert np.all(got[lens == 0] == 0.0)


def test_fp8_every_code_through_single_token_rows():
    """Length-1 requests return their V row times the V scale; with scale 1 the
    output is the e4m3fn value itself, so every finite code is checked."""
    rng = np.random.default_rng(23)
    B, Hq, Hkv, D = 2, 8, 1, 128
    case = dn.random_case(rng, B, Hq, Hkv, D, [1, 1], "fp8")
    allc = np.arange(256, dtype=np.uint16).astype(np.uint8)
    allc[0x7F] = 0
    allc[0xFF] = 0
    case["dense_v"][0][0, 0] = allc[:128]
    case["dense_v"][1][0, 0] = allc[128:]
    case["v_scale"][:] = 1.0
    kp, vp = dn.write_pools(case["dense_k"], case["dense_v"], [1, 1], case["page_lists"], case["num_pages"],
                            Hkv, D, 16, np.uint8(0x7F))
    case.update(k_pages=kp, v_pages=vp)
    ref = dn.codes_to_f64_fp8(allc).reshape(2, 128)
    for pps in (1, 2, 4):
        got = run_case(dev_case(case, "fp8"), 0.1, pages_per_step=pps)
        for b in range(2):
            for h in range(Hq):
                assert np.array_equal(got[b, h], ref[b]), f"fp8 code decode b={b} h={h} pages/step={pps}"


def test_bad_block_table_entry_is_flagged_not_read():
    rng = np.random.default_rng(24)
    case = dn.random_case(rng, 2, 8, 2, 64, [40, 20])
    d = dev_case(case)
    bl.device_errors()
    bt = d["bt"].clone()
    bt[0, 1] = case["num_pages"] + 1000      # out of the pool: must be skipped, never dereferenced
    d["bt"] = bt
    got = run_case(d, 0.125)
    assert bl.device_errors() & 4
    assert np.all(np.isnan(got[0]))
    G.assert_close(got[1:], oracle_case(dict(case, q_bits=case["q_bits"][1:], block_table=case["block_table"][1:],
                                             seq_lens=case["seq_lens"][1:]), 0.125), "bf16", "untouched request")


def test_lengths_outside_the_table_are_clamped_and_flagged():
    # a negative length attends nothing (zeros); a length past the table's
    # width attends the whole row of pages; both raise the length flag
    rng = np.random.default_rng(25)
    case = dn.random_case(rng, 3, 8, 2, 64, [0, 48, 30])   # request 1 fills its three pages
    maxL = case["block_table"].shape[1] * 16
    assert maxL == 48
    ref = oracle_case(case, 0.125)
    for waves in (0, 1, 2, 5):
        d = dev_case(case)
        sl = d["sl"].clone()
        sl[0] = -5
        sl[1] = maxL + 7
        d["sl"] = sl
        bl.device_errors()
        got = run_case(d, 0.125, max_waves=waves)
        assert bl.device_errors() & 2, f"waves={waves}"
        assert np.all(got[0] == 0.0)
        G.assert_close(got[1:], ref[1:], "bf16", f"clamped lengths waves={waves}")


def test_append_out_of_table_is_skipped():
    w = G.to_device(wl.build("tiny", seed=2))
    before_k = G.bits16(w.k_pages)
    sl = w.seq_lens.clone()
    sl[2] = w.max_pages * 16                  # no page left for this request
    bl.device_errors()
    bl.kv_append(w.k_new[0], w.v_new[0], w.k_pages, w.v_pages, w.block_table, sl)
    torch.cuda.synchronize()
    assert bl.device_errors() & 1
    assert sl[2].item() == w.max_pages * 16
    assert sl[0].item() == w.lens0[0] + 1
    after_k = G.bits16(w.k_pages)
    assert (before_k != after_k).sum() > 0


@pytest.mark.parametrize("kv,D", [("bf16", 128), ("bf16", 64), ("fp8", 128), ("fp8", 64)])
def test_append_every_slot_keeps_the_rest_of_each_sector(kv, D):
    """The append writes whole 32-byte sectors, reading back the bytes around
    the new slot: over pools of arbitrary bytes (NaN patterns included), a
    request at every slot 0..15, twice over, the whole pools must equal the
    oracle's byte for byte."""
    rng = np.random.default_rng(77 + D)
    H_kv, maxP = 4, 3
    lens = np.concatenate([np.arange(16), 16 + np.arange(16)[::-1]]).astype(np.int32)   # slots 0..15 on pages 0 and 1
    B = len(lens)
    NP = B * maxP + 3
    bt = rng.permutation(NP)[:B * maxP].astype(np.int32).reshape(B, maxP)
    if kv == "bf16":
        kp = rng.integers(0, 1 << 16, size=(NP, H_kv, D // 8, 16, 8)).astype(np.uint16)
        vp = rng.integers(0, 1 << 16, size=(NP, H_kv, D, 16)).astype(np.uint16)
        kn = rng.integers(0, 1 << 16, size=(B, H_kv, D)).astype(np.uint16)
        vn = rng.integers(0, 1 << 16, size=(B, H_kv, D)).astype(np.uint16)
        code = oracle.BF16
    else:
        kp = rng.integers(0, 256, size=(NP, H_kv, D // 16, 16, 16)).astype(np.uint8)
        vp = rng.integers(0, 256, size=(NP, H_kv, D, 16)).astype(np.uint8)
        kn = rng.integers(0, 256, size=(B, H_kv, D)).astype(np.uint8)
        vn = rng.integers(0, 256, size=(B, H_kv, D)).astype(np.uint8)
        code = oracle.FP8_E4M3FN
    ref_k, ref_v, ref_sl = kp.copy(), vp.copy(), lens.copy()
    oracle.kv_append(kn, vn, ref_k, ref_v, bt, ref_sl, code)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    if kv == "bf16":
        dk, dv = t(kp.view(np.int16)).view(torch.bfloat16), t(vp.view(np.int16)).view(torch.bfloat16)
        dkn, dvn = t(kn.view(np.int16)).view(torch.bfloat16), t(vn.view(np.int16)).view(torch.bfloat16)
        ks = vs = None
    else:
        dk, dv, dkn, dvn = t(kp), t(vp), t(kn), t(vn)
        ks = vs = torch.ones((B, H_kv), dtype=torch.float32, device="cuda")
    dsl = t(lens)
    bl.kv_append(dkn, dvn, dk, dv, t(bt), dsl, k_scale=ks, v_scale=vs)
    torch.cuda.synchronize()
    assert bl.device_errors() == 0
    assert np.array_equal(dsl.cpu().numpy(), ref_sl)
    view = (lambda x: x.view(torch.int16).cpu().numpy().view(np.uint16)) if kv == "bf16" else (lambda x: x.cpu().numpy())
    gk, gv = view(dk), view(dv)
    assert np.array_equal(gk, ref_k), f"K pool differs at {int((gk != ref_k).sum())} elements"
    assert np.array_equal(gv, ref_v), f"V pool differs at {int((gv != ref_v).sum())} elements"


def test_empty_batch_is_noop():
    q = torch.empty((0, 8, 64), dtype=torch.bfloat16, device="cuda")
    k = torch.zeros((4, 2, 8, 16, 8), dtype=torch.bfloat16, device="cuda")
    v = torch.zeros((4, 2, 64, 16), dtype=torch.bfloat16, device="cuda")
    bt = torch.empty((0, 1), dtype=torch.int32, device="cuda")
    sl = torch.empty((0,), dtype=torch.int32, device="cuda")
    out = torch.empty((0, 8, 64), dtype=torch.bfloat16, device="cuda")
    bl.decode_attention(q, k, v, bt, sl, 0.125, out)
    torch.cuda.synchronize()


# ------------------------------------------------------ quantising append ---

def test_quantising_append_every_bf16_pattern():
    """bf16 rows into fp8 pools: all 65536 bf16 bit patterns go through the
    quantiser (K in order, V permuted) under mixed scales; the whole pools
    must equal the oracle's byte for byte."""
    rng = np.random.default_rng(41)
    B, H_kv, D, NP = 64, 8, 128, 80
    maxP = 1
    lens = rng.integers(0, 16, size=B).astype(np.int32)
    bt = rng.permutation(NP)[:B].astype(np.int32).reshape(B, maxP)
    kp = rng.integers(0, 256, size=(NP, H_kv, D // 16, 16, 16)).astype(np.uint8)
    vp = rng.integers(0, 256, size=(NP, H_kv, D, 16)).astype(np.uint8)
    allbits = np.arange(1 << 16, dtype=np.uint32).astype(np.uint16)
    kn = allbits.reshape(B, H_kv, D)
    vn = rng.permutation(allbits).reshape(B, H_kv, D)
    ks = np.float32(2.0) ** rng.integers(-12, 12, size=(B, H_kv)).astype(np.float32) * \
        rng.uniform(0.5, 1.0, size=(B, H_kv)).astype(np.float32)
    vs = rng.uniform(1e-3, 10.0, size=(B, H_kv)).astype(np.float32)
    ref_k, ref_v, ref_sl = kp.copy(), vp.copy(), lens.copy()
    oracle.kv_append(kn, vn, ref_k, ref_v, bt, ref_sl, oracle.FP8_E4M3FN, ks, vs)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    dk, dv, dsl = t(kp), t(vp), t(lens)
    bl.kv_append(t(kn.view(np.int16)).view(torch.bfloat16), t(vn.view(np.int16)).view(torch.bfloat16),
                 dk, dv, t(bt), dsl, k_scale=t(ks), v_scale=t(vs))
    torch.cuda.synchronize()
    assert bl.device_errors() == 0
    assert np.array_equal(dsl.cpu().numpy(), ref_sl)
    gk, gv = dk.cpu().numpy(), dv.cpu().numpy()
    bad_k = np.argwhere(gk != ref_k)
    assert len(bad_k) == 0, f"K pool differs at {len(bad_k)} bytes, first {bad_k[:3]}"
    assert np.array_equal(gv, ref_v), f"V pool differs at {int((gv != ref_v).sum())} bytes"


def test_quantising_append_then_attention():
    """A decode run of a shrunk fp8 workload whose new rows arrive as bf16 and
    are quantised by the append; appends bit-exact, attention within the fp8
    bounds at every step."""
    rng = np.random.default_rng(42)
    B, H_q, H_kv, D, steps = 6, 64, 8, 128, 4
    lens = [1, 15, 16, 100, 333, 1000]
    case = dn.random_case(rng, B, H_q, H_kv, D, [L + steps for L in lens], "fp8")
    # values of the size the workloads have (code 448 <-> about 4 sigma of N(0, 1))
    case["k_scale"][:] = np.float32(4.0 / 448.0)
    case["v_scale"][:] = np.float32(4.0 / 448.0)
    sl0 = np.asarray(lens, dtype=np.int32)
    d = dev_case(dict(case, seq_lens=sl0), "fp8")
    kp, vp = case["k_pages"].copy(), case["v_pages"].copy()
    sl = sl0.copy()
    for s in range(steps):
        kn = torch.from_numpy(rng.standard_normal((B, H_kv, D)).astype(np.float32)).to(torch.bfloat16)
        vn = torch.from_numpy(rng.standard_normal((B, H_kv, D)).astype(np.float32)).to(torch.bfloat16)
        kb = kn.view(torch.int16).numpy().view(np.uint16)
        vb = vn.view(torch.int16).numpy().view(np.uint16)
        oracle.kv_append(kb, vb, kp, vp, case["block_table"], sl, oracle.FP8_E4M3FN, case["k_scale"], case["v_scale"])
        bl.kv_append(kn.cuda(), vn.cuda(), d["k"], d["v"], d["bt"], d["sl"], k_scale=d["ks"], v_scale=d["vs"])
        got = run_case(d, float(np.float32(1 / np.sqrt(D))))
        assert np.array_equal(d["k"].cpu().numpy(), kp) and np.array_equal(d["v"].cpu().numpy(), vp), f"step {s}"
        ref = oracle.decode_attention(case["q_bits"], kp, vp, case["block_table"], sl,
                                      float(np.float32(1 / np.sqrt(D))), oracle.FP8_E4M3FN,
                                      case["k_scale"], case["v_scale"])
        G.assert_close(got, ref, "fp8", f"quantising append step {s}")
