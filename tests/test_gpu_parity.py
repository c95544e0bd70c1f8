"""HIP path vs fp64 oracle, through the C ABI, on seeded synthetic inputs.  Needs an MI355X."""
import numpy as np
import pytest
import torch

from oracle import calidrop_ref as ref
from paper_2507_19906_amd import binding as cd
from paper_2507_19906_amd import synth
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def to_dev(x):
    return {k: v.to(DEV) for k, v in x.items()}


def run_case(wl, seed=synth.BASE_SEED, decode_steps=None, heads=None, seqs=None):
    x = to_dev(synth.make_inputs(wl, seed))
    bufs = H.gpu_compress(wl, x)
    rep = {}
    seqs = range(wl.batch) if seqs is None else seqs
    for b in seqs:
        H.check_compress(wl, x, bufs, b, heads=heads, report=rep)
    T = wl.decode_steps if decode_steps is None else decode_steps
    for t in range(T):
        bufs.decode(x["q_dec"][t])
        torch.cuda.synchronize()
        for b in seqs:
            H.check_decode_step(wl, bufs, x["q_dec"][t], b, heads=heads, report=rep)
    print(wl.name, {k: (v if k != "flags" else np.bincount(v, minlength=3).tolist())
                    for k, v in rep.items()}, flush=True)
    return rep


def small(dtype, Hq, Hkv, D, lens, w, B, k, T=4, name="small"):
    return synth.Workload(name, len(lens), Hq, Hkv, D, list(lens), w, B, k, dtype, T)


def test_config1_fp32_compress_and_16_decode_steps():
    rep = run_case(synth.config(1))
    flags = np.bincount(rep["flags"], minlength=3)
    assert flags[1] > 0 and flags[2] > 0          # calibrate and recompute branches both hit


def test_config2_bf16_llama8b_8k():
    rep = run_case(synth.config(2), decode_steps=8)
    assert rep["c_out_err"] < 2e-2


@pytest.mark.parametrize("wl", [
    small("bf16", 8, 2, 64, [777], 16, 100, 5, name="ragged_bf16_d64"),
    small("fp32", 8, 2, 128, [1031], 16, 96, 3, name="ragged_fp32_d128"),
    small("bf16", 4, 4, 128, [600], 8, 40, 1, name="mha_g1_k1"),
    small("bf16", 16, 2, 128, [900], 32, 128, 7, name="g8_two_row_blocks"),
    small("fp32", 6, 2, 64, [300, 1000, 50, 257], 16, 64, 5, name="varlen_with_short_seq"),
    small("bf16", 32, 8, 128, [513, 2049, 100, 640], 32, 512, 7, name="varlen_bf16_budget_edge"),
    small("bf16", 4, 1, 128, [65], 1, 2, 1, name="window1_budget2"),
    small("bf16", 8, 2, 64, [9000, 12000], 16, 300, 5, T=2, name="selection_16_positions_per_thread"),
    small("bf16", 28, 4, 128, [1500, 777], 32, 256, 7, name="g7_qwen_like"),
    small("bf16", 64, 8, 128, [2100], 32, 512, 7, T=2, name="g8_llama70b_like"),
    small("fp32", 10, 2, 64, [640], 16, 96, 5, name="g5_fp32"),
    small("bf16", 6, 1, 64, [999], 8, 60, 3, name="g6_d64"),
    small("bf16", 16, 1, 64, [1500, 90], 16, 200, 5, name="g16_largest_group"),
    small("fp32", 32, 2, 128, [700], 8, 100, 3, T=2, name="g16_fp32_d128"),
    small("bf16", 8, 2, 128, [20000, 300, 8300], 32, 1024, 17, T=2, name="multi_workgroup_select_bf16"),
    small("fp32", 4, 2, 64, [16500], 16, 200, 21, T=2, name="multi_workgroup_select_fp32"),
    # longest prefix one workgroup selects over (32768 positions), heads starting 1, 2 and 3 floats
    # past a 16-byte boundary in the vote buffer, and shorter odd-length neighbours
    small("bf16", 4, 4, 64, [32768 + 17, 8193 + 17, 16390 + 17], 17, 90, 5, T=1, name="full_length_prefix_misaligned_heads"),
    # more than 128 window rows per KV head: 256-row blocks (K streamed once per pass), one full, one
    # with a ragged second block (384 rows), one in fp32, one with a window that is no multiple of 4
    small("bf16", 32, 4, 128, [5000, 900], 32, 256, 7, T=2, name="g8_w32_256_rows_per_head"),
    small("bf16", 16, 1, 128, [1200], 24, 200, 5, T=2, name="g16_w24_two_256_row_blocks"),
    small("fp32", 16, 2, 64, [700, 2300], 32, 100, 3, T=2, name="g8_fp32_256_rows"),
    small("bf16", 8, 2, 128, [1500], 50, 300, 5, T=2, name="g4_w50_200_rows_odd_window"),
], ids=lambda w: w.name)
def test_shapes_and_ragged_tails(wl):
    run_case(wl)


@pytest.mark.parametrize("dtype,Hq,Hkv,D,w", [("bf16", 8, 2, 128, 32), ("bf16", 8, 1, 64, 32), ("fp32", 4, 2, 64, 16),
                                              ("fp32", 16, 1, 128, 16)])
def test_scoring_at_the_edges_of_its_key_stages(dtype, Hq, Hkv, D, w):
    # prompts and prefixes that end one short of, at and one past a stage of 64 (fp32: 32) keys, and at the
    # second and third stage; 128- and 256-row blocks
    lens = sorted({e + d + s for e in (64, 128, 192) for d in (-1, 0, 1) for s in (0, w)} | {31 + w, 33 + w})
    run_case(small(dtype, Hq, Hkv, D, [n for n in lens if n > 24 + w], w, w + 8, 5, T=1, name=f"stage_edges_{dtype}_{D}"))


@pytest.mark.parametrize("dtype,D,budget", [("bf16", 128, 64), ("fp32", 64, 200), ("bf16", 64, 300),
                                            ("bf16", 128, 600)])
def test_many_sequences_single_workgroup_decode(dtype, D, budget):
    # 200 (sequence, KV head) pairs of short caches: decode runs as one workgroup per pair, with 4 or 8 waves
    g = torch.Generator().manual_seed(budget)
    lens = torch.randint(budget // 2, 3 * budget, (100,), generator=g).tolist()
    wl = small(dtype, 8, 2, D, lens, 16, budget, 5, T=3, name=f"many_seqs_{dtype}_{D}_{budget}")
    x = to_dev(synth.make_inputs(wl, 17))
    bufs = H.gpu_compress(wl, x, extra_capacity=8)
    assert len(H.captured_launches(lambda: bufs.decode(x["q_dec"][0]))) == 1
    rep = {}
    seqs = [0, 1, 37, 99, int(np.argmin(lens)), int(np.argmax(lens))]
    for b in seqs:
        H.check_compress(wl, x, bufs, b, report=rep)
    for t in range(3):
        if t == 2:      # ragged live lengths: append rows to some sequences, empty one
            bufs.cache_lens[1::2] += 5
            bufs.cache_lens[37] = 0
        bufs.decode(x["q_dec"][t])
        torch.cuda.synchronize()
        for b in seqs:
            H.check_decode_step(wl, bufs, x["q_dec"][t], b, report=rep)
    print(wl.name, {k: v for k, v in rep.items() if k != "flags"}, flush=True)


@pytest.mark.parametrize("n,k,period,k_sel", [(16 * 40 + 16, 1, 40, 50), (20016, 17, 3000, 777), (20016, 1, 3000, 2500)])
def test_exact_ties_lower_index_wins(n, k, period, k_sel):
    # periodic keys: position j and j + period have identical keys, hence bit-identical votes
    # on both sides; the pooled scores tie exactly (away from the two ends of the prefix when
    # k > 1) and the lower position must be kept.  The long prompts take the multi-workgroup
    # selection, where a tie class spans several workgroups.
    wl = small("bf16", 8, 2, 64, [n], 16, 16 + k_sel, k, T=0, name="ties")
    x = synth.make_inputs(wl, 99)
    K = synth.seq_view(x["k"], wl, 0)
    P = wl.seq_lens[0] - wl.window
    for j in range(period, P):
        K[:, j] = K[:, j % period]
    x = to_dev(x)
    bufs = H.gpu_compress(wl, x)
    orc = H.oracle_compress(wl, x, 0)
    got = bufs.indices[0].cpu().numpy()
    assert np.array_equal(got, orc["idx"])                      # no band: exact
    sel = got[:, :k_sel]
    # the retained prefix positions contain whole tie classes from the lowest copy upwards
    half = k // 2
    n_checked = 0
    for g in range(2):
        s = set(sel[g].tolist())
        for j in s:
            if j - period >= half and j < P - half:
                assert (j - period) in s
                n_checked += 1
    assert n_checked > 0


def test_full_budget_keeps_everything_and_decode_is_exact_attention():
    wl = small("bf16", 8, 2, 128, [200, 64], 16, 256, 5, T=2, name="budget_ge_n")
    x = to_dev(synth.make_inputs(wl, 5))
    bufs = H.gpu_compress(wl, x)
    for b in range(2):
        H.check_compress(wl, x, bufs, b)
        n = wl.seq_lens[b]
        idx = bufs.indices[b].cpu().numpy()
        assert np.array_equal(idx[:, :n], np.tile(np.arange(n), (2, 1))) and np.all(idx[:, n:] == -1)
    assert torch.all(torch.isinf(bufs.c_lse)) and torch.all(bufs.c_lse < 0)
    bufs.decode(x["q_dec"][0])
    torch.cuda.synchronize()
    for b in range(2):
        K = H.to64(synth.seq_view(x["k"], wl, b)); V = H.to64(synth.seq_view(x["v"], wl, b))
        q = H.to64(x["q_dec"][0][b])
        for h in range(8):
            full, _ = ref.attention(q[h], K[h // 4], V[h // 4], 128 ** -0.5)
            assert np.abs(H.to64(bufs.out[b, h]) - full).max() < 2e-2
    assert not torch.any(bufs.flags == cd.FLAG_CALIBRATED)


@pytest.mark.parametrize("dtype,tol", [("fp32", 1e-4), ("bf16", 2e-2)])
def test_identical_query_calibration_reproduces_full_attention(dtype, tol):
    # q_cal == q_t  =>  Eq. 1 makes the calibrated output the exact attention over all tokens
    wl = small(dtype, 8, 2, 64, [1500], 16, 80, 5, T=1, name="identical_query")
    x = to_dev(synth.make_inputs(wl, 11))
    q_t = x["q_dec"][0]
    bufs = H.gpu_compress(wl, x, q_cal=q_t)
    bufs.decode(q_t)
    torch.cuda.synchronize()
    assert torch.all(bufs.flags == cd.FLAG_CALIBRATED)
    K = H.to64(synth.seq_view(x["k"], wl, 0)); V = H.to64(synth.seq_view(x["v"], wl, 0))
    q = H.to64(q_t[0])
    for h in range(8):
        full, lse = ref.attention(q[h], K[h // 4], V[h // 4], 64 ** -0.5)
        assert np.abs(H.to64(bufs.out[0, h]) - full).max() < tol
        both = np.logaddexp(bufs.a_lse[0, h].item(), bufs.c_lse[0, h].item())
        assert abs(both - lse) < 2e-3


def test_decode_with_appended_rows_and_empty_cache():
    wl = small("bf16", 8, 2, 128, [700, 900], 16, 96, 5, T=6, name="append")
    x = to_dev(synth.make_inputs(wl, 21))
    bufs = H.gpu_compress(wl, x, extra_capacity=40)
    g = torch.Generator(device=DEV).manual_seed(3)
    rep = {}
    for t in range(6):
        # the caller appends one K/V row per step and raises cache_lens
        for b in range(2):
            L = int(bufs.cache_lens[b].item())
            bufs.cache_view("k", b)[:, L] = torch.randn((2, 128), generator=g, device=DEV).bfloat16()
            bufs.cache_view("v", b)[:, L] = torch.randn((2, 128), generator=g, device=DEV).bfloat16()
        bufs.cache_lens += 1
        bufs.decode(x["q_dec"][t])
        torch.cuda.synchronize()
        for b in range(2):
            H.check_decode_step(wl, bufs, x["q_dec"][t], b, report=rep)
    assert int(bufs.cache_lens[0].item()) == 102
    # empty cache: out = c_out when calibrated (alpha_j = 1), a_lse = -inf
    bufs.cache_lens.zero_()
    p_always = H.params_for(wl, theta1=float("-inf"), theta2=float("-inf"))
    cd.calidrop_decode(p_always, x["q_dec"][0], bufs.k_c, bufs.v_c, bufs.cache_offsets, bufs.cache_lens,
                       bufs.max_cache_len, bufs.c_q, bufs.c_out, bufs.c_lse, bufs.out, bufs.a_lse,
                       bufs.flags, bufs.ws_decode)
    torch.cuda.synchronize()
    assert torch.all(torch.isinf(bufs.a_lse)) and torch.all(bufs.flags == cd.FLAG_CALIBRATED)
    assert (bufs.out.float() - bufs.c_out).abs().max().item() < 2e-2


def test_gate_thresholds_exact_on_gpu():
    # c_q = e1, q_t = (a, b, 0, ...): rho = a / sqrt(a^2 + b^2); 3-4-5 triangles are exact in fp32
    wl = small("fp32", 2, 1, 64, [40], 4, 8, 1, T=0, name="gate")
    x = to_dev(synth.make_inputs(wl, 1))
    bufs = H.gpu_compress(wl, x)
    bufs.c_q.zero_(); bufs.c_q[..., 0] = 1.0

    def flags_for(a, b, t1, t2):
        q = torch.zeros((1, 2, 64), device=DEV); q[..., 0] = a; q[..., 1] = b
        p = H.params_for(wl, theta1=t1, theta2=t2)
        cd.calidrop_decode(p, q, bufs.k_c, bufs.v_c, bufs.cache_offsets, bufs.cache_lens,
                           bufs.max_cache_len, bufs.c_q, bufs.c_out, bufs.c_lse, bufs.out,
                           bufs.a_lse, bufs.flags, bufs.ws_decode)
        torch.cuda.synchronize()
        return bufs.flags.cpu().numpy().ravel().tolist()

    f06, f08 = float(np.float32(0.6)), float(np.float32(0.8))
    assert flags_for(3, 4, 0.7, 0.85) == [2, 2]
    assert flags_for(4, 3, 0.7, 0.85) == [0, 0]
    assert flags_for(12, 5, 0.7, 0.85) == [1, 1]
    assert flags_for(3, 4, f06, 0.85) == [0, 0]        # rho == theta1: strict
    assert flags_for(4, 3, 0.7, f08) == [0, 0]         # rho == theta2: strict
    assert flags_for(0, 0, 0.7, 0.85) == [2, 2]        # zero query: rho := 0


def test_determinism_bitwise():
    wl = synth.config(2)
    wl.seq_lens = [4100]
    x = to_dev(synth.make_inputs(wl, 4))
    a = H.gpu_compress(wl, x)
    b = H.gpu_compress(wl, x)
    for name in ["indices", "k_c", "v_c", "c_out", "c_lse", "c_q", "cache_lens"]:
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    a.decode(x["q_dec"][0]); b.decode(x["q_dec"][0])
    torch.cuda.synchronize()
    assert torch.equal(a.out, b.out) and torch.equal(a.a_lse, b.a_lse)


@pytest.mark.parametrize("wl", [
    synth.config(1),
    small("bf16", 8, 2, 128, [900, 40, 2100], 16, 128, 5, T=10, name="recal_varlen_bf16"),
    small("bf16", 16, 2, 64, [1200], 32, 200, 7, T=6, name="recal_g8_d64"),
], ids=lambda w: w.name)
def test_full_decode_loop_with_recomputation(wl):
    # Alg. 2 end to end: decode, then the recomputation branch for the heads it flagged, state
    # carried across steps on the GPU; every step is checked against the oracle on the same state
    x = to_dev(synth.make_inputs(wl, 31))
    bufs = H.gpu_compress(wl, x)
    rep = {}
    for t in range(wl.decode_steps):
        q_t = x["q_dec"][t]
        bufs.decode(q_t)
        torch.cuda.synchronize()
        for b in range(wl.batch):
            H.check_decode_step(wl, bufs, q_t, b, report=rep)
        before = H.snapshot_state(bufs)
        bufs.recalibrate(q_t, x["k"], x["v"], x["seq_offsets"])
        torch.cuda.synchronize()
        for b in range(wl.batch):
            H.check_recalibrate(wl, x, bufs, q_t, b, before, report=rep)
        assert not torch.any(bufs.flags == cd.FLAG_RECOMPUTE)
    flags = np.bincount(rep.pop("flags"), minlength=4)
    print(wl.name, rep, flags.tolist(), flush=True)
    assert rep["recal_heads"] > 0 and flags[1] > 0        # both branches were exercised


@pytest.mark.parametrize("dtype,budget,m", [("bf16", 40, 0), ("fp32", 40, 50), ("bf16", 700, 0), ("bf16", 40, 900)])
def test_recomputation_at_the_edges_of_its_row_blocks(dtype, budget, m):
    # prompts that end one short of, at and one past one and several blocks of 128 rows; position lists short
    # enough to be read by the streaming pass itself (up to twice the rows of a split) and longer ones
    wl = small(dtype, 4, 2, 64, [127, 128, 129, 255, 257, 1151, 1153, 2049, 30], 16, budget, 5, T=3, name="row_blocks")
    wl.theta1 = wl.theta2 = 2.0                      # every head is recomputed at every step
    x = to_dev(synth.make_inputs(wl, 83))
    bufs = H.gpu_compress(wl, x, calib_size=m)
    rep = {}
    for t in range(wl.decode_steps):
        q_t = x["q_dec"][t]
        bufs.decode(q_t)
        torch.cuda.synchronize()
        before = H.snapshot_state(bufs)
        bufs.recalibrate(q_t, x["k"], x["v"], x["seq_offsets"])
        torch.cuda.synchronize()
        for b in range(wl.batch):
            H.check_recalibrate(wl, x, bufs, q_t, b, before, report=rep)
    assert rep["recal_heads"] == wl.batch * wl.n_q_heads * wl.decode_steps


@pytest.mark.parametrize("dtype,m", [("bf16", 0), ("fp32", 0), ("bf16", 900), ("fp32", 1280), ("bf16", 1281)])
def test_recomputation_with_several_row_blocks_per_split(dtype, m):
    # splits of 640 rows, five blocks each: lengths that end one short of, at and one past a split and a block; lists of
    # up to twice a split, read by the streaming pass itself, and one entry more; short prompts in the same batch
    wl = small(dtype, 4, 2, 64, [20001, 19840, 19841, 19839, 640, 641, 130, 30], 16, 40, 5, T=2, name="split_blocks")
    wl.theta1 = wl.theta2 = 2.0                      # every head is recomputed at every step
    x = to_dev(synth.make_inputs(wl, 84))
    bufs = H.gpu_compress(wl, x, calib_size=m)
    rep = {}
    for t in range(wl.decode_steps):
        q_t = x["q_dec"][t]
        bufs.decode(q_t)
        torch.cuda.synchronize()
        before = H.snapshot_state(bufs)
        bufs.recalibrate(q_t, x["k"], x["v"], x["seq_offsets"])
        torch.cuda.synchronize()
        for b in range(wl.batch):
            H.check_recalibrate(wl, x, bufs, q_t, b, before, report=rep)
    assert rep["recal_heads"] == wl.batch * wl.n_q_heads * wl.decode_steps


def test_recomputation_yields_exact_full_attention():
    # after recomputation with the current query, the calibrated output is the attention over
    # the whole prompt (Eq. 1 with the true query on both parts)
    wl = small("fp32", 8, 2, 64, [1500], 16, 80, 5, T=1, name="recal_exact")
    x = to_dev(synth.make_inputs(wl, 12))
    bufs = H.gpu_compress(wl, x)
    q_t = -x["q_win"][:, :, -1].contiguous()                 # rho = -1: every head is flagged
    bufs.decode(q_t)
    torch.cuda.synchronize()
    assert torch.all(bufs.flags == cd.FLAG_RECOMPUTE)
    bufs.recalibrate(q_t, x["k"], x["v"], x["seq_offsets"])
    torch.cuda.synchronize()
    assert torch.all(bufs.flags == cd.FLAG_RECOMPUTED)
    K = H.to64(synth.seq_view(x["k"], wl, 0)); V = H.to64(synth.seq_view(x["v"], wl, 0))
    q = H.to64(q_t[0])
    for h in range(8):
        full, _ = ref.attention(q[h], K[h // 4], V[h // 4], 64 ** -0.5)
        assert np.abs(H.to64(bufs.out[0, h]) - full).max() < 1e-4
    # untouched when nothing is flagged: a second call is a no-op
    snap = H.snapshot_state(bufs)
    bufs.recalibrate(q_t, x["k"], x["v"], x["seq_offsets"])
    torch.cuda.synchronize()
    after = H.snapshot_state(bufs)
    for key in snap:
        assert np.array_equal(snap[key], after[key]), key


def test_random_small_configurations():
    # seeded sweep over shapes, dtypes, windows, budgets, pooling widths, scales and lengths,
    # including the edge cases one evicted token (n = B + 1), budget = window + 1, pooling
    # wider than the in-LDS limit, and a non-default logit scale
    rng = np.random.default_rng(7)
    cases = [
        dict(dtype="bf16", Hq=4, Hkv=2, D=64, lens=[34], w=4, B=33, k=3),          # n = B + 1
        dict(dtype="fp32", Hq=2, Hkv=2, D=64, lens=[200], w=7, B=8, k=1),           # B = w + 1, odd w
        dict(dtype="bf16", Hq=8, Hkv=1, D=128, lens=[700], w=12, B=100, k=17),      # k beyond the LDS variant
        dict(dtype="fp32", Hq=16, Hkv=1, D=64, lens=[300, 90], w=8, B=64, k=5),     # G = 16
        dict(dtype="bf16", Hq=12, Hkv=4, D=128, lens=[257, 1025], w=20, B=96, k=9, scale=0.05),
    ]
    for _ in range(8):
        Hkv = int(rng.choice([1, 2, 4]))
        G = int(rng.choice([1, 2, 4, 8]))
        w = int(rng.integers(1, 40))
        B = w + int(rng.integers(1, 200))
        lens = [int(rng.integers(2, 1500)) for _ in range(int(rng.integers(1, 4)))]
        cases.append(dict(dtype=str(rng.choice(["bf16", "fp32"])), Hq=Hkv * G, Hkv=Hkv, D=int(rng.choice([64, 128])),
                          lens=lens, w=w, B=B, k=int(rng.choice([1, 3, 5, 7, 11]))))
    for i, c in enumerate(cases):
        wl = small(c["dtype"], c["Hq"], c["Hkv"], c["D"], c["lens"], c["w"], c["B"], c["k"], T=2, name=f"rand{i}")
        x = to_dev(synth.make_inputs(wl, 100 + i))
        over = {"scale": c["scale"]} if "scale" in c else {}
        bufs = H.gpu_compress(wl, x, **over)
        rep = {}
        for b in range(wl.batch):
            if "scale" in c:        # the oracle helpers use the default scale: check this one directly
                n = wl.seq_lens[b]
                K = H.to64(synth.seq_view(x["k"], wl, b)); V = H.to64(synth.seq_view(x["v"], wl, b))
                orc = ref.compress(H.to64(x["q_win"][b]), K, V, wl.window, wl.budget, wl.pool_kernel, scale=c["scale"])
                assert np.array_equal(bufs.indices[b].cpu().numpy()[:, :min(n, wl.budget)], orc["idx"])
                assert np.abs(H.to64(bufs.c_out[b]) - orc["c_out"]).max() < 2e-2
                assert np.abs(H.to64(bufs.c_lse[b]) - orc["c_lse"]).max() < 2e-3
            else:
                H.check_compress(wl, x, bufs, b, report=rep)
        if "scale" not in c:
            for t in range(2):
                bufs.decode(x["q_dec"][t])
                torch.cuda.synchronize()
                for b in range(wl.batch):
                    H.check_decode_step(wl, bufs, x["q_dec"][t], b, report=rep)
        print(wl.name, c, {k: v for k, v in rep.items() if k != "flags"}, flush=True)


def test_decode_under_hip_graph_replay():
    # the decode entry point allocates nothing and records no memset: a captured graph of
    # several steps must reproduce the eager results on every replay
    wl = small("bf16", 8, 2, 128, [600] * 100, 16, 128, 5, T=4, name="graph")
    x = to_dev(synth.make_inputs(wl, 77))
    bufs = H.gpu_compress(wl, x)
    outs = [torch.empty_like(bufs.out) for _ in range(4)]
    eager = []
    for t in range(4):
        bufs.decode(x["q_dec"][t])
        torch.cuda.synchronize()
        eager.append((bufs.out.clone(), bufs.a_lse.clone(), bufs.flags.clone()))
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        for t in range(4):                       # warm-up on the capture stream
            bufs.decode(x["q_dec"][t], stream=side)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            for t in range(4):
                bufs.decode(x["q_dec"][t], stream=torch.cuda.current_stream())
                outs[t].copy_(bufs.out)
    for rep_i in range(3):
        for o in outs:
            o.zero_()
        bufs.out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for t in range(4):
            assert torch.equal(outs[t], eager[t][0]), (rep_i, t)
        assert torch.equal(bufs.a_lse, eager[3][1]) and torch.equal(bufs.flags, eager[3][2])


@pytest.mark.parametrize("dtype,D,k,m", [("bf16", 128, 5, 1), ("bf16", 64, 7, 50), ("fp32", 64, 3, 200),
                                         ("bf16", 128, 17, 33), ("fp32", 128, 1, 5000), ("fp32", 64, 17, 300)])
def test_calibration_size(dtype, D, k, m):
    # Sec. 5.3: only the m evicted tokens of highest score are calibrated / offloaded; m larger
    # than the evicted set means all of it; k = 17 goes through the long-prefix selection kernel
    wl = small(dtype, 8, 2, D, [900, 40, 1700], 16, 96, k, T=6, name=f"calib_{dtype}_{D}_{k}_{m}")
    x = to_dev(synth.make_inputs(wl, 41))
    bufs = H.gpu_compress(wl, x, calib_size=m)
    rep = {}
    for b in range(wl.batch):
        H.check_compress(wl, x, bufs, b, report=rep)
    cal = bufs.cal_indices.cpu().numpy()
    assert cal.shape == (3, 2, m)
    n_e = 900 - 96
    assert np.all((cal[0] >= 0).sum(axis=1) == min(m, n_e))
    for t in range(wl.decode_steps):
        q_t = x["q_dec"][t]
        bufs.decode(q_t)
        torch.cuda.synchronize()
        before = H.snapshot_state(bufs)
        bufs.recalibrate(q_t, x["k"], x["v"], x["seq_offsets"])
        torch.cuda.synchronize()
        for b in range(wl.batch):
            H.check_recalibrate(wl, x, bufs, q_t, b, before, report=rep)
    rep.pop("flags", None)
    print(wl.name, rep, flush=True)
    assert rep["recal_heads"] > 0


@pytest.mark.parametrize("dtype,m", [("fp32", 1000), ("bf16", 9000)])
def test_calibration_size_with_multi_workgroup_selection(dtype, m):
    # second rank cut on the path where several workgroups share a head (prefix > 8192, k = 17)
    wl = small(dtype, 4, 2, 64, [17000, 500], 16, 300, 17, T=2, name=f"calib_wide_{dtype}_{m}")
    x = to_dev(synth.make_inputs(wl, 43))
    bufs = H.gpu_compress(wl, x, calib_size=m)
    rep = {}
    for b in range(wl.batch):
        H.check_compress(wl, x, bufs, b, report=rep)
    cal = bufs.cal_indices.cpu().numpy()
    assert np.all((cal[0] >= 0).sum(axis=1) == m) and np.all((cal[1] >= 0).sum(axis=1) == min(m, 200))
    for t in range(wl.decode_steps):
        q_t = x["q_dec"][t]
        bufs.decode(q_t)
        torch.cuda.synchronize()
        before = H.snapshot_state(bufs)
        bufs.flags.fill_(cd.FLAG_RECOMPUTE)
        before["flags"][:] = cd.FLAG_RECOMPUTE
        bufs.recalibrate(q_t, x["k"], x["v"], x["seq_offsets"])
        torch.cuda.synchronize()
        for b in range(wl.batch):
            H.check_recalibrate(wl, x, bufs, q_t, b, before, report=rep)
    rep.pop("flags", None)
    print(wl.name, rep, flush=True)


@pytest.fixture
def wide_selection():
    old = H.TEST_FLAGS
    H.TEST_FLAGS = old | cd.OPT_WIDE_SELECTION
    yield
    H.TEST_FLAGS = old


@pytest.mark.parametrize("wl", [
    small("bf16", 8, 2, 64, [777], 16, 100, 5, name="wide_ragged_bf16_d64"),
    small("fp32", 6, 2, 64, [300, 1000, 50, 257], 16, 64, 5, name="wide_varlen_with_short_seq"),
    small("bf16", 32, 8, 128, [513, 2049, 100, 640], 32, 512, 7, name="wide_varlen_bf16_budget_edge"),
    small("bf16", 4, 1, 128, [65], 1, 2, 1, name="wide_window1_budget2"),
], ids=lambda w: w.name)
def test_multi_workgroup_selection_on_short_prompts(wl, wide_selection):
    # the chain of launches long prompts use, forced on shapes with one (partial) segment per head
    run_case(wl)


@pytest.mark.parametrize("pool,m", [(1, 0), (7, 500), (15, 40000)])
def test_multi_workgroup_selection_at_segment_edges(pool, m):
    # prefixes that end one short of, at and one past a segment of 8192 scores (and at the second one): the lists of
    # the two selection variants are the same integers
    w = 16
    wl = small("bf16", 4, 2, 64, [8191 + w, 8192 + w, 8193 + w, 16384 + w, 16385 + w, 60], w, 700, pool, T=0, name="segment_edges")
    x = to_dev(synth.make_inputs(wl, 29))
    one = H.gpu_compress(wl, x, calib_size=m, flags=0)
    many = H.gpu_compress(wl, x, calib_size=m, flags=cd.OPT_WIDE_SELECTION)
    assert torch.equal(one.indices, many.indices)
    assert torch.equal(one.k_c, many.k_c) and torch.equal(one.v_c, many.v_c) and torch.equal(one.cache_lens, many.cache_lens)
    assert torch.equal(one.c_out, many.c_out) and torch.equal(one.c_lse, many.c_lse)
    if m:
        assert torch.equal(one.cal_indices, many.cal_indices)


@pytest.mark.parametrize("kind", ["normal", "flat", "tiny", "zero", "inf"])
@pytest.mark.parametrize("per,prefixes", [(2, [2048, 2047, 101]), (8, [8192, 2049, 8189]), (16, [16384, 8193]), (32, [32768, 16385, 40])])
def test_single_workgroup_selection_at_its_edges(per, prefixes, kind):
    # the longest prefix of each positions-per-thread variant, the first beyond the one before, neighbours whose votes start at
    # every offset into 16 bytes: scores, lists and skip bits are those of the multi-workgroup chain, bit for bit.  Scores
    # that crowd in one bin of the first digit (flat), below the range of the short division (tiny), all equal (zero), infinite.
    w, Hkv = 15, 3
    for pool, m in ((7, 0), (15, 300), (1, 33)):
        wl = small("bf16", 6, Hkv, 64, [n + w for n in prefixes], w, 90, pool, T=0, name="selection_edges")
        x = to_dev(synth.make_inputs(wl, 31 + per))
        if kind == "flat":
            x["k"] = x["k"] * 2.0 ** -9
        lse = dict(tiny=85.0, zero=300.0, inf=-300.0).get(kind)
        win_lse = None if lse is None else torch.full((wl.batch, 6, w), lse, device=DEV)
        one = H.gpu_compress(wl, x, calib_size=m, win_lse=win_lse, flags=cd.OPT_WRITE_SCORES)
        many = H.gpu_compress(wl, x, calib_size=m, win_lse=win_lse, flags=cd.OPT_WIDE_SELECTION)
        assert torch.equal(one.indices, many.indices), (kind, pool)
        assert torch.equal(one.c_out, many.c_out) and torch.equal(one.c_lse, many.c_lse)
        if m:
            assert torch.equal(one.cal_indices, many.cal_indices)
        s1, s2 = (b.region(cd.REGION_SCORE).view(torch.int32) for b in (one, many))
        off = 0
        for n in wl.seq_lens:
            for g in range(Hkv):
                if n > wl.budget:
                    assert torch.equal(s1[off:off + n - w], s2[off:off + n - w]), (kind, pool, n, g)
                off += n


@pytest.mark.parametrize("pool", [127, 129, 131])
def test_pooling_widths_around_what_is_staged(pool):
    # half widths of 63, 64 (the widest kept in LDS) and 65, over a segment boundary
    run_case(small("fp32", 2, 2, 64, [8192 + 16 + 300, 400], 16, 200, pool, T=0, name=f"pool_{pool}"))


def test_exact_ties_with_multi_workgroup_selection(wide_selection):
    test_exact_ties_lower_index_wins(16 * 40 + 16, 1, 40, 50)
    test_exact_ties_lower_index_wins(20016, 1, 3000, 2500)


def gathered_in(wl):
    """Where a compress call of few heads gathers the retained rows, read from its launches."""
    x = to_dev(synth.make_inputs(wl, 1))
    bufs = H.gpu_compress(wl, x)
    launches = H.captured_launches(lambda: bufs.compress(x["q_win"], x["k"], x["v"], x["seq_offsets"]))
    pass_, merge = launches[-2:]
    assert merge[1:3] == (wl.batch, 1)
    if merge[0] > wl.n_q_heads:                  # more workgroups a sequence than query heads
        return "merge"
    assert merge[0] == wl.n_q_heads and pass_[1] == wl.n_kv_heads
    return "pass" if pass_[2] > wl.batch else "elsewhere"


@pytest.mark.parametrize("dtype,budget", [("fp32", 64), ("fp32", 700), ("fp32", 2688), ("fp32", 2690), ("bf16", 1500),
                                          ("fp32", 10912), ("fp32", 10913)])
def test_gather_workgroups_behind_the_streaming_ones(dtype, budget):
    # 256 pieces of 16 bytes per gathering workgroup, 16 rows in fp32 and 32 in bf16 here.  Budget 64: 12 of them per KV head,
    # less than one plane of the streaming pass's 23 splits; 700, 2688, 2690 and 1500: 132, 504, 507 and 141, several planes
    # with a partial last one; 10912: 4092 for the six (sequence, KV head) pairs, the pass still carries them; 10913: 4098,
    # in the launch that merges the partials
    lens = [2900, budget - 1, 2850] if budget < 2800 else [11500, budget - 1, 10990]
    wl = small(dtype, 4, 2, 64, lens, 16, budget, 5, T=1, name=f"gather_{budget}")
    run_case(wl)
    assert gathered_in(wl) == ("pass" if budget < 10913 else "merge")


@pytest.mark.parametrize("n", [28672, 28673])
def test_gather_beside_short_and_long_splits(n):
    # splits of 896 and of 1024 rows: the launch that merges the partials carries the gather
    wl = small("bf16", 8, 2, 128, [n], 16, 200, 5, T=1, name=f"gather_n{n}")
    run_case(wl)
    assert gathered_in(wl) == "merge"


@pytest.mark.parametrize("dtype,D,w,lens", [
    ("bf16", 64, 16, [64 * 17]),                            # 64 rows, the rest of the block padding; 17 partials: 9 and 8
    ("fp32", 128, 33, [4097, 100, 63, 200]),                # 132 rows: a 256-row block; prompts with fewer partials and one
    ("bf16", 128, 32, [64 * 64]),                           # 64 partials, as many as pass 2 merges
    ("bf16", 64, 32, [64 * 64 * 3 + 1, 5000]),              # more: a launch of their own
    ("fp32", 64, 70, [2500])])                              # 280 rows: two row blocks
def test_chunk_partials_merged_in_pass_2_or_ahead(dtype, D, w, lens):
    wl = small(dtype, 8, 2, D, lens, w, w + 24, 5, T=0, name="merge_rows")
    x = to_dev(synth.make_inputs(wl, 63))
    bufs = H.gpu_compress(wl, x)
    for b in range(wl.batch):
        H.check_compress(wl, x, bufs, b)
    table = bufs.region(cd.REGION_ROW_LSE)
    rows = 4 * w
    stride = table.numel() // (2 * wl.batch)
    table = table.view(wl.batch, 2, stride)
    q, k, off = x["q_win"].double().cpu(), x["k"].double().cpu().view(-1, D), 0
    for b, n in enumerate(wl.seq_lens):
        for g in range(2):
            if n > wl.budget:
                z = q[b, 4 * g:4 * g + 4].reshape(rows, D) @ k[off:off + n].t() / D ** 0.5
                see = n - w + torch.arange(w).repeat(4)
                z = z.masked_fill(torch.arange(n)[None] > see[:, None], float("-inf"))
                want = torch.logsumexp(z, 1) * 1.4426950408889634
                # values up to some 100, where a float32 step is 7.6e-6: roundings of the logit, of the logarithm of the sum
                # and of adding both, and of merging partials
                assert (table[b, g, :rows].double().cpu() - want).abs().max() < 5e-5
                assert torch.isinf(table[b, g, rows:]).all()
            off += n


@pytest.mark.parametrize("dtype,Hq,Hkv,D,batch,budget,launches", [
    ("bf16", 16, 4, 128, 2, 516, 1), ("bf16", 16, 4, 128, 2, 517, 1),
    ("bf16", 16, 4, 128, 2, 519, 1),       # the last number of rows one workgroup takes and the first that are split: 8 pairs,
    ("bf16", 16, 4, 128, 2, 520, 2),       # 7.75 us / 7.73 with rows that were just read
    ("bf16", 16, 4, 128, 4, 355, 1), ("bf16", 16, 4, 128, 4, 356, 2),      # 16 pairs: more than one on an XCD
    ("fp32", 8, 2, 64, 20, 256, 1), ("fp32", 8, 2, 64, 20, 257, 2),        # two tiles a wave, and three
    ("fp32", 8, 2, 64, 20, 399, 2), ("fp32", 8, 2, 64, 20, 400, 2),
    ("bf16", 4, 4, 64, 66, 516, 1), ("bf16", 4, 4, 64, 66, 517, 2),        # more pairs than compute units: 264
    ("bf16", 4, 4, 64, 66, 750, 2),
    ("fp32", 8, 4, 128, 70, 286, 1), ("fp32", 8, 4, 128, 70, 287, 2),      # 280 pairs
    ("bf16", 8, 8, 64, 24, 1200, 1)])      # 192 pairs, 8 waves
def test_decode_forms_at_their_borders(dtype, Hq, Hkv, D, batch, budget, launches):
    lens = [budget + 40, budget - 5, 60] + [budget + 1 + b for b in range(batch - 3)]
    lens = lens[:batch]
    wl = small(dtype, Hq, Hkv, D, lens, 16, budget, 5, T=2, name=f"forms_{batch}x{budget}")
    x = to_dev(synth.make_inputs(wl, 57))
    bufs = H.gpu_compress(wl, x)
    assert len(H.captured_launches(lambda: bufs.decode(x["q_dec"][0]))) == launches
    rep = {}
    for t in range(wl.decode_steps):
        bufs.decode(x["q_dec"][t])
        torch.cuda.synchronize()
        for b in {0, 1, 2 % batch, batch - 1}:
            H.check_decode_step(wl, bufs, x["q_dec"][t], b, report=rep)


@pytest.mark.parametrize("dtype,Hq,Hkv,D,batch,budget,room,appended,launches", [
    ("bf16", 32, 8, 128, 8, 200, 824, 0, 1),       # 64 pairs, 200 of 1024 rows live: 6.0 us in one workgroup each, 9.1 split
    ("bf16", 32, 8, 128, 1, 200, 1848, 0, 1),      # 8 pairs, 200 of 2048: 5.2 / 7.4
    ("bf16", 16, 4, 64, 16, 200, 1848, 0, 1),      # 64 pairs, D = 64: 5.3 / 9.3
    ("fp32", 8, 2, 64, 32, 200, 824, 0, 1),        # fp32: 7.0 / 11.7
    ("bf16", 32, 8, 128, 1, 400, 800, 0, 1),       # 8 pairs: as compressed ...
    ("bf16", 32, 8, 128, 1, 400, 800, 600, 2),     # ... and grown to 1000 rows: 12.5 / 7.5
    ("bf16", 32, 8, 128, 1, 1500, 100, 0, 1),      # prompts of 100 tokens below the budget (lens): 100 of 1600 rows live
    ("bf16", 32, 8, 128, 1, 200, 3000, 0, 2)])     # 8 pairs with room beyond 2048 rows
def test_decode_form_follows_the_rows_that_live(dtype, Hq, Hkv, D, batch, budget, room, appended, launches):
    lens = [100] if budget == 1500 else [budget + 1 + b % 7 for b in range(batch)]
    wl = small(dtype, Hq, Hkv, D, lens, 16, budget, 5, T=1, name=f"room_{budget}+{room}")
    x = to_dev(synth.make_inputs(wl, 58))
    bufs = H.gpu_compress(wl, x, extra_capacity=room)
    rows = torch.randn((2, batch, Hkv, D), generator=torch.Generator().manual_seed(3)).to(bufs.out.dtype).to(DEV)
    for _ in range(appended):
        bufs.append(rows[0], rows[1])
    assert len(H.captured_launches(lambda: bufs.decode(x["q_dec"][0]))) == launches
    bufs.decode(x["q_dec"][0])
    torch.cuda.synchronize()
    for b in {0, batch - 1}:
        H.check_decode_step(wl, bufs, x["q_dec"][0], b)


def test_decode_of_fewer_rows_than_the_workspace_is_for():
    # room for 4224 rows (17 splits of 256), told that 4000 are the most (32 splits of 128)
    wl = small("bf16", 32, 8, 128, [4300], 16, 4000, 5, T=1, name="tighter_bound")
    x = to_dev(synth.make_inputs(wl, 60))
    bufs = H.gpu_compress(wl, x, extra_capacity=224)
    bufs.decode(x["q_dec"][0], max_cache_len=4000)
    torch.cuda.synchronize()
    H.check_decode_step(wl, bufs, x["q_dec"][0], 0)


@pytest.mark.parametrize("D,budget,threads", [(64, 128, 256), (64, 129, 512), (128, 129, 256)])
def test_waves_of_many_short_caches_with_room(D, budget, threads):
    # 512 pairs with room for 400 rows more: D = 64 has 4 waves for up to 128 live rows, 8 beyond
    wl = small("bf16", 8, 4, D, [budget + 1 + b % 5 for b in range(128)], 16, budget, 5, T=1, name=f"many_room_{budget}")
    x = to_dev(synth.make_inputs(wl, 59))
    bufs = H.gpu_compress(wl, x, extra_capacity=400)
    assert H.captured_launches(lambda: bufs.decode(x["q_dec"][0])) == [(4, 128, 1, threads)]
    bufs.decode(x["q_dec"][0])
    torch.cuda.synchronize()
    for b in (0, 127):
        H.check_decode_step(wl, bufs, x["q_dec"][0], b)


@pytest.mark.parametrize("dtype,D,lens,budget,place", [
    ("bf16", 128, [12288, 60], 300, "pass"),       # splits of 384 rows: the gather rides in the streaming pass
    ("bf16", 128, [12289, 299], 300, "merge"),     # of 512: in the launch that merges; a prompt within the budget beside it
    ("fp32", 64, [200, 150], 260, "merge")])       # nothing to evict, no pass: in the merging launch as well
def test_gather_in_the_pass_and_in_the_merge(dtype, D, lens, budget, place):
    # 16 (sequence, KV head) pairs; 512 and 256 threads a workgroup, so that 16-byte pieces end inside one
    wl = small(dtype, 16, 8, D, lens, 16, budget, 5, T=1, name=f"gather_after_{lens[0]}")
    run_case(wl)
    assert gathered_in(wl) == place


@pytest.mark.parametrize("batch", [96, 97])
def test_split_partials_merged_by_four_groups_or_one(batch):
    # 768 heads are the last that four groups of threads each merge, 776 the first with one group; 11 splits, so that
    # the groups get unequal shares, prompts with fewer splits and with none (within the budget)
    wl = small("fp32", 8, 2, 64, [1400, 60, 129 + 16, 700] + [300 + 7 * b for b in range(batch - 5)] + [1399], 16, 80, 5, T=2,
               name=f"merge_{batch}")
    wl.theta1 = wl.theta2 = 2.0                      # every head is recomputed at every step
    x = to_dev(synth.make_inputs(wl, 85))
    bufs = H.gpu_compress(wl, x)
    rep = {}
    some = (0, 1, 2, 3, batch // 2, batch - 1)
    for b in some:
        H.check_compress(wl, x, bufs, b, report=rep)
    for t in range(wl.decode_steps):
        q_t = x["q_dec"][t]
        bufs.decode(q_t)
        torch.cuda.synchronize()
        before = H.snapshot_state(bufs)
        bufs.recalibrate(q_t, x["k"], x["v"], x["seq_offsets"])
        torch.cuda.synchronize()
        for b in some:
            H.check_recalibrate(wl, x, bufs, q_t, b, before, report=rep)


@pytest.mark.parametrize("dtype,cap", [("fp32", 196608), ("bf16", 393216)])
def test_split_decode_of_small_and_large_caches(dtype, cap):
    # K and V of two such caches are 768 MiB, the most whose first rows are read through the caches; with a third
    # sequence they are read around them.  The splits are the same, so the first two sequences repeat bit for bit
    D, Hkv, Hq = 128, 2, 8
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device=DEV).manual_seed(91)
    lens = [cap, 7001, 33]
    kv = torch.randn((2, Hkv, cap, D), generator=gen, device=DEV, dtype=dt)
    q = torch.randn((3, Hq, D), generator=gen, device=DEV, dtype=dt)
    outs = []
    for nb in (2, 3):
        p = cd.make_params(dtype=cd.BF16 if dtype == "bf16" else cd.FP32, batch=nb, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D,
                           window=16, budget=64, pool_kernel=5)
        bufs = cd.CompressBuffers(p, [64] * nb, DEV, capacities=[cap] * nb)
        for cache, x in ((bufs.k_c, kv[0]), (bufs.v_c, kv[1])):
            cache.view(nb, Hkv, cap, D).copy_(x)
        bufs.cache_lens.copy_(torch.tensor(lens[:nb], dtype=torch.int32))
        bufs.decode(q[:nb].contiguous())
        torch.cuda.synchronize()
        outs.append((bufs.out.clone(), bufs.a_lse.clone()))
    assert torch.equal(outs[0][0], outs[1][0][:2]) and torch.equal(outs[0][1], outs[1][1][:2])
    for b, n in enumerate(lens):
        for h in range(Hq):
            k, v = (x[h // (Hq // Hkv), :n].double() for x in kv)
            z = k @ q[b, h].double() * D ** -0.5
            o = torch.softmax(z, 0) @ v
            assert (outs[1][0][b, h].double() - o).abs().max() < (2e-2 if dtype == "bf16" else 1e-4)
            assert (outs[1][1][b, h].double() - torch.logsumexp(z, 0)).abs() < (2e-3 if dtype == "bf16" else 1e-4)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_scoring_chunks_of_equal_length(dtype):
    # many short prompts of two query-row blocks: one round of 512 workgroups would be 1408 keys each, which are evened
    # out over the longest prompt (1500 keys: two of 768), with prompts that end one short of, at and one past them
    lens = [1500, 767, 768, 769, 1499] + [1090] * 35
    run_case(small(dtype, 40, 8, 64, lens, 64, 80, 7, T=0, name=f"even_chunks_{dtype}"))


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_window_scoring_with_logits_far_above_the_reference(dtype):
    # pass 1 sums against the first logit of each key chunk and redoes a stage against its true
    # maximum only when a sum outgrows 2^64: tiny first keys and a few huge later keys force that
    # path (including fp32 overflow of the first attempt)
    wl = small(dtype, 8, 2, 128, [3000], 16, 128, 5, T=2, name=f"huge_logits_{dtype}")
    x = synth.make_inputs(wl, 77)
    K = synth.seq_view(x["k"], wl, 0)
    K[:, 0] *= 0.01
    K[:, 256] *= 0.01
    K[:, 300] *= 12.0
    K[:, 1500] *= 30.0
    x = to_dev(x)
    bufs = H.gpu_compress(wl, x)
    rep = {}
    H.check_compress(wl, x, bufs, 0, report=rep)
    lse = bufs.region(cd.REGION_ROW_LSE)[:2 * 128].cpu().numpy()
    assert np.isfinite(lse[lse < 1e30]).all() and lse[lse < 1e30].max() > 150.0        # log2 units
    for t in range(wl.decode_steps):
        bufs.decode(x["q_dec"][t])
        torch.cuda.synchronize()
        H.check_decode_step(wl, bufs, x["q_dec"][t], 0, report=rep)
    rep.pop("flags")
    print(wl.name, rep, flush=True)


@pytest.mark.parametrize("n", [1200, 20000])
def test_whole_step_under_hip_graph_replay(n):
    # compress, decode and the recomputation branch allocate nothing, synchronise nothing and
    # record no memset, so the whole per-layer step can live in one captured graph; every
    # replay on fresh inputs must reproduce the eager results (n = 20000 needs more than 48 KiB
    # of dynamic LDS in the selection kernel)
    wl = small("bf16", 8, 2, 128, [n, 700], 16, 128, 5, T=2, name=f"graph_step_{n}")
    xs = [to_dev(synth.make_inputs(wl, 500 + j)) for j in range(3)]
    live = {k: v.clone() for k, v in xs[0].items()}              # the tensors the graph reads
    eager = []
    for x in xs:
        b = H.gpu_compress(wl, x)
        b.decode(x["q_dec"][0])
        b.recalibrate(x["q_dec"][0], x["k"], x["v"], x["seq_offsets"])
        torch.cuda.synchronize()
        eager.append({k: getattr(b, k).clone() for k in ("indices", "k_c", "c_out", "c_lse", "out", "flags", "a_lse")})
    bufs = H.gpu_compress(wl, live)                              # warm-up (also sets the LDS attribute)
    bufs.recalibrate(live["q_dec"][0], live["k"], live["v"], live["seq_offsets"])
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        bufs.compress(live["q_win"], live["k"], live["v"], live["seq_offsets"], stream=side)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            st = torch.cuda.current_stream()
            bufs.compress(live["q_win"], live["k"], live["v"], live["seq_offsets"], stream=st)
            bufs.decode(live["q_dec"][0], stream=st)
            bufs.recalibrate(live["q_dec"][0], live["k"], live["v"], live["seq_offsets"], stream=st)
    for rep_i in range(2):
        for j, x in enumerate(xs):
            for k in live:
                live[k].copy_(x[k])
            bufs.out.zero_(); bufs.indices.zero_(); bufs.c_out.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for k, want in eager[j].items():
                assert torch.equal(getattr(bufs, k), want), (rep_i, j, k)


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("fp32", 64)])
def test_append_grows_the_cache_on_the_device(dtype, D):
    # decode-time tokens are appended (never evicted): calidrop_append writes the new rows at
    # cache_lens and bumps it, all on the device; every step is checked against the oracle on the
    # grown cache, a full cache stays unchanged, and the loop replays from a HIP graph
    wl = small(dtype, 8, 2, D, [700, 60, 900], 16, 96, 5, T=6, name=f"append_{dtype}")
    x = to_dev(synth.make_inputs(wl, 23))
    bufs = H.gpu_compress(wl, x, extra_capacity=4)
    g = torch.Generator(device=DEV).manual_seed(5)
    news = [(torch.randn((3, 2, D), generator=g, device=DEV).to(bufs.k_c.dtype),
             torch.randn((3, 2, D), generator=g, device=DEV).to(bufs.k_c.dtype)) for _ in range(6)]
    lens0 = bufs.cache_lens.clone()
    k0, v0 = bufs.k_c.clone(), bufs.v_c.clone()
    rep = {}
    outs = []
    for t in range(6):
        bufs.append(*news[t])
        bufs.decode(x["q_dec"][t])
        torch.cuda.synchronize()
        for b in range(3):
            L0 = int(lens0[b])
            grown = min(t + 1, bufs.cap - L0)                     # capacity = budget + 4 rows per head
            assert int(bufs.cache_lens[b]) == L0 + grown
            for j in range(grown):
                assert torch.equal(bufs.cache_view("k", b)[:, L0 + j], news[j][0][b])
                assert torch.equal(bufs.cache_view("v", b)[:, L0 + j], news[j][1][b])
            H.check_decode_step(wl, bufs, x["q_dec"][t], b, report=rep)
        outs.append(bufs.out.clone())
    # the same loop from a graph, starting from the same state
    bufs.k_c.copy_(k0); bufs.v_c.copy_(v0); bufs.cache_lens.copy_(lens0)
    got = [torch.empty_like(bufs.out) for _ in range(6)]
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        bufs.decode(x["q_dec"][0], stream=side)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            st = torch.cuda.current_stream()
            for t in range(6):
                bufs.append(*news[t], stream=st)
                bufs.decode(x["q_dec"][t], stream=st)
                got[t].copy_(bufs.out)
    for rep_i in range(2):
        bufs.k_c.copy_(k0); bufs.v_c.copy_(v0); bufs.cache_lens.copy_(lens0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for t in range(6):
            assert torch.equal(got[t], outs[t]), (rep_i, t)


def test_inconsistent_offsets_are_contained_by_the_kernels():
    # seq_offsets lives in device memory, so the host cannot validate it; the kernels treat a
    # sequence whose offsets break the contract (negative length, longer than max_seq_len, beyond
    # total_tokens) as empty and touch nothing of it, while the other sequences are unaffected
    wl = small("bf16", 8, 2, 128, [700, 500, 900], 16, 96, 5, T=1, name="bad_offsets")
    x = to_dev(synth.make_inputs(wl, 31))
    good = H.gpu_compress(wl, x)
    p = H.params_for(wl)
    for bad in ([0, 700, 600, 2100], [0, 700, 700 + 5000, 2100], [0, 700, 1200, 2100 + 64]):
        bufs = cd.CompressBuffers(p, wl.seq_lens, DEV)
        bufs.k_c.fill_(7.0); bufs.v_c.fill_(7.0)
        so = torch.tensor(bad, dtype=torch.int32, device=DEV)
        bufs.compress(x["q_win"], x["k"], x["v"], so)
        bufs.decode(x["q_dec"][0])
        torch.cuda.synchronize()
        broken = [b for b in range(3) if not (0 <= bad[b + 1] - bad[b] <= 900 and bad[b + 1] <= 2100 and bad[b] >= 0)]
        assert broken, bad
        for b in range(3):
            if b in broken:
                assert int(bufs.cache_lens[b]) == 0 and torch.all(bufs.indices[b] == -1)
                assert torch.all(bufs.cache_view("k", b) == 7.0) and torch.all(bufs.cache_view("v", b) == 7.0)
                assert torch.all(torch.isinf(bufs.c_lse[b])) and torch.all(bufs.out[b] == 0)
            elif bad[b] == [0, 700, 1200, 2100][b] and bad[b + 1] == [0, 700, 1200, 2100][b + 1]:
                assert torch.equal(bufs.indices[b], good.indices[b])
                assert torch.equal(bufs.cache_view("k", b), good.cache_view("k", b))
                assert torch.equal(bufs.c_out[b], good.c_out[b])
        assert torch.isfinite(bufs.out.float()).all()


@pytest.mark.parametrize("dtype,D,lens,budget", [("bf16", 128, [900, 40, 3000, 517], 512), ("fp32", 64, [700, 100], 96),
                                                 ("bf16", 64, [5000], 2048), ("bf16", 128, [9000, 300], 4096)])
def test_decode_without_offsets_equals_decode_with_offsets(dtype, D, lens, budget):
    # uniform capacity: leaving cache_offsets out must not change a bit, with full, partly filled
    # (n < budget) and appended caches, in the one-workgroup and in the split form of the step
    wl = small(dtype, 8, 2, D, lens, 16, budget, 5, T=3, name="uniform_offsets")
    x = to_dev(synth.make_inputs(wl, 77))
    bufs = H.gpu_compress(wl, x, extra_capacity=2)
    gen = torch.Generator(device=DEV).manual_seed(9)
    for t in range(3):
        q_t = x["q_dec"][t]
        bufs.decode(q_t, pass_offsets=True)
        want = (bufs.out.clone(), bufs.a_lse.clone(), bufs.flags.clone())
        bufs.out.zero_(); bufs.a_lse.zero_(); bufs.flags.zero_()
        bufs.decode(q_t, pass_offsets=False)
        torch.cuda.synchronize()
        assert torch.equal(bufs.out, want[0]) and torch.equal(bufs.a_lse, want[1]) and torch.equal(bufs.flags, want[2])
        bufs.append(*(torch.randn((len(lens), 2, D), generator=gen, device=DEV).to(bufs.k_c.dtype) for _ in range(2)))


def window_lse_by_library(wl, x):
    """[batch][Hq][w] fp32 log-sum-exp of the window rows over their causal span, by torch.logsumexp
    on dense fp64 logits (what a prefill attention kernel would hand over)."""
    G, w, D = wl.group, wl.window, wl.head_dim
    out = torch.zeros((wl.batch, wl.n_q_heads, w), dtype=torch.float64)
    for b in range(wl.batch):
        n = wl.seq_lens[b]
        if n < w:
            continue
        K = synth.seq_view(x["k"], wl, b).cpu().double()                    # [Hkv][n][D]
        q = x["q_win"][b].cpu().double()                                    # [Hq][w][D]
        S = torch.einsum("hwd,hnd->hwn", q, K.repeat_interleave(G, dim=0)) * D ** -0.5
        col = torch.arange(n).view(1, 1, n)
        row = torch.arange(w).view(1, w, 1)
        out[b] = torch.logsumexp(S.masked_fill(col > n - w + row, float("-inf")), dim=-1)
    return out.to(torch.float32).to(x["k"].device)


@pytest.mark.parametrize("dtype,D,lens,w,B,m", [("fp32", 64, [700, 50, 1300], 16, 96, 0), ("bf16", 128, [2100, 9000], 32, 256, 0),
                                                ("bf16", 64, [20000], 16, 300, 500), ("bf16", 128, [900], 12, 64, 0)])
def test_compress_with_the_window_log_sum_exp_supplied(dtype, D, lens, w, B, m):
    # pass 1 skipped: the normalisers come from the caller.  Exact ones reproduce the default call's
    # result (same oracle, same protocol); ones that are off by per-row constants are used as given
    wl = small(dtype, 8, 2, D, lens, w, B, 5, T=1, name="supplied_lse")
    x = to_dev(synth.make_inputs(wl, 41))
    lse = window_lse_by_library(wl, x)
    bufs = H.gpu_compress(wl, x, win_lse=lse, calib_size=m)
    for b in range(wl.batch):
        H.check_compress(wl, x, bufs, b)
    g = torch.Generator(device=DEV).manual_seed(3)
    skew = lse + torch.randn(lse.shape, generator=g, device=DEV) * 0.7
    bufs2 = H.gpu_compress(wl, x, win_lse=skew, calib_size=m)
    for b in range(wl.batch):
        H.check_compress(wl, x, bufs2, b, win_lse=skew)


@pytest.mark.parametrize("wl", [
    small("bf16", 8, 2, 128, [900, 40, 2100], 16, 128, 5, T=2, name="no_export_8_per_thread"),
    small("bf16", 8, 2, 64, [9000, 12000], 16, 300, 5, T=2, name="no_export_16_per_thread"),
    small("fp32", 4, 2, 64, [20000, 500], 16, 200, 7, T=2, name="no_export_32_per_thread"),
], ids=lambda w: w.name)
def test_compress_with_default_options_no_score_export(wl):
    # flags = 0 is what a caller (and the benchmark) uses: the selection kernel then skips the store
    # of the pooled scores.  Same checks as everywhere else minus the scores, and bit-identical
    # outputs to the call that exports them.
    x = to_dev(synth.make_inputs(wl, 88))
    bufs = H.gpu_compress(wl, x, flags=0)
    twin = H.gpu_compress(wl, x, flags=cd.OPT_WRITE_SCORES)
    rep = {}
    for b in range(wl.batch):
        H.check_compress(wl, x, bufs, b, report=rep)
    assert "score_rel_err" not in rep
    for name in ["indices", "k_c", "v_c", "c_out", "c_lse", "c_q", "cache_lens"]:
        assert torch.equal(getattr(bufs, name), getattr(twin, name)), name
    for t in range(2):
        bufs.decode(x["q_dec"][t])
        torch.cuda.synchronize()
        for b in range(wl.batch):
            H.check_decode_step(wl, bufs, x["q_dec"][t], b, report=rep)


def test_first_library_call_of_a_process_may_be_under_stream_capture():
    # the only host-side setting the library makes (the dynamic-LDS limit of the selection kernel, once
    # per device) enqueues nothing, so even the very first call of a process can be captured: a fresh
    # interpreter captures compress + decode of a prompt whose selection needs more than 48 KiB of LDS
    # without any warm-up, replays the graph and compares with eager calls made afterwards
    import subprocess
    import sys
    code = r"""
import torch
from paper_2507_19906_amd import binding as cd, synth
wl = synth.Workload("capture_first", 2, 8, 2, 128, [20000, 700], 16, 128, 5, "bf16", 1)
x = {k: v.to("cuda:0") for k, v in synth.make_inputs(wl, 501).items()}
p = cd.make_params(dtype="bf16", batch=2, n_q_heads=8, n_kv_heads=2, head_dim=128, window=16, budget=128, pool_kernel=5)
a, b = cd.CompressBuffers(p, wl.seq_lens, "cuda:0"), cd.CompressBuffers(p, wl.seq_lens, "cuda:0")
torch.cuda.synchronize()
side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
with torch.cuda.stream(side):
    with torch.cuda.graph(graph, stream=side):
        st = torch.cuda.current_stream()
        a.compress(x["q_win"], x["k"], x["v"], x["seq_offsets"], stream=st)
        a.decode(x["q_dec"][0], stream=st)
torch.cuda.synchronize()
for rep in range(2):
    a.out.zero_(); a.indices.zero_(); a.c_out.zero_()
    torch.cuda.synchronize()
    graph.replay()
    torch.cuda.synchronize()
    if rep == 0:
        b.compress(x["q_win"], x["k"], x["v"], x["seq_offsets"])
        b.decode(x["q_dec"][0])
        torch.cuda.synchronize()
    for name in ("indices", "k_c", "v_c", "c_out", "c_lse", "out", "a_lse", "flags"):
        assert torch.equal(getattr(a, name), getattr(b, name)), (rep, name)
assert int(a.indices[0, 0, -1]) == 19999
print("captured first call ok")
"""
    import os
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=240, cwd=root)
    assert r.returncode == 0 and "captured first call ok" in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]
