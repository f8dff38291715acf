"""GPU kernels at the sizes where they can go wrong (tile edges, remainders, smallest and largest of a dispatch
range), against the float64 oracle.  Tolerances as in test_gpu_parity.py: derived there from the storage type."""
import numpy as np
import pytest
import torch

from esa_inputs import segment_bounds
from oracle import esa_oracle as orc
from support import f64_to_dev, to_f64
from test_gpu_parity import F_TOL, O_TOL, bf16_ulp, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def esa():
    import paper_2502_14477_amd as lib
    return lib


def attend_inputs(seed, dtype, B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel):
    rng = np.random.default_rng(seed)
    S = t0 + l_C
    q = orc.round_to_storage(rng.standard_normal((B, l_C, H, d)), dtype)
    K = orc.round_to_storage(rng.standard_normal((B, S, H_kv, d)), dtype)
    V = orc.round_to_storage(rng.standard_normal((B, S, H_kv, d)), dtype)
    i_end, l_start = segment_bounds(t0, l_I, l_L)
    sel = np.stack([np.sort(rng.choice(np.arange(i_end, l_start), n_sel, replace=False)) for _ in range(B)]).astype(np.int32) \
        if n_sel else np.empty((B, 0), np.int32)
    return q, K, V, sel


def attend_reencoded_rounded(q, K, V, t0, l_I, l_L, sel, w, base):
    """The oracle's Section 3.2 over bf16 rows: each encoded query and key is rounded once."""
    l_C, l_start = q.shape[0], segment_bounds(t0, l_I, l_L)[1]
    K_l = np.zeros_like(K)
    K_l[l_start:t0 + l_C] = orc.rope(K[l_start:t0 + l_C], np.arange(t0 + l_C - l_start), base)
    q_l, q_g = orc.rope(q, t0 - l_start + np.arange(l_C), base), orc.rope(q, np.full(l_C, w), base)
    q_l, q_g, K_l = (orc.round_to_storage(x, "bf16") for x in (q_l, q_g, K_l))
    return orc.attend_two_encodings(q_l, q_g, K_l, K, V, t0, l_I, l_L, sel, 1.0 / np.sqrt(q.shape[2]))


# one token of a 32-row wave tile more or less, row tiles of unequal filling, one slice and many, every group size
@pytest.mark.parametrize("B,H,H_kv,d,t0,l_C,l_I,l_L,n_sel", [
    (1, 4, 4, 64, 900, 16, 8, 64, 31), (1, 8, 4, 64, 700, 17, 8, 100, 64), (2, 8, 2, 64, 1000, 65, 0, 130, 129),
    (1, 16, 2, 64, 1100, 33, 16, 64, 200), (1, 8, 2, 64, 0, 63, 16, 64, 0), (1, 32, 8, 64, 3000, 257, 128, 512, 700),
    (1, 32, 8, 64, 3000, 41, 128, 1000, 1500), (2, 32, 8, 64, 3000, 41, 128, 1000, 1500), (1, 8, 8, 64, 3000, 399, 16, 1000, 700),      # few bytes of slices, many
    (1, 16, 2, 128, 1100, 33, 16, 64, 200), (2, 8, 2, 128, 1000, 65, 0, 130, 129), (1, 8, 8, 128, 700, 259, 8, 100, 64)])
def test_matrix_core_attention_head_sizes_and_row_tiles(esa, B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel):
    say(f"attend B={B} H={H} H_kv={H_kv} d={d} t0={t0} l_C={l_C} l_I={l_I} l_L={l_L} n_sel={n_sel}")
    q, K, V, sel = attend_inputs(d + l_C, "bf16", B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)
    qd, Kd, Vd, idx = f64_to_dev(q, "bf16"), f64_to_dev(K, "bf16"), f64_to_dev(V, "bf16"), torch.from_numpy(sel).cuda()
    O, lse = esa.esa_attend_indexed(qd, Kd, Vd, t0, l_I, l_L, idx, return_lse=True)
    ks, vs = esa.esa_gather_kv(Kd, Vd, idx) if n_sel else (None, None)
    O_re = esa.esa_attend_reencoded(qd, Kd, Vd, t0, l_I, l_L, ks, vs, 4096.0, 5e5)
    for b in range(B):
        want, want_lse = orc.attend(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d))
        assert np.max(np.abs(to_f64(O[b]) - want)) <= O_TOL["bf16"]
        assert np.max(np.abs(to_f64(lse[b]) - want_lse)) <= 1e-3
        want, _ = orc.attend_reencoded(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d), 4096.0, 5e5)
        assert np.max(np.abs(to_f64(O_re[b]) - want)) <= O_TOL["bf16"]


# Rows and pointers that are not 16-byte aligned: every head size but 128 takes them, in one call, in two and re-encoded
@pytest.mark.parametrize("dtype,d,l_C,pad,shift", [("bf16", 64, 40, 4, 0), ("bf16", 64, 16, 0, 1), ("bf16", 64, 3, 4, 1), ("f32", 32, 20, 1, 0)])
def test_head_sizes_that_take_unaligned_rows(esa, dtype, d, l_C, pad, shift):
    say(f"unaligned rows {dtype} d={d} l_C={l_C} pad={pad} shift={shift}")
    H, H_kv, t0, l_I, l_L, n_sel = 8, 2, 700, 16, 130, 90
    q, K, V, sel = attend_inputs(d + l_C, dtype, 1, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)
    q, K, V, sel = q[0], K[0], V[0], sel[0]

    def rows(x):                    # token rows `pad` elements apart, the first one `shift` elements into its buffer
        x = f64_to_dev(x, dtype)
        n, width = x.shape[0], x.shape[1] * d
        buf = torch.zeros(n * (width + pad) + shift, dtype=x.dtype, device="cuda")
        view = buf[shift:].as_strided((n, x.shape[1], d), (width + pad, d, 1), shift)
        view.copy_(x)
        return view

    qd, Kd, Vd, idx = f64_to_dev(q, dtype), rows(K), rows(V), torch.from_numpy(sel).cuda()
    ks, vs = esa.esa_gather_kv(Kd, Vd, idx)
    want, _ = orc.attend(q, K, V, t0, l_I, l_L, sel, 1.0 / np.sqrt(d))
    got = [esa.esa_attend_indexed(qd, Kd, Vd, t0, l_I, l_L, idx), esa.esa_attend(qd, Kd, Vd, t0, l_I, l_L, ks, vs)]
    for split in (esa.ESA_SPLIT_I_EARLY, esa.ESA_SPLIT_ALGORITHM1):
        for k_cache, v_cache, k_sel in ((Kd, Vd, ks), (f64_to_dev(K, dtype), f64_to_dev(V, dtype), ks), (Kd, Vd, rows(to_f64(ks)) if pad == 0 else ks)):
            esa.esa_attend_local(qd, k_cache, v_cache, t0, l_I, l_L, split=split)
            got.append(esa.esa_attend_finish(qd, k_cache, v_cache, t0, l_I, l_L, k_sel, vs, split=split))
    for O in got:
        assert np.max(np.abs(to_f64(O) - want)) <= O_TOL[dtype]
    want, _ = orc.attend_reencoded(q, K, V, t0, l_I, l_L, sel, 1.0 / np.sqrt(d), 4096.0, 5e5)
    O = esa.esa_attend_reencoded(qd, Kd, Vd, t0, l_I, l_L, ks, vs, 4096.0, 5e5)
    assert np.max(np.abs(to_f64(O) - want)) <= O_TOL[dtype]


# Probabilities and partial sums in fp32: a few tokens, and head size 64 at any length.  Outputs are then off by about
# 2^-22 of their rms, so that one in a thousand or two is not the bf16 number nearest to the exact result (an output's
# last place is 2^-8 of itself or less; small outputs count most).  Probabilities of 16 bits, 2^-17.8 of the rms, leave
# 2.3e-3 of them elsewhere, probabilities of 8 bits 0.4.
@pytest.mark.parametrize("H,H_kv,d,l_C", [(32, 8, 128, 5), (16, 2, 128, 15), (32, 8, 64, 9), (32, 8, 64, 40), (16, 2, 64, 96), (8, 8, 64, 33)])
def test_attention_outputs_are_the_exact_ones_rounded(esa, H, H_kv, d, l_C):
    say(f"attend, nearest outputs H={H} H_kv={H_kv} d={d} l_C={l_C}")
    t0, l_I, l_L, n_sel = 6000, 128, 2048, 2048
    q, K, V, sel = attend_inputs(d + l_C, "bf16", 1, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)
    O = esa.esa_attend_indexed(f64_to_dev(q[0], "bf16"), f64_to_dev(K[0], "bf16"), f64_to_dev(V[0], "bf16"), t0, l_I, l_L,
                               torch.from_numpy(sel[0]).cuda())
    want, _ = orc.attend(q[0], K[0], V[0], t0, l_I, l_L, sel[0], 1.0 / np.sqrt(d))
    elsewhere = np.mean(to_f64(O) != orc.round_to_storage(want, "bf16"))
    print(f"{elsewhere:.2e} of {want.size} outputs are not the nearest", flush=True)
    assert elsewhere <= 1.5e-3


# Two tiles of one slice, the second with the larger logit (head size 64, where the reference follows the maximum at once): the
# sum of exponentials moves to the new reference and takes the new tile's 1 with one rounding.  (Rounded twice, a fifth of these
# sums are another number.)  The logits are products of two bf16 numbers, so everything up to the sum is known exactly but for
# the exponentials, which torch takes from the same instruction.
def test_sum_of_exponentials_is_rounded_once_when_its_reference_moves(esa):
    say("attend, one slice of two tiles")
    B, H, d, l_C, t0 = 32, 8, 64, 16, 128
    rng = np.random.default_rng(d)
    bf = lambda x: torch.from_numpy(np.asarray(x, np.float32)).bfloat16()
    a = bf(1.0 + rng.random((B, l_C, H)))                       # the only component of a query
    b = bf(-rng.random((2, B, H)) * 0.6 - 0.05)                 # ... of keys 0 and 1; key 64 has logit 0, all others vanish
    q = torch.zeros((B, l_C, H, d), dtype=torch.bfloat16)
    K = torch.zeros((B, t0 + l_C, H, d), dtype=torch.bfloat16)
    q[..., 0] = a
    K[..., 0] = -1024.0
    K[:, 0, :, 0], K[:, 1, :, 0], K[:, 64, :, 0] = b[0], b[1], 0.0
    V = torch.zeros_like(K)
    _, lse = esa.esa_attend(q.cuda(), K.cuda(), V.cuda(), t0, 64, 64, None, None, scale=1.0, return_lse=True)

    f32 = lambda x: x.to(torch.float32)
    c2 = float(np.float32(1.4426950408889634))
    s = a.double()[None] * b.double()[:, :, None, :]             # exact, as are the differences below in float64
    m = f32(s.max(0)[0] * c2)
    p = torch.exp2(f32(s * c2 - m.double()).cuda()).cpu()
    first = p[0] + p[1]
    corr = torch.exp2(m.cuda()).cpu()
    total = f32(first.double() * corr.double() + 1.0)
    twice = first * corr + 1.0
    want, other = torch.log(total.cuda()).double(), torch.log(twice.cuda()).double()
    # one place of the sum apart, 1 to 1.2e-7 / sum: at most two places of the logarithm, which itself errs by up to one: it cannot
    # hide the difference in more than half of the rows, and a sum that is rounded twice is nearer in none but those
    told = want != other
    near = float(((lse - want).abs() < (lse - other).abs())[told].double().mean())
    print(f"{float(told.double().mean()):.2f} of the rows tell, {near:.3f} of these are nearer to one rounding", flush=True)
    assert told.sum() > 400 and near > 0.5


# the shortest shares, shares with every number of load groups in flight, two blocks of queries; the first block through LDS
# (more than 192 queries): behind a short share, in the place of the last tiles of a long one, a block that is not full
@pytest.mark.parametrize("B,l_c,n,d_c,eps", [(1, 40, 1, 64, 0), (1, 64, 8193, 64, 0), (2, 512, 33000, 64, 0), (1, 530, 66000, 64, 1),
                                             (1, 20, 131072, 64, 0), (1, 96, 40000, 128, 0), (1, 192, 33000, 128, 0), (1, 193, 20, 128, 0),
                                             (2, 500, 20000, 128, 0), (1, 257, 40000, 128, 0), (1, 700, 131072, 128, 0), (1, 449, 66000, 128, 1),
                                             # later blocks through LDS, whole, by halves and not: the longest shares that leave room and one token more, last
                                             # blocks of few and all waves
                                             (1, 513, 16384, 128, 0), (1, 1537, 16385, 128, 0), (1, 1025, 81920, 128, 0), (1, 1025, 81921, 128, 0), (1, 600, 32768, 128, 0), (1, 600, 32769, 128, 0), (1, 2049, 700, 128, 2), (3, 1024, 5000, 128, 0), (1, 1100, 131072, 64, 0), (2, 1500, 131072, 64, 0)])
def test_matrix_core_score_sweeps(esa, B, l_c, n, d_c, eps):
    say(f"score B={B} l_c={l_c} n={n} d_c={d_c} eps={eps}")
    rng = np.random.default_rng(n + l_c)
    qc = orc.round_to_storage(rng.standard_normal((B, l_c, d_c)) * 1.5, "bf16")
    kc = orc.round_to_storage(rng.standard_normal((B, n + 8, d_c)), "bf16")
    got = to_f64(esa.esa_score(f64_to_dev(qc, "bf16"), f64_to_dev(kc, "bf16"), 3, n + 3, eps=eps))
    for b in range(B):
        want = orc.importance(qc[b], kc[b, 3:n + 3])
        want = orc.proximity(want, eps) if eps else want
        assert np.max(np.abs(got[b] - want)) <= F_TOL["bf16"]
        assert got[b].max() == 0.0


# Shares of whole rounds of workgroups: the longest row of one round and one token more, rows of two rounds and of three, several
# sequences whose shares together make a round, one more than that; rows that each round up to a share too many; the longest row that the second
# sweep pools in one round, one that it does not
@pytest.mark.parametrize("B,l_c,n,d_c,eps", [(1, 17, 131072, 64, 0), (1, 17, 131073, 64, 0), (1, 33, 140000, 128, 0), (1, 20, 263000, 64, 1), (4, 64, 20000, 128, 0),
                                             (2, 70, 65536, 64, 0), (2, 70, 65537, 64, 2), (300, 20, 70, 64, 0), (3, 20, 10894, 64, 0), (7, 40, 4661, 128, 1), (24, 17, 18849, 64, 0),
                                             (1, 33, 130560, 64, 1), (1, 33, 130561, 64, 1), (1, 300, 131072, 128, 16)])
def test_score_sweeps_in_whole_rounds(esa, B, l_c, n, d_c, eps):
    say(f"score rounds B={B} l_c={l_c} n={n} d_c={d_c} eps={eps}")
    g = torch.Generator(device="cuda").manual_seed(n + l_c)
    qc, kc = (torch.randn((B, m, d_c), generator=g, device="cuda").bfloat16() for m in (l_c, n + 8))
    got = esa.esa_score(qc, kc, 3, n + 3, eps=eps)
    for b in range(0, B, max(1, B // 2)):
        want = orc.importance(to_f64(qc[b]), to_f64(kc[b, 3:n + 3]))
        want = orc.proximity(want, eps) if eps else want
        assert np.max(np.abs(to_f64(got[b]) - want)) <= F_TOL["bf16"], b
        assert got[b].max() == 0.0


# How a workgroup's waves share out queries and tiles changes no bit: the same queries once, in few waves, and again and again, in all eight.
# Shares of two, four and six tiles, of sixteen, two to a workgroup; up to 64, 128 and 256 queries and one more
@pytest.mark.parametrize("d_c", [64, 128])
@pytest.mark.parametrize("n", [16384, 16385, 32768, 32769, 131072, 140000])
@pytest.mark.parametrize("l_c", [17, 64, 65, 128, 129, 256])
def test_waves_that_share_queries_find_the_same_scores(esa, l_c, n, d_c):
    say(f"score by shared waves l_c={l_c} n={n} d_c={d_c}")
    g = torch.Generator(device="cuda").manual_seed(n + l_c)
    qc, kc = (torch.randn((m, d_c), generator=g, device="cuda").bfloat16() for m in (l_c, n))
    got = esa.esa_score(qc, kc, 0, n)
    assert torch.equal(got, esa.esa_score(qc.repeat(512 // l_c + 1, 1)[:512], kc, 0, n))
    some = torch.randperm(n, generator=g, device="cuda")[:64]
    S = qc.double() @ kc.double().T
    want = (S - S.max(dim=1, keepdim=True).values).max(dim=0).values[some]
    assert (got[some].double() - want).abs().max().item() <= F_TOL["bf16"]


# No workgroup of the sweeps depends on another one's being resident: told to wait for 0 or 2 us only, they do each other's row maxima,
# and the scores have the same bits.  One share, a few, a round of them, two rounds, several rows; both query paths, several blocks of queries
@pytest.mark.parametrize("B,l_c,n,d_c,eps", [(1, 20, 30, 128, 0), (1, 40, 20000, 64, 1), (1, 77, 48000, 128, 0), (1, 530, 130000, 128, 0),
                                             (1, 300, 140000, 128, 3), (3, 40, 70000, 128, 0), (2, 512, 33000, 128, 0), (1, 1300, 9000, 128, 0), (3, 600, 70000, 64, 0)])
def test_score_sweeps_that_do_not_wait_for_each_other(esa, B, l_c, n, d_c, eps):
    import ctypes
    say(f"score without waiting B={B} l_c={l_c} n={n} d_c={d_c} eps={eps}")
    g = torch.Generator(device="cuda").manual_seed(n + l_c)
    qc, kc = (torch.randn((B, m, d_c), generator=g, device="cuda").bfloat16() for m in (l_c, n + 8))
    want = esa.esa_score(qc, kc, 3, n + 3, eps=eps)
    call = ctypes.CDLL(esa.lib_path()).esa_internal_score_waiting
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    i64 = ctypes.c_int64
    size = esa.lib.esa_score_workspace_bytes(l_c, n, eps, B)
    for ticks in (0, 200):
        got, ws = torch.full_like(want, 7.0), torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
        rc = call(ptr(qc), l_c, ptr(kc), i64(3), i64(n + 3), d_c, eps, ptr(got), esa.ESA_BF16, B, i64(l_c * d_c), i64((n + 8) * d_c), i64(n),
                  ptr(ws), ctypes.c_size_t(size), ticks, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == 0 and torch.equal(got, want), ticks


def test_score_of_many_rows_costs_what_its_rows_cost(esa):
    """A workgroup finds a share's row in a time that does not grow with the number of rows: four times as many rows take about four times
    as long, and below eight times (looked for row by row they took 11.1 times as long; 4.0 now)."""
    say("score of 1024 and 4096 rows")
    g = torch.Generator(device="cuda").manual_seed(11)
    qc, kc = (torch.randn((4096, m, 128), generator=g, device="cuda").bfloat16() for m in (17, 600))
    took = {}
    for B in (1024, 4096):
        best = None
        for _ in range(5):                             # the first one warms up
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                got = esa.esa_score(qc[:B], kc[:B], 0, 600)
            b.record()
            b.synchronize()
            best = a.elapsed_time(b) if best is None else min(best, a.elapsed_time(b))
        took[B] = best
        for row in (0, 511, B - 1):
            want = orc.importance(to_f64(qc[row]), to_f64(kc[row]))
            assert np.max(np.abs(to_f64(got[row]) - want)) <= F_TOL["bf16"], row
    assert took[4096] < 8 * took[1024], took


def test_score_sweeps_on_several_streams_at_once(esa):
    """Calls that compete for the compute units, each workgroup of which waits for the others of its call: the same bits, and an end."""
    say("score on four streams")
    g = torch.Generator(device="cuda").manual_seed(8)
    shapes = [(77, 48000), (512, 130000), (300, 60000), (20, 128000)]
    data = [tuple(torch.randn((m, 128), generator=g, device="cuda").bfloat16() for m in (l_c, n)) for l_c, n in shapes]
    want = [esa.esa_score(q, k, 0, k.shape[0]) for q, k in data]
    streams = [torch.cuda.Stream() for _ in data]
    torch.cuda.synchronize()
    for _ in range(5):
        got = []
        for s, (q, k) in zip(streams, data):
            with torch.cuda.stream(s):
                got += [esa.esa_score(q, k, 0, k.shape[0]) for _ in range(4)]
        torch.cuda.synchronize()
        for i, g_ in enumerate(got):
            assert torch.equal(g_, want[i // 4]), i


# Pooling by the second sweep: one workgroup's tokens, one more, one less; a single token; the widest window it takes in the shortest
# share and in long ones, the narrowest, one that keeps its own pass; windows across every workgroup's edge hold the row's largest scores
@pytest.mark.parametrize("B,l_c,n,d_c,eps", [(1, 17, 1, 128, 1), (2, 40, 62, 128, 1), (1, 40, 63, 128, 1), (1, 20, 61, 64, 1), (1, 33, 32, 64, 16),
                                             (1, 33, 4097, 64, 16), (1, 600, 33000, 128, 16), (1, 70, 131077, 128, 2), (3, 40, 9000, 128, 3), (1, 70, 131000, 128, 2),
                                             (1, 33, 500, 128, 17)])
def test_pooling_in_the_second_sweep(esa, B, l_c, n, d_c, eps):
    say(f"score B={B} l_c={l_c} n={n} d_c={d_c} eps={eps}")
    rng = np.random.default_rng(n + l_c)
    qc = orc.round_to_storage(rng.standard_normal((B, l_c, d_c)) * 1.5, "bf16")
    kc = orc.round_to_storage(rng.standard_normal((B, n + 8, d_c)), "bf16")
    qd, kd, k = f64_to_dev(qc, "bf16"), f64_to_dev(kc, "bf16"), max(n // 3, 1)
    score = esa.esa_score(qd, kd, 3, n + 3, eps=eps)
    fused, idx, _, _ = esa.esa_score_select_gather(qd, kd, 3, n + 3, k, eps=eps)
    assert n <= k or torch.equal(fused, score)
    assert torch.equal(idx, esa.esa_select_topk(score, k, base=3))
    raw = to_f64(esa.esa_score(qd, kd, 3, n + 3))
    for b in range(B):
        want = orc.proximity(orc.importance(qc[b], kc[b, 3:n + 3]), eps)
        assert np.max(np.abs(to_f64(score[b]) - want)) <= F_TOL["bf16"]
        assert np.array_equal(to_f64(score[b]), orc.proximity(raw[b], eps))         # the same scores, pooled


def _bin_crowd(rng, n, crowd, kind):
    """Scores of which `crowd` lie so close below -1 that they share a bin of a short row's histogram and the first digits of a long row's."""
    s = (-2.0 - rng.random(n) * 60.0).astype(np.float32)
    at = rng.choice(n, crowd, replace=False) if kind != "run" else np.arange(n // 3, n // 3 + crowd)
    s[at] = np.float32(-1.0) - (np.float32(0.0) if kind == "equal" else rng.random(crowd).astype(np.float32) * np.float32(2 ** -7))
    s[rng.choice(n, 40, replace=False)] = np.linspace(-0.9, 40.0, 40).astype(np.float32)        # both signs above it
    return s


# around the longest row one workgroup takes; scores that share many leading bits, or all of them
@pytest.mark.parametrize("n,k,crowd,kind", [
    (1024, 1023, 900, "spread"), (8192, 2048, 5000, "spread"), (8193, 2048, 2040, "spread"), (8192, 700, 3000, "equal"),
    (40000, 500, 1900, "run"), (100000, 2048, 2100, "spread"), (100000, 900, 2000, "equal"), (100000, 60000, 90000, "equal")])
def test_select_topk_where_the_threshold_bin_is_crowded(esa, n, k, crowd, kind):
    say(f"select n={n} k={k} crowd={crowd} {kind}")
    rng = np.random.default_rng(n + crowd)
    s = np.stack([_bin_crowd(rng, n, crowd, kind) for _ in range(2)])
    got = esa.esa_select_topk(torch.from_numpy(s).cuda(), k, base=5).cpu().numpy()
    for b in range(2):
        order = np.lexsort((np.arange(n), -s[b].astype(np.float64)))[:k]
        assert np.array_equal(got[b], np.sort(order) + 5)


# rows whose scores lie together far from zero (one token stands out of a decode step), of any scale, with infinities and
# masked entries
@pytest.mark.parametrize("n,k,centre,spread", [(260000, 2048, -500.0, 11.0), (9001, 700, 3e4, 5.0), (100000, 8192, 0.0, 1e-6),
                                               (8193, 8192, -1e6, 0.01), (20000, 1, 1e31, 1e28), (50000, 25000, 40.0, 1e-5)])
def test_selection_from_scores_far_from_zero(esa, n, k, centre, spread):
    say(f"select n={n} k={k} centre={centre} spread={spread}")
    rng = np.random.default_rng(n + k)
    s = (centre + spread * rng.standard_normal((2, n))).astype(np.float32)
    s[1, rng.choice(n, n // 3, replace=False)] = np.float32(-3e38)
    s[1, rng.choice(n, 5, replace=False)] = -np.inf
    s[1, 17] = np.inf
    got = esa.esa_select_topk(torch.from_numpy(s).cuda(), k, base=3).cpu().numpy()
    for b in range(2):
        order = np.lexsort((np.arange(n), -s[b].astype(np.float64)))[:k]
        assert np.array_equal(got[b], np.sort(order) + 3)


def _time_us(call, passes=20):
    """Median device time of a call, in microseconds."""
    call()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(passes):
            call()
    times = []
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        graph.replay()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / passes)
    return sorted(times)[3]


# The selection's time does not depend on how the scores lie: tokens of a passage score alike, a row lies far from zero, one
# query of a chunk is much larger than the others (its row maximum, too).  Twice the time of N(0, 1) scores leaves room for
# noise; a selection whose lists overflowed took 5 to 11 times as long.
@pytest.mark.parametrize("kind", ["passage", "far", "pooled"])
def test_selection_time_does_not_depend_on_the_scores(esa, kind):
    say(f"select, {kind} scores against N(0, 1)")
    n, k = 200000, 2048
    g = torch.Generator(device="cuda").manual_seed(11)
    plain = torch.randn(n, generator=g, device="cuda")
    s = 3.0 * plain - 100.0
    if kind == "passage":
        s[1000:4000] = -30.0 + 0.3 * plain[1000:4000]
    elif kind == "far":
        s = plain - 700.0
    else:
        s = torch.nn.functional.max_pool1d(s[None], 33, 1, 16)[0].contiguous()
    a, b = _time_us(lambda: esa.esa_select_topk(plain, k)), _time_us(lambda: esa.esa_select_topk(s, k))
    print(f"{a:.1f} us, {kind} {b:.1f} us", flush=True)
    assert b <= 2.0 * a
    order = np.lexsort((np.arange(n), -s.cpu().numpy().astype(np.float64)))[:k]
    assert np.array_equal(esa.esa_select_topk(s, k).cpu().numpy(), np.sort(order))


@pytest.mark.parametrize("l_c", [5, 64])
def test_selection_time_does_not_depend_on_one_large_query(esa, l_c):
    say(f"score and select, {l_c} queries of which the first is large")
    n, k = 100000, 2048
    g = torch.Generator(device="cuda").manual_seed(l_c)
    q = torch.randn((l_c, 128), generator=g, device="cuda").to(torch.bfloat16)
    kc = torch.randn((n, 128), generator=g, device="cuda").to(torch.bfloat16)
    large = q.clone()
    large[0] *= 50.0
    a, b = _time_us(lambda: esa.esa_score_select_gather(q, kc, 0, n, k)), _time_us(lambda: esa.esa_score_select_gather(large, kc, 0, n, k))
    print(f"{a:.1f} us, one large query {b:.1f} us", flush=True)
    assert b <= 2.0 * a
    score, idx, _, _ = esa.esa_score_select_gather(large, kc, 0, n, k)
    order = np.lexsort((np.arange(n), -score.cpu().numpy().astype(np.float64)))[:k]
    assert np.array_equal(idx.cpu().numpy(), np.sort(order))


# local and global part of a re-encoded attention laid end to end: one slice of both, the seam inside a slice and between two,
# a part of one tile, parts that end inside a tile
@pytest.mark.parametrize("B,H,H_kv,d,t0,l_C,l_I,l_L,n_sel", [
    (33, 8, 8, 128, 700, 40, 16, 100, 130), (40, 8, 8, 64, 300, 17, 3, 70, 90), (1, 8, 2, 64, 1200, 70, 5, 63, 300),
    (1, 8, 8, 128, 900, 16, 64, 48, 64), (2, 16, 2, 128, 1500, 33, 1, 700, 1), (1, 32, 8, 128, 3000, 65, 128, 1000, 130)])
def test_reencoded_attention_over_slices_of_both_parts(esa, B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel):
    say(f"attend_reencoded B={B} H={H} H_kv={H_kv} d={d} t0={t0} l_C={l_C} l_I={l_I} l_L={l_L} n_sel={n_sel}")
    q, K, V, sel = attend_inputs(d + l_C, "bf16", B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)
    Kd, Vd = f64_to_dev(K, "bf16"), f64_to_dev(V, "bf16")
    ks, vs = esa.esa_gather_kv(Kd, Vd, torch.from_numpy(sel).cuda())
    O = esa.esa_attend_reencoded(f64_to_dev(q, "bf16"), Kd, Vd, t0, l_I, l_L, ks, vs, 4096.0, 5e5)
    for b in range(B):
        want, _ = orc.attend_reencoded(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d), 4096.0, 5e5)
        assert np.max(np.abs(to_f64(O[b]) - want)) <= O_TOL["bf16"], b


# The softmax reference moves (head size 128: when half a tile's exponentials add up to too much): `rises` are virtual keys from which
# on all logits are larger by 10.  In either half of the first tile, of a later one, of the last that every row sees, of the causal
# one; several in a row; a first half far below the rest; slices of nine to twenty tiles, whose rows are found eight tiles at a time.
@pytest.mark.parametrize("B,H,H_kv,d,t0,l_C,l_I,l_L,n_sel,rises", [
    (1, 8, 8, 128, 400, 16, 64, 128, 90, (5,)), (1, 8, 8, 128, 400, 16, 64, 128, 90, (40, 70, 100, 130, 161)), (2, 8, 2, 128, 500, 40, 10, 300, 64, (32, 64, 352)),
    (1, 8, 2, 128, 500, 70, 10, 300, 64, (374, 400, 410)), (1, 32, 8, 128, 300, 65, 10, 200, 64, (276, 300, 338)), (1, 8, 2, 64, 500, 70, 10, 300, 64, (40, 374, 400)),
    (4, 8, 8, 128, 9000, 16, 100, 2000, 3000, (2000,)), (1, 64, 64, 128, 9000, 17, 100, 2000, 3001, ()), (4, 8, 8, 64, 9000, 16, 100, 2000, 3000, (30,))])
def test_attention_where_the_reference_moves_and_over_long_slices(esa, B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel, rises):
    say(f"attend, moving reference B={B} H={H} H_kv={H_kv} d={d} t0={t0} l_C={l_C} l_I={l_I} l_L={l_L} n_sel={n_sel} rises={rises}")
    q, K, V, sel = attend_inputs(d + l_C, "bf16", B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)
    i_end, l_start = segment_bounds(t0, l_I, l_L)
    q[..., 0] = 8.0
    for b in range(B):
        rows = np.concatenate([np.arange(i_end), sel[b], np.arange(l_start, t0 + l_C)])       # the virtual keys' rows
        level = sum((np.arange(rows.size) >= r).astype(float) for r in rises) if rises else np.zeros(rows.size)
        K[b, rows, :, 0] = orc.round_to_storage(10.0 * np.sqrt(d) / 8.0 * level, "bf16")[:, None]
    qd, Kd, Vd, idx = f64_to_dev(q, "bf16"), f64_to_dev(K, "bf16"), f64_to_dev(V, "bf16"), torch.from_numpy(sel).cuda()
    ks, vs = esa.esa_gather_kv(Kd, Vd, idx)
    O, lse = esa.esa_attend(qd, Kd, Vd, t0, l_I, l_L, ks, vs, return_lse=True)
    O_idx, lse_idx = esa.esa_attend_indexed(qd, Kd, Vd, t0, l_I, l_L, idx, return_lse=True)
    assert torch.equal(O, O_idx) and torch.equal(lse, lse_idx)
    for b in range(B):
        want, want_lse = orc.attend(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d))
        # an output is a mean of bf16 values near 1 with weights in 8 bits: half a place of either, with the largest value 4
        assert np.max(np.abs(to_f64(O[b]) - want)) <= O_TOL["bf16"], b
        assert np.max(np.abs(to_f64(lse[b]) - want_lse)) <= 1e-3, b


# Workgroups of five waves (bf16): the fewest and the most keys they take for 8, 16 and 64 pairs of sequence and KV head, one key less and
# one more, a last tile of one key; in one part and in Section 3.2's two
@pytest.mark.parametrize("B,H,H_kv,d,l_C,keys", [(1, 16, 8, 128, 1, 4096), (1, 16, 8, 128, 1, 4097), (1, 16, 8, 64, 1, 5120), (1, 16, 8, 128, 1, 5121), (1, 16, 8, 128, 5, 4300),
                                                 (2, 8, 8, 64, 1, 2049), (2, 8, 8, 128, 1, 2560), (8, 8, 8, 128, 1, 513), (8, 8, 8, 64, 3, 640), (1, 8, 1, 128, 15, 9000)])
def test_split_key_attention_in_workgroups_of_five_waves(esa, B, H, H_kv, d, l_C, keys):
    say(f"attend, five waves B={B} H={H} H_kv={H_kv} d={d} l_C={l_C} keys={keys}")
    l_I, n_sel = 64, keys // 3
    l_L = keys - l_C - l_I - n_sel
    t0 = l_I + 2 * n_sel + l_L
    q, K, V, sel = attend_inputs(d + l_C, "bf16", B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)
    qd, Kd, Vd, idx = f64_to_dev(q, "bf16"), f64_to_dev(K, "bf16"), f64_to_dev(V, "bf16"), torch.from_numpy(sel).cuda()
    O, lse = esa.esa_attend_indexed(qd, Kd, Vd, t0, l_I, l_L, idx, return_lse=True)
    ks, vs = esa.esa_gather_kv(Kd, Vd, idx)
    O_re = esa.esa_attend_reencoded(qd, Kd, Vd, t0, l_I, l_L, ks, vs, 4096.0, 5e5)
    for b in range(B):
        want, want_lse = orc.attend(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d))
        assert np.max(np.abs(to_f64(O[b]) - want)) <= O_TOL["bf16"]
        assert np.max(np.abs(to_f64(lse[b]) - want_lse)) <= 1e-3
        want, _ = orc.attend_reencoded(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d), 4096.0, 5e5)
        assert np.max(np.abs(to_f64(O_re[b]) - want)) <= O_TOL["bf16"]


# Plans of the one-call form: row tiles of 128 and of 256 rows, one slice and 32, more workgroups than one round of compute units, fewer
# keys than slices would take, group sizes; Section 3.2's two parts with the same plans
@pytest.mark.parametrize("B,H,H_kv,d,l_C,l_I,l_L,n_sel", [
    (1, 32, 8, 128, 33, 64, 500, 400), (1, 32, 8, 128, 64, 64, 3000, 1000), (1, 32, 8, 128, 65, 64, 500, 400), (1, 32, 8, 128, 160, 64, 500, 400), (1, 16, 4, 128, 352, 64, 900, 700),
    (1, 4, 4, 128, 20, 128, 9000, 7200), (1, 16, 2, 64, 17, 64, 500, 400), (2, 8, 8, 64, 130, 64, 500, 400), (33, 8, 8, 128, 16, 16, 40, 20), (3, 8, 1, 128, 700, 0, 30, 1), (40, 8, 8, 64, 257, 0, 0, 0)])
def test_matrix_core_attention_plans(esa, B, H, H_kv, d, l_C, l_I, l_L, n_sel):
    t0 = l_I + n_sel + n_sel // 2 + l_L
    say(f"attend plan B={B} H={H} H_kv={H_kv} d={d} t0={t0} l_C={l_C} l_I={l_I} l_L={l_L} n_sel={n_sel}")
    q, K, V, sel = attend_inputs(d + l_C, "bf16", B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)
    qd, Kd, Vd, idx = f64_to_dev(q, "bf16"), f64_to_dev(K, "bf16"), f64_to_dev(V, "bf16"), torch.from_numpy(sel).cuda()
    O, lse = esa.esa_attend_indexed(qd, Kd, Vd, t0, l_I, l_L, idx, return_lse=True)
    ks, vs = esa.esa_gather_kv(Kd, Vd, idx) if n_sel else (None, None)
    O_re = esa.esa_attend_reencoded(qd, Kd, Vd, t0, l_I, l_L, ks, vs, 4096.0, 5e5)
    for b in range(0, B, max(1, B // 3)):
        want, want_lse = orc.attend(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d))
        assert np.max(np.abs(to_f64(O[b]) - want)) <= O_TOL["bf16"]
        assert np.max(np.abs(to_f64(lse[b]) - want_lse)) <= 1e-3
        want, _ = orc.attend_reencoded(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d), 4096.0, 5e5)
        assert np.max(np.abs(to_f64(O_re[b]) - want)) <= O_TOL["bf16"]


# Distance (2-norm) of a chunk's outputs from the 64-bit result where a row is cut into fewer slices than one round of workgroups of 256 rows takes.
# Rounding the outputs to bf16 makes 1.66e-3 of it and rounding every probability as much again, 2.35e-3; a key at which the softmax reference has
# stood is exact.  On these inputs it was 2.3002e-3 and 2.2934e-3 with that many slices (the bounds: the same inputs always,
# so that only the kernel's roundings differ), 2.318 and 2.303 with fewer and the reference moved no oftener, and is 2.287 and 2.281 now.
@pytest.mark.parametrize("H,H_kv,l_C,l_L,n_sel,most", [(16, 2, 300, 2048, 1024, 2.301e-3), (32, 8, 128, 2048, 2048, 2.294e-3)])
def test_matrix_core_attention_in_few_slices_is_no_further_from_64_bits(esa, H, H_kv, l_C, l_L, n_sel, most):
    say(f"distance from 64 bits H={H} H_kv={H_kv} l_C={l_C} l_L={l_L} n_sel={n_sel}")
    d, l_I, squares = 128, 128, []
    t0 = l_L + n_sel + 300
    for seed in range(4):
        g = torch.Generator(device="cuda").manual_seed(seed)
        q, K, V = (torch.randn((n, h, d), generator=g, device="cuda", dtype=torch.bfloat16) for n, h in ((l_C, H), (t0 + l_C, H_kv), (t0 + l_C, H_kv)))
        idx = (l_I + torch.randperm(t0 - l_L - l_I, generator=g, device="cuda")[:n_sel].sort()[0]).to(torch.int32)
        O = esa.esa_attend_indexed(q, K, V, t0, l_I, l_L, idx).double()
        rows = torch.cat([torch.arange(l_I, device="cuda"), idx.long(), torch.arange(t0 - l_L, t0 + l_C, device="cuda")])
        keys, values = K[rows].double(), V[rows].double()
        hidden = torch.arange(rows.numel(), device="cuda")[None] > rows.numel() - l_C + torch.arange(l_C, device="cuda")[:, None]
        off = size = 0.0
        for h in range(H):
            logits = (q[:, h].double() @ keys[:, h * H_kv // H].T.contiguous() / d ** 0.5).masked_fill(hidden, float("-inf"))
            want = torch.softmax(logits, 1) @ values[:, h * H_kv // H].contiguous()
            off, size = off + (O[:, h] - want).square().sum().item(), size + want.square().sum().item()
        squares.append(off / size)
    distance = (sum(squares) / len(squares)) ** 0.5
    print(f"distance {distance:.4e}", flush=True)
    assert distance <= most


# Few tokens: an encoded copy of the local keys below 8192 of them in all (batch entries x KV heads x keys), turned as they are read from there
# on.  No local key but the tokens' own, a tile of keys, one less and one more, windows whose slices end inside; 32 rows to a KV head (the
# most), one more (an encoded copy); head sizes, group sizes, a padded cache
@pytest.mark.parametrize("B,H,H_kv,d,t0,l_C,l_I,l_L,n_sel,pad", [
    (1, 8, 2, 128, 300, 1, 16, 0, 40, 0), (1, 8, 2, 128, 300, 1, 16, 31, 40, 0), (2, 8, 8, 128, 300, 2, 16, 31, 0, 64), (1, 32, 8, 128, 3000, 1, 128, 2048, 500, 0),
    (2, 32, 8, 128, 900, 8, 16, 333, 64, 8), (2, 32, 8, 128, 900, 9, 16, 333, 64, 0), (3, 16, 2, 128, 900, 4, 0, 400, 65, 0), (1, 6, 2, 128, 500, 10, 16, 100, 33, 0),
    (1, 8, 2, 64, 300, 1, 16, 32, 40, 0), (2, 16, 2, 64, 2500, 4, 16, 2000, 100, 8), (4, 8, 8, 64, 700, 15, 16, 200, 31, 0), (1, 8, 4, 64, 0, 7, 16, 32, 0, 0),
    (32, 8, 8, 128, 80, 1, 16, 30, 20, 0), (32, 8, 8, 128, 80, 1, 16, 31, 20, 0), (32, 8, 8, 128, 80, 1, 16, 32, 0, 0), (33, 32, 8, 128, 90, 4, 16, 30, 20, 8),
    (16, 32, 8, 128, 300, 8, 16, 64, 100, 0), (1, 8, 8, 128, 1200, 1, 0, 1100, 0, 0), (256, 3, 1, 64, 60, 10, 4, 22, 9, 8), (32, 16, 2, 64, 300, 4, 16, 130, 31, 0),
    (32, 8, 8, 64, 90, 15, 0, 17, 31, 0), (4, 32, 8, 64, 700, 8, 16, 300, 64, 0)])
def test_reencoded_attention_of_few_tokens_turns_the_local_keys(esa, B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel, pad):
    say(f"re-encoded, few tokens B={B} H={H} H_kv={H_kv} d={d} t0={t0} l_C={l_C} l_I={l_I} l_L={l_L} n_sel={n_sel} pad={pad}")
    q, K, V, sel = attend_inputs(d + l_C, "bf16", B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)

    def rows(x):                    # token rows `pad` elements apart
        x = f64_to_dev(x, "bf16")
        buf = torch.zeros((B, t0 + l_C, H_kv * d + pad), dtype=x.dtype, device="cuda")
        view = buf.as_strided((B, t0 + l_C, H_kv, d), ((t0 + l_C) * (H_kv * d + pad), H_kv * d + pad, d, 1))
        view.copy_(x)
        return view

    qd, Kd, Vd, idx = f64_to_dev(q, "bf16"), rows(K), rows(V), torch.from_numpy(sel).cuda()
    ks, vs = esa.esa_gather_kv(Kd, Vd, idx) if n_sel else (None, None)
    O, lse = esa.esa_attend_reencoded(qd, Kd, Vd, t0, l_I, l_L, ks, vs, 4096.0, 5e5, return_lse=True)
    for b in range(0, B, max(1, B // 4)):
        want, want_lse = attend_reencoded_rounded(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 4096.0, 5e5)
        # fp32 arithmetic on the rows that the oracle has too, and one rounding (a tile of 2048 keys turned by its neighbour's angle: O 2.0e-3, lse 7.5e-4)
        assert np.all(np.abs(to_f64(O[b]) - want) <= 0.502 * bf16_ulp(want) + 5e-5), b
        assert np.max(np.abs(to_f64(lse[b]) - want_lse)) <= 5e-5, b


# Section 3.2's rows are encoded in 64 bits and rounded once.  Every row of queries is made from one local key, each tile of the window
# having its turn, and that key takes the whole softmax: lse is its logit, so a single element of it or of the query that is rounded to the
# other bf16 number shows (7e-4 in the median; products and sums of fp32 err by 1e-5), and a tile encoded with another one's positions gives
# another key's value.
@pytest.mark.parametrize("B,H,H_kv,d,l_C,l_L", [(8, 32, 8, 128, 8, 2048), (1, 8, 8, 128, 1, 2048), (4, 16, 8, 64, 15, 2000), (2, 16, 2, 128, 3, 4096),
                                                (1, 32, 8, 128, 4, 4096), (1, 8, 8, 64, 2, 4096),     # (workgroups of five waves)
                                                (1, 32, 8, 128, 64, 2048), (1, 16, 8, 64, 100, 1000), (2, 8, 8, 128, 130, 1500)])
def test_reencoded_rows_are_the_exact_ones_rounded_once(esa, B, H, H_kv, d, l_C, l_L):
    say(f"re-encoded rows rounded once B={B} H={H} H_kv={H_kv} d={d} l_C={l_C} l_L={l_L}")
    base, w, l_I, n_sel = 5e5, 4096.0, 64, 256
    t0, gain = l_I + 300 + l_L, 24.0 / np.sqrt(d)
    rng = np.random.default_rng(d + l_C)
    bf16 = lambda x: orc.round_to_storage(x, "bf16")
    K, V = (bf16(rng.standard_normal((B, t0 + l_C, H_kv, d))) for _ in range(2))
    sel = (l_I + np.sort(rng.permutation(300)[:n_sel])).astype(np.int32)
    n_tiles, group = -(-l_L // 32), H // H_kv
    q = np.zeros((B, l_C, H, d))
    for b in range(B):
        for c in range(l_C):
            for h in range(H):
                tile = (2 * (c * group + h % group) + b * H_kv + h // group) % n_tiles
                j = min(32 * tile + int(rng.integers(32)), l_L - 1)
                q[b, c, h] = gain * orc.rope(K[b, t0 - l_L + j, h // group][None, None], [j - (l_L + c)], base)[0, 0]
    q = bf16(q)
    qd, Kd, Vd, idx = f64_to_dev(q, "bf16"), f64_to_dev(K, "bf16"), f64_to_dev(V, "bf16"), torch.from_numpy(np.tile(sel, (B, 1))).cuda()
    ks, vs = esa.esa_gather_kv(Kd, Vd, idx)
    O, lse = esa.esa_attend_reencoded(qd, Kd, Vd, t0, l_I, l_L, ks, vs, w, base, return_lse=True)
    for b in range(B):
        want, want_lse = attend_reencoded_rounded(q[b], K[b], V[b], t0, l_I, l_L, sel, w, base)
        assert np.max(np.abs(to_f64(lse[b]) - want_lse)) <= 5e-5, b
        # half a unit in the last place from the rounding of the output, half from that of a probability
        assert np.all(np.abs(to_f64(O[b]) - want) <= bf16_ulp(want) + 1e-4), b


# Gathered rows: segment boundaries at a tile's edge, one key beside it, two of them inside one tile, no boundary but the sequence's
# end; slices that end between.  The index-driven form takes the same keys in the same order.
@pytest.mark.parametrize("B,H,H_kv,d,t0,l_C,l_I,l_L,n_sel", [
    (1, 8, 8, 128, 900, 16, 64, 64, 64), (2, 8, 2, 128, 901, 33, 63, 65, 129), (1, 8, 2, 64, 800, 70, 1, 63, 62), (1, 16, 2, 64, 1500, 257, 0, 700, 640),
    (3, 8, 8, 128, 700, 40, 20, 30, 10), (1, 32, 8, 128, 3000, 512, 128, 1000, 1), (1, 32, 8, 128, 600, 48, 0, 0, 500)])
def test_attention_over_gathered_rows_is_the_index_driven_one(esa, B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel):
    say(f"attend gathered B={B} H={H} H_kv={H_kv} d={d} t0={t0} l_C={l_C} l_I={l_I} l_L={l_L} n_sel={n_sel}")
    q, K, V, sel = attend_inputs(d + l_C, "bf16", B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)
    qd, Kd, Vd, idx = f64_to_dev(q, "bf16"), f64_to_dev(K, "bf16"), f64_to_dev(V, "bf16"), torch.from_numpy(sel).cuda()
    ks, vs = esa.esa_gather_kv(Kd, Vd, idx)
    O, lse = esa.esa_attend(qd, Kd, Vd, t0, l_I, l_L, ks, vs, return_lse=True)
    O_idx, lse_idx = esa.esa_attend_indexed(qd, Kd, Vd, t0, l_I, l_L, idx, return_lse=True)
    assert torch.equal(O, O_idx) and torch.equal(lse, lse_idx)
    for b in range(B):
        want, _ = orc.attend(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d))
        assert np.max(np.abs(to_f64(O[b]) - want)) <= O_TOL["bf16"], b


# 1.000 measured; 1.034 to 1.036 where one kernel served both forms and chose base and stride for each row
def test_attention_over_gathered_rows_is_no_slower_than_the_index_driven_one(esa):
    say("attend, 1024 queries, 8192 gathered rows")
    l_C, t0, n_sel = 1024, 24000, 8192
    g = torch.Generator(device="cuda").manual_seed(3)
    q, K, V = (torch.randn((n, h, 128), generator=g, device="cuda").to(torch.bfloat16) for n, h in ((l_C, 32), (t0 + l_C, 8), (t0 + l_C, 8)))
    idx = 128 + torch.randperm(t0 - 8192 - 128, generator=g, device="cuda")[:n_sel].sort()[0].to(torch.int32)
    ks, vs = esa.esa_gather_kv(K, V, idx)
    ratios = sorted(_time_us(lambda: esa.esa_attend(q, K, V, t0, 128, 8192, ks, vs), 40) /
                    _time_us(lambda: esa.esa_attend_indexed(q, K, V, t0, 128, 8192, idx), 40) for _ in range(15))
    print("gathered / indexed: " + " ".join(f"{r:.3f}" for r in ratios), flush=True)
    assert ratios[7] <= 1.02


# more pairs of batch entry and KV head than a grid takes in z (65535): few tokens and a chunk
@pytest.mark.parametrize("l_C", [1, 16])
def test_attention_over_more_pairs_than_one_grid(esa, l_C):
    say(f"attend 8193 x 9 pairs l_C={l_C}")
    B, H, d, t0 = 8193, 9, 64, 5
    g = torch.Generator(device="cuda").manual_seed(l_C)
    q, K, V = (torch.randn((B, n, H, d), generator=g, device="cuda", dtype=torch.bfloat16) for n in (l_C, t0 + l_C, t0 + l_C))
    O = esa.esa_attend(q, K, V, t0, 2, 3, None, None)
    for b in (0, 1, 4096, 7281, 7282, 8192):        # pair 65535 is entry 7281's
        want, _ = orc.attend(to_f64(q[b]), to_f64(K[b]), to_f64(V[b]), t0, 2, 3, np.empty(0, np.int32), 1.0 / np.sqrt(d))
        assert np.max(np.abs(to_f64(O[b]) - want)) <= O_TOL["bf16"], b


# a workgroup's 64 rows, one less, one more, a single row; the most rows in all of that kernel and one more
@pytest.mark.parametrize("B,n,d_c", [(1, 1, 128), (3, 63, 64), (2, 64, 256), (5, 65, 128), (1, 131072, 64), (1, 131073, 64)])
def test_score_of_one_token_in_workgroups_of_64_rows_and_of_256(esa, B, n, d_c):
    say(f"score l_c=1 B={B} n={n} d_c={d_c}")
    rng = np.random.default_rng(n + d_c)
    qc = orc.round_to_storage(rng.standard_normal((B, 1, d_c)), "bf16")
    kc = orc.round_to_storage(rng.standard_normal((B, n + 3, d_c)), "bf16")
    got = to_f64(esa.esa_score(f64_to_dev(qc, "bf16"), f64_to_dev(kc, "bf16"), 2, 2 + n))
    for b in range(B):
        assert np.max(np.abs(got[b] - orc.importance(qc[b], kc[b, 2:2 + n]))) <= F_TOL["bf16"], b
        assert got[b].max() == 0.0


@pytest.mark.parametrize("B,l_c,n,d_c,k,eps", [(2, 1, 8192, 128, 2048, 0), (3, 1, 8192, 128, 100, 3), (1, 1, 8193, 128, 2048, 3),
                                               (1, 33, 8192, 64, 1, 16), (2, 40, 2050, 128, 2048, 17), (2, 1, 1025, 128, 1024, 1)])
def test_scores_finished_by_the_selection_equal_the_separate_calls(esa, B, l_c, n, d_c, k, eps):
    say(f"fused score+select B={B} l_c={l_c} n={n} d_c={d_c} k={k} eps={eps}")
    g = torch.Generator(device="cuda").manual_seed(n + l_c)
    qc = torch.randn((B, l_c, d_c), generator=g, device="cuda").to(torch.bfloat16)
    kc = torch.randn((B, n + 20, d_c), generator=g, device="cuda").to(torch.bfloat16)
    score, idx, _, _ = esa.esa_score_select_gather(qc, kc, 7, n + 7, k, eps=eps)
    want = esa.esa_score(qc, kc, 7, n + 7, eps=eps)
    assert torch.equal(score, want)
    assert torch.equal(idx, esa.esa_select_topk(want, k, base=7))


# one key, fewer keys than waves, rows that fill a 32-row tile or run one over, group sizes that divide nothing, a single
# slice and many, every head size and storage type of the kernel
@pytest.mark.parametrize("dtype,B,H,H_kv,d,t0,l_C,l_I,l_L,n_sel", [
    ("bf16", 1, 8, 2, 64, 0, 1, 16, 64, 0), ("bf16", 2, 8, 2, 128, 700, 8, 16, 64, 33), ("bf16", 1, 8, 1, 128, 900, 5, 7, 129, 300),
    ("bf16", 40, 16, 8, 64, 300, 15, 3, 70, 90), ("bf16", 3, 6, 2, 128, 500, 11, 0, 31, 1), ("bf16", 1, 32, 8, 128, 9000, 2, 128, 2048, 2048),
    ("f32", 1, 4, 2, 32, 700, 130, 16, 64, 100), ("f32", 2, 6, 2, 64, 400, 11, 0, 31, 1), ("f32", 1, 8, 1, 128, 600, 33, 7, 129, 300),
    ("f32", 1, 4, 2, 128, 0, 3, 7, 129, 0), ("f32", 1, 4, 2, 64, 5000, 1, 32, 2500, 1000),
    ("f32", 1, 4, 2, 64, 60, 4, 7, 129, 0), ("f32", 1, 4, 2, 64, 60, 5, 7, 129, 0), ("f32", 2, 32, 8, 32, 100, 8, 3, 20, 30),
    ("f32", 2, 32, 8, 32, 100, 9, 3, 20, 30)])
def test_split_key_attention(esa, dtype, B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel):
    say(f"split attend {dtype} B={B} H={H} H_kv={H_kv} d={d} t0={t0} l_C={l_C} l_I={l_I} l_L={l_L} n_sel={n_sel}")
    q, K, V, sel = attend_inputs(d + l_C, dtype, B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)
    qd, Kd, Vd, idx = f64_to_dev(q, dtype), f64_to_dev(K, dtype), f64_to_dev(V, dtype), torch.from_numpy(sel).cuda()
    O, lse = esa.esa_attend_indexed(qd, Kd, Vd, t0, l_I, l_L, idx, return_lse=True)
    ks, vs = esa.esa_gather_kv(Kd, Vd, idx) if n_sel else (None, None)
    O_re = esa.esa_attend_reencoded(qd, Kd, Vd, t0, l_I, l_L, ks, vs, 4096.0, 5e5)
    for b in range(B):
        want, want_lse = orc.attend(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d))
        assert np.max(np.abs(to_f64(O[b]) - want)) <= O_TOL[dtype]
        assert np.max(np.abs(to_f64(lse[b]) - want_lse)) <= (1e-5 if dtype == "f32" else 1e-3)
        want, _ = orc.attend_reencoded(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d), 4096.0, 5e5)
        assert np.max(np.abs(to_f64(O_re[b]) - want)) <= O_TOL[dtype]


@pytest.mark.parametrize("dtype,d,l_C", [("bf16", 128, 1), ("bf16", 64, 5), ("f32", 64, 1), ("f32", 128, 40), ("bf16", 64, 40), ("bf16", 128, 40)])
def test_a_key_that_is_no_number_is_not_left_out(esa, dtype, d, l_C):
    """A NaN in one selected key reaches every output of its KV head's queries, and no other."""
    say(f"NaN key {dtype} d={d} l_C={l_C}")
    H, H_kv, t0, l_I, l_L, n_sel = 8, 2, 3000, 16, 130, 900
    q, K, V, sel = attend_inputs(d + l_C, dtype, 1, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)
    K[0, sel[0, 17], 0, 3] = np.nan
    Kd = torch.from_numpy(K[0]).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16)
    O, lse = esa.esa_attend_indexed(f64_to_dev(q[0], dtype), Kd, f64_to_dev(V[0], dtype), t0, l_I, l_L, torch.from_numpy(sel[0]).cuda(),
                                    return_lse=True)
    assert torch.isnan(O[:, :H // H_kv]).all() and torch.isnan(lse[:, :H // H_kv]).all()
    assert torch.isfinite(O[:, H // H_kv:]).all() and torch.isfinite(lse[:, H // H_kv:]).all()


# S stored: a few queries on the matrix cores (one token, tile and workgroup remainders), every other shape in fp32 FMAs;
# pooled by the finishing pass (windows up to 16) or by the pass of its own
@pytest.mark.parametrize("dtype,B,l_c,n,d_c,eps", [
    ("bf16", 2, 2, 1, 128, 0), ("bf16", 1, 16, 1025, 128, 16), ("bf16", 3, 5, 9999, 64, 1), ("bf16", 17, 3, 60000, 128, 0),
    ("bf16", 1, 7, 30001, 128, 17), ("bf16", 1, 6, 2500, 256, 2), ("f32", 2, 17, 64, 32, 16), ("f32", 1, 130, 1633, 32, 3),
    ("f32", 1, 1, 20001, 48, 0), ("f32", 2, 16, 4097, 16, 1), ("bf16", 1, 40, 12000, 32, 5), ("bf16", 2, 1, 30000, 128, 5)])
def test_score_with_s_stored(esa, dtype, B, l_c, n, d_c, eps):
    say(f"score {dtype} B={B} l_c={l_c} n={n} d_c={d_c} eps={eps}")
    rng = np.random.default_rng(n + l_c)
    qc = orc.round_to_storage(rng.standard_normal((B, l_c, d_c)) * 1.5, dtype)
    kc = orc.round_to_storage(rng.standard_normal((B, n + 8, d_c)), dtype)
    qd, kd, k = f64_to_dev(qc, dtype), f64_to_dev(kc, dtype), min(n, 700)
    got = esa.esa_score(qd, kd, 3, n + 3, eps=eps)
    for b in range(B):
        want = orc.importance(qc[b], kc[b, 3:n + 3])
        want = orc.proximity(want, eps) if eps else want
        assert np.max(np.abs(to_f64(got[b]) - want)) <= F_TOL[dtype]
        assert float(got[b].max()) == 0.0
    score, idx, _, _ = esa.esa_score_select_gather(qd, kd, 3, n + 3, k, eps=eps)
    assert score is None or torch.equal(score, got)
    assert torch.equal(idx, esa.esa_select_topk(got, k, base=3))


@pytest.mark.parametrize("dtype,B,n_tok,d_in,d_c,packed", [("f32", 2, 1, 1, 16, True), ("f32", 1, 17, 257, 48, False),
                                                           ("f32", 3, 15, 1030, 256, True), ("bf16", 2, 33, 130, 16, True)])
def test_compress_with_plain_fmas(esa, dtype, B, n_tok, d_in, d_c, packed):
    """Any shape, both inputs in one launch; d_in products of rounded unit-scale numbers added in fp32."""
    say(f"compress {dtype} B={B} n_tok={n_tok} d_in={d_in} d_c={d_c} packed={packed}")
    rng = np.random.default_rng(n_tok + d_in)
    x = orc.round_to_storage(rng.standard_normal((B, n_tok, d_in)), dtype)
    W = orc.round_to_storage(rng.standard_normal((d_in, d_c)) / np.sqrt(d_in), dtype)
    xd, Wd = f64_to_dev(x, dtype), f64_to_dev(W, dtype)
    Wd = esa.esa_pack_weights(Wd) if packed else Wd
    q, k = esa.esa_compress_qk(xd, Wd, xd[:, :, :].clone(), Wd)
    ulp = 2.0 ** -7 if dtype == "bf16" else 0.0
    for b in range(B):
        want = x[b] @ W
        for got in (to_f64(q[b]), to_f64(k[b])):
            assert np.all(np.abs(got - want) <= 1e-5 + ulp * np.abs(want))


# one piece of the reduction for one wave, pieces that do not share out evenly, row tiles of 16 and of 32 with and without
# remainders, rows numbered through the batch, both inputs in a workgroup and one in each
@pytest.mark.parametrize("B,n_tok,d_q,d_k,d_c", [(1, 5, 64, 64, 16), (1, 16, 192, 64, 48), (3, 11, 1088, 576, 128), (16, 1, 4096, 1024, 128),
                                                 (1, 257, 1024, 256, 128), (1, 513, 576, 192, 128), (2, 300, 4096, 1024, 64), (1, 4097, 128, 64, 16)])
def test_compress_packed_row_tiles(esa, B, n_tok, d_q, d_k, d_c):
    say(f"compress_qk B={B} n_tok={n_tok} d_q={d_q} d_k={d_k} d_c={d_c}")
    rng = np.random.default_rng(d_q + n_tok)
    xs = [orc.round_to_storage(rng.standard_normal((B, n_tok, d)), "bf16") for d in (d_q, d_k)]
    Ws = [orc.round_to_storage(rng.standard_normal((d, d_c)) / np.sqrt(d), "bf16") for d in (d_q, d_k)]
    bias = orc.round_to_storage(rng.standard_normal(d_c) * 0.1, "bf16")
    xd, Wd = [f64_to_dev(x, "bf16") for x in xs], [esa.esa_pack_weights(f64_to_dev(W, "bf16")) for W in Ws]
    cache = torch.full((B, n_tok + 6, d_c), 3.0, dtype=torch.bfloat16, device="cuda")
    got_q, _ = esa.esa_compress_qk(xd[0], Wd[0], xd[1], Wd[1], bias_q=f64_to_dev(bias, "bf16"), out_k=cache[:, 2:2 + n_tok])
    assert torch.all(cache[:, :2] == 3.0) and torch.all(cache[:, 2 + n_tok:] == 3.0)
    assert torch.equal(cache[:, 2:2 + n_tok], esa.esa_compress(xd[1], Wd[1]))        # the same arithmetic, bit for bit
    for got, x, W, b in ((got_q, xs[0], Ws[0], bias), (cache[:, 2:2 + n_tok], xs[1], Ws[1], None)):
        for e in range(B):
            want = orc.compress(x[e], W, b, "bf16")
            assert np.all(np.abs(to_f64(got[e]) - want) <= bf16_ulp(want) * 1.001)


# a row or two of many heads, sixteen rows and one more, a step that is not one, positions on both sides of zero; one, eight and
# sixteen rows to a workgroup
@pytest.mark.parametrize("dtype,B,n_tok,heads,d,pos0,step", [("bf16", 1, 1, 32, 128, 70000.0, 1.0), ("bf16", 40, 33, 8, 64, -16.0, 1.0),
                                                              ("f32", 1, 17, 5, 256, 3.0, 2.5), ("bf16", 1, 19, 200, 128, 9.0, 1.0),
                                                              ("f32", 2, 16, 1, 2, 100.0, 1.0), ("bf16", 1, 97, 32, 64, 5.0, 1.0),
                                                              ("f32", 1, 4500, 8, 32, 0.0, 1.0), ("bf16", 2, 5001, 8, 32, 7.0, 1.0)])
def test_rope_rows(esa, dtype, B, n_tok, heads, d, pos0, step):
    say(f"rope {dtype} B={B} n_tok={n_tok} heads={heads} d={d} pos0={pos0} step={step}")
    rng = np.random.default_rng(n_tok + heads)
    x = orc.round_to_storage(rng.standard_normal((B, n_tok, heads, d)), dtype)
    want = np.stack([orc.round_to_storage(orc.rope(x[b], pos0 + step * np.arange(n_tok), 5e5), dtype) for b in range(B)])
    got = to_f64(esa.esa_rope(f64_to_dev(x, dtype), pos0, step, 5e5))
    # one rounding on each side of fp64 values that differ in their last bits
    assert np.all(np.abs(got - want) <= np.abs(want) * (2.0 ** -7 if dtype == "bf16" else 2.0 ** -23))
    assert np.count_nonzero(got != want) <= max(2, 1e-5 * want.size)


def test_calls_on_two_streams_and_threads_do_not_share_scratch(esa):
    """Each thread runs steps of its own on a stream of its own; their results are those of the same steps run alone."""
    say("two threads, two streams, different steps")
    import threading
    l_I, l_L, k, passes = 128, 1024, 512, 12

    def step(t0, l_C, seed):
        g = torch.Generator(device="cuda").manual_seed(seed)
        mk = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)
        q, K, V, qc, kc = mk(l_C, 8, 128), mk(t0 + l_C, 2, 128), mk(t0 + l_C, 2, 128), mk(l_C, 128), mk(t0 + l_C, 128)

        def run():
            score, idx, ks, vs = esa.esa_score_select_gather(qc, kc, l_I, t0 - l_L, k, K, V)
            return (score, idx, esa.esa_select_topk(score, 64), esa.esa_attend_indexed(q, K, V, t0, l_I, l_L, idx),
                    esa.esa_attend_reencoded(q, K, V, t0, l_I, l_L, ks, vs, 4096.0, 5e5))
        return run

    steps = [step(60000, 1, 1), step(45000, 40, 2)]
    want = [run() for run in steps]
    torch.cuda.synchronize()
    got = [[], []]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(passes):
                got[i].append(steps[i]())
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert len(got[i]) == passes
        for results in got[i]:
            for a, b in zip(results, want[i]):
                assert torch.equal(a, b)


# K' as a stream: one token with the shortest row and one token less, the fewest bytes in all and one token less, a workgroup's 512 rows and one more
# in the last one, short rows that are mostly padding; a few queries with the fewest bytes and one row less, batches, every row length
@pytest.mark.parametrize("B,l_c,n,d_c", [(1, 1, 196608, 128), (1, 1, 196609, 128), (3, 1, 65537, 256), (2, 1, 131072, 64), (24, 1, 8705, 128), (1, 2, 262143, 128),
                                         (1, 2, 262144, 128), (3, 16, 200001, 64), (16, 1, 18432, 128), (16, 1, 18431, 128), (4, 1, 147456, 64),
                                         (4, 1, 147455, 64), (2, 1, 98304, 256), (162, 1, 1821, 128), (163, 1, 1820, 128), (600, 1, 577, 128)])
def test_score_of_streamed_compressed_keys(esa, B, l_c, n, d_c):
    say(f"score, K' streamed B={B} l_c={l_c} n={n} d_c={d_c}")
    rng = np.random.default_rng(n + d_c)
    qc = orc.round_to_storage(rng.standard_normal((B, l_c, d_c)), "bf16")
    kd = torch.randn((B, n + 3, d_c), generator=torch.Generator(device="cuda").manual_seed(n), device="cuda").bfloat16()
    got = esa.esa_score(f64_to_dev(qc, "bf16"), kd, 2, 2 + n)
    for b in range(0, B, max(1, B // 24)):
        s = torch.from_numpy(qc[b]).cuda() @ kd[b, 2:2 + n].double().T
        want = (s - s.max(1, keepdim=True).values).max(0).values
        assert float((got[b].double() - want).abs().max()) <= F_TOL["bf16"], b
        assert float(got[b].max()) == 0.0


def test_sequences_that_share_a_cache_read_it_from_cache(esa):
    """One K' for eight sequences (batch stride 0): the results of eight copies of it, bit for bit, in well under their time (0.46 of it; fetched
    past the caches 0.96).  Keys and values of 16 sequences and five tokens the same."""
    say("score and attention over one shared cache")
    g = torch.Generator(device="cuda").manual_seed(5)
    draw = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    one, q = draw(130000, 128), draw(8, 1, 128)
    same, own = one.expand(8, -1, -1), one.repeat(8, 1, 1)
    took = {}
    for name, k in (("same", same), ("own", own)):
        for _ in range(4):                             # the first one warms up
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                score = esa.esa_score(q, k, 0, 130000)
            b.record()
            b.synchronize()
            took[name] = min(took.get(name, (1e9,))[0], a.elapsed_time(b)), score
    assert torch.equal(took["same"][1], took["own"][1])
    assert took["same"][0] < 0.75 * took["own"][0], {name: t[0] for name, t in took.items()}
    for l_c in (1, 5):
        q, k, v = draw(16, l_c, 32, 128), draw(20000 + l_c, 8, 128), draw(20000 + l_c, 8, 128)
        idx = torch.stack([(128 + torch.randperm(17000, generator=g, device="cuda")[:2048].sort()[0]).to(torch.int32) for _ in range(16)])
        want = esa.esa_attend_indexed(q, k.repeat(16, 1, 1, 1), v.repeat(16, 1, 1, 1), 20000, 128, 2048, idx)
        assert torch.equal(esa.esa_attend_indexed(q, k.expand(16, -1, -1, -1), v.expand(16, -1, -1, -1), 20000, 128, 2048, idx), want)


# Keys and values as a stream (64 MB together and more, one row tile): the fewest keys and one less, rows that fill the tile, both head sizes
@pytest.mark.parametrize("B,H,H_kv,d,l_C,keys", [(4, 32, 8, 128, 1, 4096), (4, 32, 8, 128, 1, 4095), (8, 32, 8, 64, 8, 4097), (2, 16, 16, 128, 5, 4100)])
def test_split_key_attention_over_streamed_rows(esa, B, H, H_kv, d, l_C, keys):
    say(f"attend, streamed B={B} H={H} H_kv={H_kv} d={d} l_C={l_C} keys={keys}")
    l_I, n_sel = 64, keys // 3
    l_L = keys - l_C - l_I - n_sel
    t0 = l_I + n_sel + 200 + l_L
    q, K, V, sel = attend_inputs(d + l_C, "bf16", B, H, H_kv, d, t0, l_C, l_I, l_L, n_sel)
    O, lse = esa.esa_attend_indexed(*(f64_to_dev(x, "bf16") for x in (q, K, V)), t0, l_I, l_L, torch.from_numpy(sel).cuda(), return_lse=True)
    for b in range(B):
        want, want_lse = orc.attend(q[b], K[b], V[b], t0, l_I, l_L, sel[b], 1.0 / np.sqrt(d))
        assert np.max(np.abs(to_f64(O[b]) - want)) <= O_TOL["bf16"]
        assert np.max(np.abs(to_f64(lse[b]) - want_lse)) <= 1e-3


# fp32 scores on the matrix cores: one token and one more than a block, tiles of queries and one more, every number of steps in flight; rows that
# are not 16-byte aligned take plain FMAs
@pytest.mark.parametrize("B,l_c,n,d_c,eps,shift", [(1, 2, 1, 16, 0, 0), (2, 65, 63, 48, 1, 0), (3, 33, 65, 32, 0, 0), (1, 64, 4097, 256, 17, 0), (2, 100, 3000, 112, 2, 0),
                                                   (1, 33, 500, 32, 0, 1), (2, 5, 700, 64, 1, 2)])
def test_fp32_scores_of_several_queries(esa, B, l_c, n, d_c, eps, shift):
    say(f"score fp32 B={B} l_c={l_c} n={n} d_c={d_c} eps={eps} shift={shift}")
    rng = np.random.default_rng(n + l_c)
    qc, kc = (orc.round_to_storage(rng.standard_normal((B, m, d_c)), "f32") for m in (l_c, n + 5))
    kd = torch.zeros(B * (n + 5) * d_c + shift, device="cuda")[shift:].view(B, n + 5, d_c)
    kd.copy_(f64_to_dev(kc, "f32"))
    got = to_f64(esa.esa_score(f64_to_dev(qc, "f32"), kd, 3, n + 3, eps=eps))
    for b in range(B):
        want = orc.importance(qc[b], kc[b, 3:n + 3])
        want = orc.proximity(want, eps) if eps else want
        assert np.max(np.abs(got[b] - want)) <= F_TOL["f32"]
        assert got[b].max() == 0.0


# fp32: a token's score has the same bits whatever the call's other sizes and alignment.  One query, several on the matrix cores, several whose
# rows are not 16-byte aligned, and more scores than are stored
@pytest.mark.parametrize("n,d_c", [(15000, 16), (14337, 32), (14500, 48), (15000, 128), (14400, 256)])
def test_fp32_scores_do_not_depend_on_the_call(esa, n, d_c):
    say(f"score fp32 n={n} d_c={d_c}")
    g = torch.Generator(device="cuda").manual_seed(n + d_c)
    q, kc = torch.randn((1, d_c), generator=g, device="cuda"), torch.randn((n, d_c), generator=g, device="cuda")

    def shifted(t):                        # the same rows, 4 bytes further
        room = torch.empty(t.numel() + 1, device="cuda")
        room[1:] = t.reshape(-1)
        return room[1:].view(t.shape)

    one = esa.esa_score(q, kc, 0, n)
    for name, other in (("three", (q.repeat(3, 1), kc)), ("three, shifted", (shifted(q.repeat(3, 1)), kc)), ("one, shifted", (q, shifted(kc))),
                        ("three hundred", (q.repeat(300, 1), kc)), ("three hundred, shifted", (q.repeat(300, 1), shifted(kc)))):
        assert torch.equal(one, esa.esa_score(*other, 0, n)), name

