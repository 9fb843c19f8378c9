"""GPU parity: copris_lmhead_logprob through the C ABI vs the fp64 oracle."""
import math

import numpy as np
import pytest

from oracle import copris_oracle as O
from paper_2511_05589_amd import workloads as W
from tests import parity as P
from tests.test_launch_rules import NARROW, RUNS, SMALL, WIDE

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    from paper_2511_05589_amd import runner
    runner.require_gpu()
    return runner


def test_tiny_config_fp32(R):
    cfg = W.DECODE_CONFIGS[0]
    inp = W.make_decode_inputs(cfg, with_attn=False)
    tok, lp, lse = R.run_lmhead_logprob(inp, cfg.dtype)
    P.check_lmhead(tok, lp, lse, P.oracle_lmhead(inp, cfg.dtype), "cfg0")


@pytest.mark.parametrize("dtype", [W.F32, W.BF16])
@pytest.mark.parametrize("C,H,V", [(1, 64, 50), (3, 256, 1000), (17, 512, 4099), (64, 1536, 9000),
                                   (256, 128, 2500), (33, 3584, 777),
                                   (300, 512, 3001),      # two batch blocks, ragged vocabulary tail
                                   (129, 192, 70000),     # more tiles than persistent workgroups
                                   (5, 72, 260)])         # hidden size the matrix-core kernel does not take
def test_small_shapes(R, dtype, C, H, V):
    inp = W.make_small_lmhead_case(C * 7 + V, C, H, V, dtype, w_std=0.05)
    tok, lp, lse = R.run_lmhead_logprob(inp, dtype)
    n_exempt = P.check_lmhead(tok, lp, lse, P.oracle_lmhead(inp, dtype), f"{dtype} {C}x{H}x{V}")
    assert n_exempt <= 2          # expected near-ties: about C / 1000


@pytest.mark.parametrize("C,H,V", [(1, 64, 49152), (32, 128, 49153), (33, 64, 50257), (64, 192, 65537), (63, 64, 66001),   # too short a hidden state
                                   (32, 1024, 3), (31, 1024, 65), (5, 1088, 4099),    # fewer rows than a wave, one workgroup and a row
                                   (65, 64, 49153), (20, 64, 49151),                  # just outside the rule
                                   # the skinny kernel: three slabs per tile and more, tiles of equal and unequal fill, a
                                   # vocabulary that ends inside a Philox block
                                   (32, 192, 78125), (1, 320, 49152), (31, 320, 49153), (32, 1024, 32769), (33, 384, 65537),
                                   (64, 256, 97657), (63, 384, 66001), (64, 832, 49155),
                                   (8, 1024, 3), (17, 1792, 3), (31, 1856, 65), (5, 1792, 4099)])
def test_few_rows_over_the_whole_vocabulary(R, C, H, V):
    inp = W.make_small_lmhead_case(C * 11 + V, C, H, V, W.BF16, w_std=0.1)
    tok, lp, lse = R.run_lmhead_logprob(inp, W.BF16)
    P.check_lmhead(tok, lp, lse, P.oracle_lmhead(inp, W.BF16), f"{C}x{H}x{V}")
    # the same rows scored as given tokens, the ends of tiles and runs among them
    given = np.where(np.arange(C) % 2 == 0, tok, np.minimum(np.arange(C) * 37 % V, V - 1)).astype(np.int32)
    given[-1] = V - 1
    lp2, lse2 = R.run_token_logprob(inp["hidden"], inp["weight"], given, 1.0, W.BF16)
    P.check_token_logprob(lp2, lse2, P.oracle_token_logprob(inp["hidden"], inp["weight"], given, 1.0, W.BF16), f"given {C}x{H}x{V}")


@pytest.mark.parametrize("C", [65, 128, 129, 160, 192, 193, 257, 301, 320, 383, 384, 385, 520])
def test_row_blocks_of_every_width(R, C):
    # row blocks of 128, 192 and 256, one, two and three of them, the rows shared evenly or the last block
    # with the rest; more tiles than workgroups per block in the larger ones (57 of 256 places have one
    # more: with two blocks the second deals them from the end)
    H, V = 64, 40000 if C > 256 else 9001
    inp = W.make_small_lmhead_case(C * 13, C, H, V, W.BF16, w_std=0.1)
    tok, lp, lse = R.run_lmhead_logprob(inp, W.BF16)
    P.check_lmhead(tok, lp, lse, P.oracle_lmhead(inp, W.BF16), f"{C}x{H}x{V}")
    if C < 384:
        lp2, lse2 = R.run_token_logprob(inp["hidden"], inp["weight"], tok, 1.0, W.BF16)
        np.testing.assert_allclose(lp2, lp, atol=2e-5)
        np.testing.assert_allclose(lse2, lse, atol=2e-5)


@pytest.mark.parametrize("C,H,V", sorted({(65, 768, 32769), (128, 1024, 45003), (160, 768, 33001), (129, 3072, 32770), (192, 768, 40001),
                                   (193, 768, 32771), (256, 768, 50257), (150, 64, 3), (256, 64, 12288), (200, 128, 8195),
                                   # two tiles per workgroup, the last of at most 128 rows and of more
                                   (130, 3072, 98307), (200, 1536, 98313), (250, 1536, 109999), (90, 3072, 120001),
                                   # 320 columns (one tile, two), two blocks of 160 (one slab per tile; more tiles), of 192, 256 and 320
                                   (257, 1024, 33001), (320, 1536, 65539), (301, 1024, 84003), (258, 64, 50257), (320, 64, 3),
                                   (321, 512, 16385), (384, 512, 20003), (385, 512, 16387), (512, 512, 20001), (600, 2048, 20001), *RUNS}))
def test_runs_of_vocabulary_rows(R, C, H, V):
    inp = W.make_small_lmhead_case(C * 19 + V, C, H, V, W.BF16, w_std=0.1)
    (tok, lp, lse), kernels = P.kernels_of(lambda: R.run_lmhead_logprob(inp, W.BF16))
    if (C, H, V) in RUNS:
        assert kernels == ["lmhead_run_kernel", "lmhead_merge_kernel"]
    # every row's log-sum-exp and log-prob follow from the logits; tokens are checked on a sample of rows (the noise
    # of a row is V numbers)
    rows = np.unique(np.concatenate([np.arange(0, C, max(1, C // 12)), [C - 1]]))
    P.check_lmhead(tok[rows], lp[rows], lse[rows], P.oracle_lmhead(inp, W.BF16, rows=rows), f"{C}x{H}x{V}")
    ref = P.oracle_token_logprob(inp["hidden"], inp["weight"], tok, 1.0, W.BF16)
    P.check_token_logprob(lp, lse, ref, f"{C}x{H}x{V}")
    if C < 384:   # the same tokens as given ones, and the vocabulary's ends
        given = tok.copy()
        given[:2] = [0, V - 1]
        lp2, lse2 = R.run_token_logprob(inp["hidden"], inp["weight"], given, 1.0, W.BF16)
        np.testing.assert_allclose(lp2[2:], lp[2:], atol=2e-5)
        np.testing.assert_allclose(lse2, lse, atol=2e-5)
        P.check_token_logprob(lp2[:2], lse2[:2], P.oracle_token_logprob(inp["hidden"], inp["weight"], given, 1.0, W.BF16, rows=np.arange(2)), "ends")


@pytest.mark.parametrize("C,H,V", [(1, 4, 3), (16, 60, 64), (17, 68, 65), (32, 132, 63), (33, 1028, 129), (8, 12, 4000)])
def test_fp32_ends_of_rows_and_quarters(R, C, H, V):
    # hidden sizes that leave a quarter, a step or part of a granule group empty
    inp = W.make_small_lmhead_case(C * 17 + H, C, H, V, W.F32, w_std=0.2)
    tok, lp, lse = R.run_lmhead_logprob(inp, W.F32)
    P.check_lmhead(tok, lp, lse, P.oracle_lmhead(inp, W.F32), f"f32 {C}x{H}x{V}")
    given = (np.arange(C) * 31 % V).astype(np.int32)
    lp2, lse2 = R.run_token_logprob(inp["hidden"], inp["weight"], given, 1.0, W.F32)
    P.check_token_logprob(lp2, lse2, P.oracle_token_logprob(inp["hidden"], inp["weight"], given, 1.0, W.F32), f"f32 given {C}x{H}x{V}")


@pytest.mark.parametrize("C,H,V", [*NARROW, *WIDE])
def test_tiles_of_many_narrow_row_blocks(R, C, H, V):
    # two to five blocks of 128 columns, more tiles than workgroups of one; one to three of 192 and of 256 (which of them:
    # test_row_blocks_narrow_and_wide)
    inp = W.make_small_lmhead_case(C * 29 + V, C, H, V, W.BF16, w_std=0.1)
    (tok, lp, lse), kernels = P.kernels_of(lambda: R.run_lmhead_logprob(inp, W.BF16))
    assert kernels == ["lmhead_mfma_kernel", "lmhead_merge_kernel"]
    rows = np.unique(np.concatenate([np.arange(0, C, max(1, C // 12)), [C - 1]]))
    P.check_lmhead(tok[rows], lp[rows], lse[rows], P.oracle_lmhead(inp, W.BF16, rows=rows), f"{C}x{H}x{V}")
    ref = P.oracle_token_logprob(inp["hidden"], inp["weight"], tok, 1.0, W.BF16)
    P.check_token_logprob(lp, lse, ref, f"{C}x{H}x{V}")
    if C < 384:
        lp2, lse2 = R.run_token_logprob(inp["hidden"], inp["weight"], tok, 1.0, W.BF16)
        P.check_token_logprob(lp2, lse2, ref, f"given {C}x{H}x{V}")


@pytest.mark.parametrize("dtype", [W.BF16, W.F32])
@pytest.mark.parametrize("C,H,V", [*SMALL, (1, 64, 1), (16, 64, 15), (17, 64, 17), (33, 128, 33), (65, 576, 65), (512, 64, 129),   # ends of tiles
                                   (15, 512, 63), (31, 1088, 1021), (64, 1984, 131), (3, 8192, 333)])   # runs of unequal and of no steps
def test_small_calls(R, dtype, C, H, V):
    inp = W.make_small_lmhead_case(C * 23 + V, C, H, V, dtype, w_std=0.05)
    (tok, lp, lse), kernels = P.kernels_of(lambda: R.run_lmhead_logprob(inp, dtype))
    assert kernels == ["lmhead_small_kernel", "lmhead_merge_kernel"]
    P.check_lmhead(tok, lp, lse, P.oracle_lmhead(inp, dtype), f"{dtype} {C}x{H}x{V}")
    given = np.where(np.arange(C) % 2 == 0, tok, np.arange(C) * 37 % V).astype(np.int32)
    given[-1] = V - 1
    lp2, lse2 = R.run_token_logprob(inp["hidden"], inp["weight"], given, 1.0, dtype)
    P.check_token_logprob(lp2, lse2, P.oracle_token_logprob(inp["hidden"], inp["weight"], given, 1.0, dtype), f"given {dtype} {C}x{H}x{V}")


@pytest.mark.parametrize("dtype", [W.BF16, W.F32])
def test_small_calls_with_room_for_a_partial_per_64_rows_only(R, dtype):
    # 16 x 16 tiles want four times as many: a workspace without the room takes larger tiles, and nothing is refused
    import torch

    from paper_2511_05589_amd import binding
    C, H, V = 5, 1024, 3003
    inp = W.make_small_lmhead_case(77, C, H, V, dtype, w_std=0.05)
    ref = P.oracle_lmhead(inp, dtype)
    least = -(-C * -(-V // 64) * 20 // 256) * 256
    for room in (least, 2 * least, binding.lmhead_logprob_workspace_bytes(C, H, V)):
        d = R.stage_lmhead(inp, dtype)
        d.ws = torch.empty(room + 4096, dtype=torch.uint8, device=d.ws.device).fill_(0x5a)[:room]
        behind = torch.as_strided(d.ws, (4096,), (1,), room)
        d.run()
        torch.cuda.synchronize()
        P.check_lmhead(d.token.cpu().numpy(), d.logprob.cpu().numpy(), d.lse.cpu().numpy(), ref, f"{dtype} {room}")
        assert (behind == 0x5a).all()
    assert binding.lmhead_logprob_workspace_bytes(C, H, V) > least


@pytest.mark.parametrize("dtype,C,H,V", [(W.BF16, 1, 3584, 3483), (W.BF16, 3, 512, 1009), (W.BF16, 8, 2048, 7732), (W.BF16, 24, 3584, 3185), (W.BF16, 41, 3584, 3251),
                                         (W.F32, 6, 256, 1009), (W.F32, 5, 1024, 3003), (W.F32, 20, 512, 5000), (W.F32, 48, 256, 146851)])
def test_small_calls_do_not_depend_on_the_room(R, dtype, C, H, V):
    # tiles of 16 and 32 vocabulary rows with the workspace that is asked for, of 64 with the smallest that is accepted: the same bits
    import torch

    from paper_2511_05589_amd import binding
    inp = W.make_small_lmhead_case(C * 19 + V, C, H, V, dtype, w_std=0.05)
    least, asked = -(-C * -(-V // 64) * 20 // 256) * 256, binding.lmhead_logprob_workspace_bytes(C, H, V)
    assert asked > least
    got = []
    for room in (asked, least, 2 * least - 256, 4 * asked):
        d = R.stage_lmhead(inp, dtype)
        d.ws = torch.empty(room, dtype=torch.uint8, device=d.ws.device)
        d.run()
        torch.cuda.synchronize()
        got.append([x.cpu().numpy() for x in (d.token, d.logprob, d.lse)])
    for other in got[1:]:
        for a, b in zip(got[0], other):
            np.testing.assert_array_equal(a, b)


def test_small_calls_infinities(R):
    # as in the other kernels: an infinite logit has no log-prob, minus infinity no weight, and no other row is touched
    import torch
    for dtype in (W.BF16, W.F32):
        C, H, V = 6, 64, 700
        inp = W.make_small_lmhead_case(3, C, H, V, dtype, w_std=0.05)
        clean = R.run_lmhead_logprob(inp, dtype)
        d = R.stage_lmhead(inp, dtype)
        d.weight[5].fill_(0.0)
        d.weight[5, 0] = float("inf")                    # logit of entry 5: infinite where hidden[0] is not 0
        d.hidden[:, 0] = -1.0
        d.hidden[2, 0] = float("nan")
        d.run()
        torch.cuda.synchronize()
        tok, lp, lse = d.token.cpu().numpy(), d.logprob.cpu().numpy(), d.lse.cpu().numpy()
        others = np.arange(C) != 2
        assert np.isfinite(lp[others]).all() and np.isfinite(lse[others]).all() and (tok[others] != 5).all()
        assert not np.isfinite(lp[2])
        assert np.isfinite(clean[1]).all()


def test_zero_weights_token_is_argmax_of_the_noise(R):
    # isolates the Philox counter layout and the uniform -> Gumbel mapping
    C, H, V = 16, 64, 5000
    inp = W.make_small_lmhead_case(1, C, H, V, W.F32)
    inp["weight"] = np.zeros_like(inp["weight"])
    inp["seq_id"][3] = (7 << 32) | 5             # exercise the high counter word
    inp["step"][4] = 70000
    tok, lp, lse = R.run_lmhead_logprob(inp, W.F32)
    for c in range(C):
        g = O.gumbel_noise(inp["seed"], int(inp["seq_id"][c]), int(inp["step"][c]), V)
        order = np.argsort(-g)
        assert tok[c] == order[0] or (g[order[0]] - g[order[1]] < P.NEAR_TIE and tok[c] == order[1])
    np.testing.assert_allclose(lp, -math.log(V), atol=1e-5)


def test_temperature_and_row_permutation(R):
    inp = W.make_small_lmhead_case(9, 24, 256, 3000, W.BF16, w_std=0.1)
    inp["temperature"] = 0.6
    tok, lp, lse = R.run_lmhead_logprob(inp, W.BF16)
    P.check_lmhead(tok, lp, lse, P.oracle_lmhead(inp, W.BF16), "T=0.6")
    perm = np.random.default_rng(0).permutation(24)
    inp2 = dict(inp)
    for k in ("hidden", "seq_id", "step"):
        inp2[k] = inp[k][perm]
    tok2, lp2, lse2 = R.run_lmhead_logprob(inp2, W.BF16)
    np.testing.assert_array_equal(tok[perm], tok2)
    np.testing.assert_array_equal(lp[perm], lp2)


@pytest.mark.parametrize("C", [48, 200])
def test_log_sum_exp_has_no_bias(R, C):
    # an fp32 result near 11 is rounded by up to 4.8e-7, 2.8e-7 rms: the mean of C rows stays within 4 / sqrt(C) of that
    # plus 5e-8 for the exponentials' and the scale's own rounding (logf in the last step was 3.2e-7 off on average)
    inp = W.make_small_lmhead_case(77, C, 512, 20001, W.BF16, w_std=0.05)
    _, _, lse = R.run_lmhead_logprob(inp, W.BF16)
    assert abs((lse.astype(np.float64) - P.oracle_lmhead(inp, W.BF16)["lse"]).mean()) <= 4 * 2.8e-7 / math.sqrt(C) + 5e-8


# (C, H, V): together these reach every kernel, sampling and with given tokens (rows of 128 .. 320, the skinny one, the
# 256 x 256 one with a last block of another width and without, the generic one)
EVERY_KERNEL = [(48, 384, 65537), (20, 64, 5003), (200, 64, 20011), (200, 128, 8195), (150, 512, 8195), (300, 512, 3001), (320, 1024, 33001),
                (400, 64, 20011), (448, 64, 20011), (5, 72, 260)]
WIDE_BLOCKS = [(160, 512, 20011), (200, 512, 20011)]   # tiles with 192 and 256 columns


def _scored(R, hidden, weight, temperature):
    """tokens, log-probs, log-sum-exps of a sampling call, and the latter two of its tokens as given ones (stored operands)"""
    C, V = len(hidden), len(weight)
    inp = dict(hidden=hidden, weight=weight, seq_id=np.arange(C, dtype=np.int64), step=np.zeros(C, np.int32), seed=5,
               temperature=temperature, C=C, H=hidden.shape[1], V=V, dtype=W.BF16)
    tok, lp, lse = R.run_lmhead_logprob(inp, W.BF16)
    assert ((0 <= tok) & (tok < V)).all()
    return tok, (lp, lse), R.run_token_logprob(hidden, weight, tok, temperature, W.BF16)


@pytest.mark.parametrize("C,H,V", EVERY_KERNEL + WIDE_BLOCKS + [(5, 64, 1), (200, 64, 1), (300, 64, 1), (400, 64, 1)])
def test_a_peaked_row_has_no_positive_log_prob(R, C, H, V):
    # one logit of lo .. 2 * lo, the others noise around 0: the log-prob is -ln(1 + less than 70000 e^-35), so 0 up to the
    # rounding of a sum near 1 and of its logarithm.  The last two are near the end of fp32's range.
    rng = np.random.default_rng(C + V)
    noise, peak = rng.standard_normal(V), V // 3
    for T, lo, amp in ((1.0, 40.0, 1.0), (0.6, 40.0, 1.0), (0.1, 40.0, 1.0), (1.0, 1.5e38, 1.0), (3.5e-39, 0.5, 0.0)):
        hidden, weight = np.zeros((C, H), np.float32), np.zeros((V, H), np.float32)
        hidden[:, 0] = lo * (1 + np.arange(C) % 128 / 128)
        hidden[:, 1] = 1
        weight[:, 1] = amp * T * noise
        weight[peak] = 0
        weight[peak, 0] = 1
        hidden = W.to_storage(hidden, W.BF16)
        tok, *scored = _scored(R, hidden, W.to_storage(weight, W.BF16), T)
        assert (tok == peak).all()
        z = W.to_f32(hidden, W.BF16)[:, 0] * (np.float32(1) / np.float32(T))
        for lp, lse in scored:
            assert (lp <= 0).all() and (lp >= -1e-6).all(), (T, lo, lp.min(), lp.max())
            np.testing.assert_allclose(lse, z, rtol=3e-7)


@pytest.mark.parametrize("C,H,V", EVERY_KERNEL + WIDE_BLOCKS)
def test_log_probs_have_no_bias_at_any_temperature(R, C, H, V):
    # Logits whose fp32 sums are exact (small whole numbers over a power of two), deviation 3 to 5 around 20, so that what
    # differs from the 64-bit log-prob is the rounding of the temperature, of the exponentials and of the results.
    rng = np.random.default_rng(C * 3 + H)
    hidden, weight = (rng.integers(-4, 5, size=(n, H), dtype=np.int8).astype(np.float32) for n in (C, V))
    weight /= 2.0 ** round(math.log2(6.67 * math.sqrt(H) / 4))
    hidden[:, 0], weight[:, 0] = 4, 5
    logits = (hidden @ weight.T).astype(np.float64)
    hidden, weight = W.to_storage(hidden, W.BF16), W.to_storage(weight, W.BF16)
    for T in (0.1, 0.55, 0.6, 1.0, 1.05, 1.1):
        tok, *scored = _scored(R, hidden, weight, T)
        z = logits / float(np.float32(T))
        m = z.max(axis=1, keepdims=True)
        p = np.exp(z - m)
        s = p.sum(axis=1)
        lse, chosen, mean = m[:, 0] + np.log(s), z[np.arange(C), tok], (p * z).sum(axis=1) / s
        # 1 / T and log2(e) / T are off by up to 2^-24 of a logit's distance from the mean one; the chosen logit and the
        # maximum are rounded to 24 bits, and so is the result (ulp / sqrt(12) each, four deviations of the rows' mean);
        # 1e-7 for the hardware's exponential and logarithm
        ulp = lambda x: 2.0 ** (np.ceil(np.log2(np.abs(x).max())) - 24)  # noqa: E731
        bound = (2.0 ** -24 * (np.abs(chosen - mean) + (m[:, 0] - mean)).mean() + 1e-7
                 + 4 * math.sqrt((2 * ulp(m) ** 2 + ulp(chosen - lse) ** 2) / 12 / C))
        for what, (lp, _) in zip(("sampled", "given"), scored):
            bias = (lp - (chosen - lse)).mean()
            print(f"{what} {C}x{H}x{V} T={T}: bias {bias:+.2e}, bound {bound:.2e}", flush=True)
            assert abs(bias) <= bound, (what, T, bias, bound)


def test_bitwise_reproducible(R):
    inp = W.make_small_lmhead_case(10, 40, 512, 7000, W.BF16)
    a, b = R.run_lmhead_logprob(inp, W.BF16), R.run_lmhead_logprob(inp, W.BF16)
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("k", [1, 2])
def test_full_size_configs_every_row(R, k):
    # the 1.5B- and 7B-shaped LM heads (vocabulary 151936): every one of the C rows
    cfg = W.DECODE_CONFIGS[k]
    inp = W.make_decode_inputs(cfg, with_attn=False)
    tok, lp, lse = R.run_lmhead_logprob(inp, cfg.dtype)
    assert ((0 <= tok) & (tok < cfg.V)).all() and np.isfinite(lp).all() and (lp <= 0).all()
    exempt = 0
    for r0 in range(0, cfg.C, 64):            # 64 rows of full log-softmax at a time (78 MB in fp64)
        rows = np.arange(r0, min(r0 + 64, cfg.C))
        ref = P.oracle_lmhead(inp, cfg.dtype, rows=rows)
        exempt += P.check_lmhead(tok[rows], lp[rows], lse[rows], ref, f"cfg{k} rows {r0}..")
    assert exempt <= 2
