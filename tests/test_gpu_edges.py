"""GPU kernels at the sizes where their tilings and dispatch rules change, against plain restatements in
64-bit arithmetic (or the oracle)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _fb():
    from paper_2511_05534_amd import binding as fb
    return fb


DECODE_EDGES = {  # budgets, q heads, kv heads, head_dim, and "f32" for fp32 caches
    "tile_remainders": ([1, 15, 16, 17, 127, 128, 129, 255], 7, 1, 128),
    "tile_remainders_d64": ([1, 15, 16, 17, 127, 128, 129, 257], 4, 2, 64),
    "cut_into_several": ([416, 417, 831, 832, 833, 2000], 2, 1, 128),
    "whole": ([416], 16, 1, 128),
    "whole_at_the_limit": ([512, 400], 16, 1, 128),
    "equal_parts": ([1500, 1500], 7, 1, 128),
    "equal_parts_with_a_remainder": ([1501], 4, 1, 64),
    "two_passes_over_the_heads": ([33, 450], 17, 1, 64),
    "two_launches_of_sequences": ([3 + (i % 5) for i in range(66)], 2, 2, 64),
    "longest": ([13400], 1, 1, 64),
    "longest_of_unequal": ([20000, 511, 513], 1, 1, 64),
    "two_waves": ([1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 97, 128] * 5, 45, 15, 128),
    "two_waves_d64_two_passes_over_the_heads": ([1, 16, 17, 32, 33, 64, 65, 129] * 5, 272, 16, 64),
    "four_waves": ([1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 500, 512] * 4, 40, 10, 128),
    "four_waves_d64": ([70, 127, 257, 512] * 12, 32, 8, 64),
    "one_long_among_short": ([5000] + [20] * 59, 18, 18, 64),
    # more than 1024 tasks: units in turn, then the last ones' tasks by length
    "units_in_turn_then_by_length": ([1, 17, 40, 64, 100, 129, 33, 80, 96], 64, 64, 64),
    "units_in_turn_eight_tasks": ([129, 5, 64, 16, 15, 100, 128, 33], 65, 65, 64),
    "units_in_turn_cut": ([20, 16, 2000, 15, 40, 512, 17, 1, 21], 60, 60, 64),
    "parts_without_rests": ([1024, 1536, 512], 2, 1, 64),
    "nearly_equal_on_few_more_units_than_half": ([1700, 1690], 65, 65, 128),
    "long_one_in_the_last_launch": ([200 + i % 3 for i in range(128)] + [1100, 150], 2, 2, 64),
    "one_far_above_the_others": ([40, 30, 20, 60, 4100, 50, 33, 17], 64, 64, 64),
    "long_ones_in_order": ([980, 160, 500, 700, 300, 820, 400, 640], 56, 56, 64),
    "f32_units_in_turn": ([1, 17, 40, 64, 100, 129, 33, 80, 96], 64, 64, 64, "f32"),
    "f32_trip_remainders": ([1, 7, 8, 31, 32, 33, 65], 7, 1, 128, "f32"),
    "f32_trip_remainders_d64": ([1, 15, 16, 63, 64, 65, 129], 4, 2, 64, "f32"),
    "f32_cut_into_several": ([416, 417, 833, 2000], 2, 1, 128, "f32"),
    "f32_equal_parts": ([830], 7, 1, 128, "f32"),
    "f32_one_head": ([700, 300], 1, 1, 64, "f32"),
    "f32_two_passes_over_the_heads": ([33, 450], 11, 1, 64, "f32"),
    "f32_two_launches_of_sequences": ([40 + 50 * (i % 3) for i in range(66)], 4, 2, 64, "f32"),
    "f32_longest": ([13400], 3, 1, 64, "f32"),
}


@pytest.mark.parametrize("name", list(DECODE_EDGES))
def test_decode_attention_at_tile_edges(name):
    import torch
    fb = _fb()
    budgets, Hq, Hkv, d, dtype = (*DECODE_EDGES[name], "bf16")[:5]
    print(f"case {name}: budgets {budgets[:8]} Hq {Hq} Hkv {Hkv} d {d} {dtype}", flush=True)
    n = len(budgets)
    params = fb.Params(2, Hq, Hkv, d, dtype, budgets, budgets, [[(0, B, 0)] for B in budgets], 1, 0.25, [1.0] * n)
    bufs = fb.DeviceBuffers(params)
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    bufs.K_out.normal_(generator=gen)
    bufs.V_out.normal_(generator=gen)
    q = (2.0 * torch.randn((2, Hq, n, d), generator=gen, device="cuda:0")).to(bufs.K_out.dtype)
    out = torch.full_like(q, float("nan"))
    bufs.decode_attention(q, out, stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    K, V, qd, got = (t.double().cpu().numpy() for t in (bufs.K_out, bufs.V_out, q, out))
    cu, G = np.concatenate([[0], np.cumsum(budgets)]), Hq // Hkv
    for l in range(2):
        for h in range(Hq):
            for b in range(n):
                rows = slice(cu[b], cu[b + 1])
                s = K[l, h // G, rows] @ qd[l, h, b] / np.sqrt(d)
                p = np.exp(s - s.max())
                want = (p / p.sum()) @ V[l, h // G, rows]
                # rounding to the 8 (24) significant bits of bf16 (fp32) is at most 2^-8 (2^-24) of the value; the weights carry the fp32 rounding of logits up to
                # |s| ~ 30 (2^-24 |s| a weight) and of exp2, at values up to max |V|
                tol = (2.0 ** -8 if dtype == "bf16" else 2.0 ** -24) * np.abs(want) * 1.01 + 1e-5 * np.abs(V[l, h // G, rows]).max()
                assert (np.abs(got[l, h, b] - want) <= tol).all(), (l, h, b, np.abs(got[l, h, b] - want).max())


@pytest.mark.parametrize("name,cut", [("nearly_equal_on_few_more_units_than_half", True), ("long_one_in_the_last_launch", True),
                                      ("one_far_above_the_others", True), ("long_ones_in_order", False), ("two_launches_of_sequences", False)])
def test_decode_attention_cuts_sequences(name, cut):
    """A sequence goes to several workgroups (whose results a second kernel puts together) where a compute unit would be left with much more than its
    share, counted over the sequences of its launch."""
    import torch
    from parity_utils import launched
    fb = _fb()
    budgets, Hq, Hkv, d = DECODE_EDGES[name]
    n = len(budgets)
    params = fb.Params(2, Hq, Hkv, d, "bf16", budgets, budgets, [[(0, B, 0)] for B in budgets], 1, 0.25, [1.0] * n)
    bufs = fb.DeviceBuffers(params)
    bufs.K_out.zero_()
    bufs.V_out.zero_()
    q = torch.zeros((2, Hq, n, d), dtype=torch.bfloat16, device="cuda:0")
    with launched() as kernels:
        bufs.decode_attention(q, torch.empty_like(q), stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    assert "decode_partial" in kernels and ("decode_combine" in kernels) == cut, kernels


def test_decode_attention_rows_of_no_weight():
    """Rows whose logit is -inf for every head weigh nothing, also where they fill whole tiles of 16."""
    import torch
    fb = _fb()
    B, Hq, d = 200, 7, 128
    params = fb.Params(1, Hq, 1, d, "bf16", [B], [B], [[(0, B, 0)]], 1, 0.25, [1.0])
    bufs = fb.DeviceBuffers(params)
    gen = torch.Generator(device="cuda:0").manual_seed(4)
    bufs.K_out.normal_(generator=gen)
    bufs.V_out.normal_(generator=gen)
    q = torch.randn((1, Hq, 1, d), generator=gen, device="cuda:0").to(torch.bfloat16)
    q[..., 0] = 1.0
    out = torch.empty_like(q)
    for masked in (slice(0, 40), slice(150, 200), slice(30, 190)):
        K = bufs.K_out.clone()
        bufs.K_out[..., masked, 0] = float("-inf")
        bufs.decode_attention(q, out, stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        seen = torch.ones(B, dtype=torch.bool)
        seen[masked] = False
        Kd, V, qd, got = (t.double().cpu().numpy() for t in (K[0, 0], bufs.V_out[0, 0], q[0, :, 0], out[0, :, 0]))
        s = qd @ Kd[seen.numpy()].T / np.sqrt(d)
        p = np.exp(s - s.max(axis=1, keepdims=True))
        want = (p / p.sum(axis=1, keepdims=True)) @ V[seen.numpy()]
        tol = 2.0 ** -8 * np.abs(want) * 1.01 + 1e-5 * np.abs(V).max()  # as above
        assert (np.abs(got - want) <= tol).all(), (masked, np.abs(got - want).max())
        bufs.K_out.copy_(K)


@pytest.mark.parametrize("dtype,d,B", [("bf16", 64, 40), ("bf16", 128, 200), ("bf16", 128, 900), ("f32", 64, 40), ("f32", 128, 200)])
def test_decode_attention_of_infinite_values(dtype, d, B):
    """An infinite element of a V row makes its output channel infinite, also where the row's weight is a power of two."""
    import torch
    fb = _fb()
    print(f"{dtype} d {d} B {B}", flush=True)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    params = fb.Params(1, 2, 1, d, dtype, [B], [B], [[(0, B, 0)]], 1, 0.25, [1.0])
    bufs = fb.DeviceBuffers(params)
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    bufs.K_out.normal_(generator=gen)
    bufs.V_out.normal_(generator=gen)
    V = bufs.V_out[0, 0]
    V[3, 0], V[17, 1], V[B // 2, d - 1] = float("inf"), float("-inf"), float("inf")
    q = torch.randn((1, 2, 1, d), generator=gen, device="cuda:0").to(tdt)
    q[0, 0], q[0, 1] = 0.0, bufs.K_out[0, 0, 17]  # every weight 1 before the sum; row 17 the largest
    out = torch.empty_like(q)
    bufs.decode_attention(q, out, stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    Kd, Vd, qd, got = (t.double().cpu().numpy() for t in (bufs.K_out[0, 0], V, q[0, :, 0], out[0, :, 0]))
    s = qd @ Kd.T / np.sqrt(d)
    p = np.exp(s - s.max(axis=1, keepdims=True))
    want = (p / p.sum(axis=1, keepdims=True)) @ Vd
    inf = np.isinf(want)
    assert inf.sum() == 6 and (got[inf] == want[inf]).all(), got[inf]
    tol = 2.0 ** -8 * np.abs(want[~inf]) * 1.01 + 1e-5 * np.abs(Vd[np.isfinite(Vd)]).max()  # as above
    assert (np.abs(got[~inf] - want[~inf]) <= tol).all()


@pytest.mark.parametrize("batch,dtype,d", [(1, "bf16", 64), (8, "bf16", 128), (9, "f32", 64), (64, "f32", 128), (67, "bf16", 64)])
def test_cache_append_batches(batch, dtype, d):
    """One new row per sequence at the batch sizes where the launches change; everything else stays as it was."""
    import torch
    fb = _fb()
    print(f"batch {batch} {dtype} d {d}", flush=True)
    caps = [2 + b % 3 for b in range(batch)]
    cu = np.concatenate([[0], np.cumsum(caps)])
    lengths = np.array([b % c for b, c in enumerate(caps)], dtype=np.int64)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    params = fb.Params(3, 4, 2, d, dtype, caps, [1] * batch, [[(0, c, 0)] for c in caps], 1, 0.25, [1.0] * batch)
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    K, V = (torch.randn((3, 2, int(cu[-1]), d), generator=gen, device="cuda:0").to(tdt) for _ in range(2))
    k, v = (torch.randn((3, 2, batch, d), generator=gen, device="cuda:0").to(tdt) for _ in range(2))
    want_K, want_V = K.clone(), V.clone()
    rows = torch.from_numpy(cu[:-1] + lengths).to("cuda:0")
    want_K[:, :, rows], want_V[:, :, rows] = k, v
    fb.flowmm_cache_append(params, cu, lengths, K.data_ptr(), V.data_ptr(), k.data_ptr(), v.data_ptr(),
                           torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(K, want_K) and torch.equal(V, want_V)


def test_cache_append_takes_any_token_stride():
    """The token stride of a cache may exceed 32 bits of 16-byte chunks (here with one row per sequence in use)."""
    import torch
    fb = _fb()
    d = 64
    params = fb.Params(1, 1, 1, d, "bf16", [4], [1], [[(0, 4, 0)]], 1, 0.25, [1.0], k_strides=(0, 0, 1 << 35))
    K, V, k, v = (torch.randn((1, 1, 1, d), device="cuda:0").to(torch.bfloat16) for _ in range(4))
    fb.flowmm_cache_append(params, [0, 4], [0], K.data_ptr(), V.data_ptr(), k.data_ptr(), v.data_ptr(),
                           torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(K, k) and torch.equal(V, v)


FLOW_EDGES = {  # lengths, q heads, kv heads, head_dim, dtype, span lengths cycled through (text first), token stride or 0
    "block_remainders": ([1, 31, 32, 33, 63, 64, 65, 127], 3, 1, 128, "bf16", [5, 40, 3], 0),
    "tile_remainders_d64": ([128, 129, 191, 255, 257, 300], 8, 2, 64, "bf16", [64, 64], 0),
    "many_spans_in_a_block": ([150, 70], 2, 2, 128, "bf16", [1, 2, 1, 7], 0),
    "f32_remainders": ([1, 31, 33, 64, 65, 129], 3, 1, 128, "f32", [5, 40, 3], 0),
    "f32_d64": ([97, 256, 130], 2, 2, 64, "f32", [32, 33], 0),
    "rows_beyond_32_bit_offsets": ([39], 1, 1, 128, "bf16", [5, 11], 1 << 24),
    "keys_in_four": ([700, 129, 33], 5, 1, 64, "bf16", [100, 300], 0),
    "keys_in_two": ([900, 64], 96, 32, 64, "bf16", [100, 300], 0),
    "keys_whole": ([130, 65, 64, 129, 40, 130, 1], 512, 128, 64, "bf16", [30, 50], 0),
    "units_in_unequal_groups": ([40, 9] * 300, 6, 6, 64, "bf16", [7, 12], 0),
    "units_not_a_multiple_of_eight": ([260, 65], 15, 5, 128, "bf16", [64, 32, 7], 0),
    "f32_keys_in_two": ([500, 66], 3, 1, 128, "f32", [100, 150], 0),
    "f32_keys_in_four": ([500, 66], 3, 1, 64, "f32", [100, 150], 0),
}


@pytest.mark.parametrize("name", list(FLOW_EDGES))
def test_flow_exact_at_tile_edges(name):
    """The ratio over all queries where query blocks, key tiles and modality spans end, against the dense attention in 64 bits."""
    import torch
    fb = _fb()
    lens, Hq, Hkv, d, dtype, cycle, stride = FLOW_EDGES[name]
    print(f"case {name}: lengths {lens} Hq {Hq} Hkv {Hkv} d {d} {dtype}", flush=True)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    spans = []
    for L in lens:
        one, pos, j = [], 0, 0
        while pos < L:
            end = min(L, pos + cycle[j % len(cycle)])
            one.append((pos, end, j % 2))
            pos, j = end, j + 1
        spans.append(one)
    T, n = sum(lens), len(lens)
    layers = 1 if stride else 2
    params = fb.Params(layers, Hq, Hkv, d, dtype, lens, [1] * n, spans, 1, 0.25, [1.0] * n,
                       k_strides=(Hkv * T * stride, T * stride, stride) if stride else None)
    gen = torch.Generator(device="cuda:0").manual_seed(2)
    K = torch.randn((layers, Hkv, T, d), generator=gen, device="cuda:0").to(tdt)
    Q = (2.0 * torch.randn((layers, Hq, T, d), generator=gen, device="cuda:0")).to(tdt)
    Kd = K
    if stride:
        Kd = torch.empty((T - 1) * stride + d, dtype=tdt, device="cuda:0")
        Kd.as_strided((T, d), (stride, 1)).copy_(K[0, 0])
    bufs = fb.DeviceBuffers(params)
    bufs.rho.fill_(-1.0)
    bufs.flow_exact(Kd, Q, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = bufs.rho.cpu().numpy()
    Kn, Qn = K.double().cpu().numpy(), Q.double().cpu().numpy()
    cu = np.concatenate([[0], np.cumsum(lens)])
    for l in range(layers):
        for b, L in enumerate(lens):
            sl = slice(cu[b], cu[b + 1])
            img = np.zeros(L, bool)
            for s, e, m in spans[b]:
                img[s:e] = m == 1
            want = 0.0
            for h in range(Hq):
                s = Qn[l, h, sl] @ Kn[l, h // (Hq // Hkv), sl].T / np.sqrt(d)
                s[np.triu_indices(L, 1)] = -np.inf
                p = np.exp(s - s.max(axis=1, keepdims=True))
                p /= p.sum(axis=1, keepdims=True)
                want += (p * (img[:, None] != img[None, :])).sum() / L / Hq
            # every weight carries the fp32 rounding of its logit (2^-24 |s|, |s| up to ~ 40) and of exp2 and the sums: below 1e-5
            assert abs(got[l, b] - want) <= 1e-5 * want + 1e-7, (l, b, got[l, b], want)


SCORE_EDGES = {  # lengths, q heads, kv heads, head_dim, window, dtype
    "one_workgroup_of_eight": ([70, 511, 512, 321], 6, 2, 128, 33, "bf16"),
    "one_workgroup_of_sixteen": ([513, 1024, 960, 961], 6, 2, 128, 33, "bf16"),
    "several_workgroups": ([1025, 512, 40], 6, 2, 128, 33, "bf16"),
    "sixteen_waves_d64": ([1023, 65], 8, 1, 64, 32, "bf16"),
    "f32_eight": ([256, 255, 97], 4, 1, 64, 40, "f32"),
    "f32_sixteen": ([512, 257], 2, 1, 128, 16, "f32"),
    "f32_several": ([513, 64], 2, 1, 128, 16, "f32"),
    "streamed_128_rows": ([1025, 1152, 1153, 64], 8, 2, 128, 32, "bf16"),
    "streamed_224_rows_text_window": ([2048, 1100, 40, 3001], 7, 1, 128, 20, "bf16"),
    "streamed_256_rows_mixed_window": ([1281, 130, 1279], 4, 1, 128, 64, "bf16"),
    "streamed_96_rows_d64_text_window": ([1055, 1056, 1057], 3, 1, 64, 32, "bf16"),
    "streamed_long_runs_text_window": ([4300, 2049], 8, 1, 64, 32, "bf16"),
    "resident_sixteen_by_units": ([1024, 800], 68, 68, 64, 32, "bf16"),
    "streamed_short_by_units": ([700, 513], 8, 1, 64, 32, "bf16"),
    "streamed_below_one_tile": ([100, 33], 7, 1, 128, 20, "bf16"),
    "streamed_short_of_unequal_lengths": ([1000, 100, 33, 70], 96, 32, 64, 32, "bf16"),
    "f32_three_kernels_by_units": ([512, 300], 4, 1, 64, 40, "f32"),
    "f32_sixteen_by_units": ([500], 66, 66, 64, 16, "f32"),
    "streamed_runs_of_three_tiles": ([5000], 24, 8, 64, 32, "bf16"),
    "streamed_runs_of_four_tiles_mixed_window": ([8300, 1100, 300], 56, 8, 64, 20, "bf16"),
    "streamed_one_run_text_window": ([1100, 1025], 384, 128, 64, 32, "bf16"),
    # windows that are no whole blocks of 32 query rows lie next to each other; one to six blocks of rows
    "streamed_four_heads_of_16": ([1100, 1025, 70], 4, 1, 64, 16, "bf16"),
    "streamed_three_heads_of_5_text_window": ([1300, 600], 6, 2, 128, 5, "bf16"),
    "streamed_heads_across_blocks_text_window": ([1030, 1500], 5, 1, 128, 20, "bf16"),
    "streamed_heads_across_blocks": ([1030, 1500], 5, 1, 64, 20, "bf16"),
    "streamed_32_rows_text_window": ([2049, 1100], 2, 2, 128, 32, "bf16"),
    "streamed_64_rows": ([2049, 130], 2, 1, 128, 32, "bf16"),
    "streamed_160_rows": ([1100, 900], 10, 2, 128, 32, "bf16"),
    "streamed_192_rows_text_window": ([1100, 385], 12, 2, 64, 32, "bf16"),
    "streamed_on_ten_units": ([3000], 10, 5, 64, 16, "bf16"),
    "resident_four_heads_of_16": ([500, 300], 4, 1, 64, 16, "bf16"),
    "resident_sixteen_two_heads_of_9": ([1000], 88, 44, 64, 9, "bf16"),
    "three_kernels_nine_heads_of_33": ([1100, 200], 18, 2, 64, 33, "bf16"),
    "f32_three_heads_of_10": ([700, 64], 6, 2, 64, 10, "f32"),
    "f32_six_heads_of_11": ([600, 300], 12, 2, 128, 11, "f32"),
}


@pytest.mark.parametrize("name", list(SCORE_EDGES))
def test_importance_where_the_score_kernels_change(name):
    """Importances and the proxy flow ratio against dense attention in 64 bits, around the lengths that one workgroup takes whole."""
    import torch
    fb = _fb()
    lens, Hq, Hkv, d, W, dtype = SCORE_EDGES[name]
    print(f"case {name}: lengths {lens} Hq {Hq} Hkv {Hkv} d {d} W {W} {dtype}", flush=True)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    n, T, G = len(lens), sum(lens), Hq // Hkv
    tail = W + 3 if "text_window" in name else W // 2  # text tokens at the end
    spans = [[(0, L // 3, 0), (L // 3, L - tail, 1), (L - tail, L, 0)] if L // 3 < L - tail else [(0, L, 0)] for L in lens]
    budgets = [min(L, W + 5) for L in lens]
    params = fb.Params(2, Hq, Hkv, d, dtype, lens, budgets, spans, W, 0.25, [1.0] * n, flags=fb.FLOWMM_FLAG_GENERIC_PATH)
    gen = torch.Generator(device="cuda:0").manual_seed(4)
    K = torch.randn((2, Hkv, T, d), generator=gen, device="cuda:0").to(tdt)
    Q = torch.randn((2, Hq, n * W, d), generator=gen, device="cuda:0").to(tdt)
    bufs = fb.DeviceBuffers(params)
    bufs.importance.fill_(float("nan"))
    bufs.plan(K, Q, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got, rho = bufs.importance.cpu().numpy(), bufs.rho.cpu().numpy()
    Kn, Qn = K.double().cpu().numpy(), Q.double().cpu().numpy()
    cu = np.concatenate([[0], np.cumsum(lens)])
    for l in range(2):
        for b, L in enumerate(lens):
            img = np.zeros(L, bool)
            img[L // 3:L - tail] = True
            cross = 0.0
            for g in range(Hkv):
                want = np.zeros(L)
                for h in range(g * G, g * G + G):
                    s = Qn[l, h, b * W:(b + 1) * W] @ Kn[l, g, cu[b]:cu[b + 1]].T / np.sqrt(d)
                    s[np.triu_indices(W, L - W + 1, L)] = -np.inf
                    p = np.exp(s - s.max(axis=1, keepdims=True))
                    p /= p.sum(axis=1, keepdims=True)
                    want += p.sum(axis=0) / (G * W)
                    cross += (p * (img[L - W:, None] != img[None, :])).sum() / W / Hq
                # a weight carries the fp32 rounding of its logit (2^-24 |s|, |s| < 10), of its row's constant and of exp2: below 1e-5
                assert np.allclose(got[l, g, cu[b]:cu[b + 1]], want, rtol=1e-5, atol=1e-9), (l, b, g)
            assert abs(rho[l, b] - cross) <= 1e-5 * cross + 1e-12, (l, b, rho[l, b], cross)


@pytest.mark.parametrize("L,B,dtype,d", [(129, 128, "bf16", 128), (300, 127, "bf16", 128), (700, 256, "bf16", 128), (640, 257, "bf16", 64),
                                         (3000, 2500, "bf16", 128), (3000, 2100, "bf16", 128), (400, 129, "f32", 128), (400, 200, "f32", 64)])
def test_remerge_in_place_gives_the_rows_of_a_merge_beside_it(L, B, dtype, d):
    """The rows a re-merge leaves at the head of the range against flowmm_plan_merge of the same rows; the rest stays as it was.
    (The sizes are around a round of slots, and on both sides of what fits LDS.)"""
    import torch
    fb = _fb()
    print(f"L {L} B {B} {dtype} d {d}", flush=True)
    W, Hq, Hkv = 20, 8, 2
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda:0").manual_seed(6)
    K = torch.randn((2, Hkv, L, d), generator=gen, device="cuda:0")
    K[:, :, : L // 2] = 0.9 * K[:, :, L // 4:L // 4 + 1] + 0.3 * K[:, :, : L // 2]  # many tokens resemble one
    K, V, Q = K.to(tdt), torch.randn((2, Hkv, L, d), generator=gen, device="cuda:0").to(tdt), None
    Q = torch.randn((2, Hq, W, d), generator=gen, device="cuda:0").to(tdt)
    stream = torch.cuda.current_stream().cuda_stream
    beside = fb.DeviceBuffers(fb.Params(2, Hq, Hkv, d, dtype, [L], [B], [[(0, L, 0)]], W, -1.0, [4.0 / B]))
    beside.plan_merge(K, V, Q, stream)
    params = fb.Params(2, Hq, Hkv, d, dtype, [L], [B], [[(0, L, 0)]], W, 0.25, [4.0 / B])
    sizes, ws = fb.flowmm_cache_remerge_sizes(params, [0, L], 0, L)
    kinds = [torch.float32, torch.float32, torch.int32, torch.int32, torch.int32, torch.int32]
    plan = [torch.empty(s // 4, dtype=t, device="cuda:0") for s, t in zip(sizes, kinds)]
    Kc, Vc = K.clone(), V.clone()
    space = torch.empty(ws, dtype=torch.uint8, device="cuda:0")
    fb.flowmm_cache_remerge(params, [0, L], [L], 0, Kc.data_ptr(), Vc.data_ptr(), Q.data_ptr(), [t.data_ptr() for t in plan],
                            space.data_ptr(), ws, stream)
    torch.cuda.synchronize()
    assert torch.equal(plan[3].view_as(beside.kept_idx), beside.kept_idx) and torch.equal(plan[4].view_as(beside.assign), beside.assign)
    assert torch.equal(Kc[:, :, B:], K[:, :, B:]) and torch.equal(Vc[:, :, B:], V[:, :, B:])
    for got, want, rows in ((Kc, beside.K_out, K), (Vc, beside.V_out, V)):
        # fp32 sums in another order (at most 3000 terms: 3000 x 2^-24 of the largest row), then one rounding to the data type
        a, b = got[:, :, :B].double(), want.double()
        tol = 2.0 ** (-7 if dtype == "bf16" else -23) * b.abs() + 3000 * 2.0 ** -24 * rows.double().abs().max()
        assert bool(((a - b).abs() <= tol).all())


@pytest.mark.parametrize("L,d,Hq,W,pct", [(256, 64, 2, 16, 20), (257, 64, 4, 16, 10), (385, 64, 2, 33, 20), (769, 64, 2, 16, 10), (1024, 64, 4, 8, 20),
                                          (256, 128, 2, 16, 20), (385, 128, 2, 40, 10), (512, 128, 4, 16, 25), (513, 128, 2, 16, 20)])
def test_f32_unit_path_lengths(oracle, L, d, Hq, W, pct):
    """fp32 prompts where the unit-resident kernels change their waves and key tiles, in both strategies, stage by stage against the oracle."""
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, run_gpu
    w = wl.make_workload("f32_unit", "f32", L, 2, Hq, 2, d, W, [[L // 5, L // 2, L - L // 5 - L // 2]], [pct])
    for theta in (-1.0, 2.0):
        print(f"L {L} d {d} Hq {Hq} W {W} theta {theta}", flush=True)
        gpu = run_gpu(w, theta=theta, fused=theta < 0)
        for l in range(w.n_layers):
            check_layer(oracle, w, gpu, l, theta=theta)


@pytest.mark.parametrize("layers,L,d,pct", [(12, 768, 64, 20), (12, 769, 64, 20), (12, 512, 128, 20), (20, 1024, 64, 20), (20, 1025, 64, 20), (20, 513, 128, 20),
                                            (11, 600, 64, 20), (11, 400, 128, 20)])
def test_f32_unit_path_by_units(oracle, layers, L, d, pct):
    """Longer fp32 prompts, which go to the unit-resident or the generic kernels by the number of units (88, 96, 160)."""
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, run_gpu
    w = wl.make_workload("f32_units", "f32", L, layers, 8, 8, d, 16, [[L // 5, L // 2, L - L // 5 - L // 2]], [pct])
    print(f"layers {layers} L {L} d {d}", flush=True)
    gpu = run_gpu(w, fused=True)
    for l in (0, layers - 1):
        check_layer(oracle, w, gpu, l)


@pytest.mark.parametrize("L,Hq,pct,dtype,d", [(385, 8, 10, "bf16", 128), (512, 16, 20, "bf16", 128), (513, 8, 20, "bf16", 128), (700, 16, 10, "bf16", 128),
                                              (768, 8, 10, "bf16", 64), (769, 8, 10, "bf16", 128), (520, 8, 10, "f32", 64)])
def test_unit_path_with_more_units_than_compute_units(oracle, L, Hq, pct, dtype, d):
    """Prompts whose plan workgroups share compute units (264 units), in both strategies, first and last layer against the oracle."""
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, run_gpu
    w = wl.make_workload("many_units", dtype, L, 33, Hq, 8, d, 24, [[L // 5, L // 2, L - L // 5 - L // 2]], [pct])
    for theta in (-1.0, 2.0):
        print(f"L {L} Hq {Hq} {dtype} d {d} theta {theta}", flush=True)
        gpu = run_gpu(w, theta=theta, fused=theta > 0)
        for l in (0, 32):
            check_layer(oracle, w, gpu, l, theta=theta)


@pytest.mark.parametrize("L,Hq,Hkv,W,pct,dtype,d", [(412, 4, 1, 16, 20, "bf16", 64), (1000, 8, 2, 16, 10, "bf16", 64), (300, 10, 2, 12, 20, "bf16", 128),
                                                    (200, 12, 1, 5, 20, "bf16", 128), (300, 3, 1, 21, 20, "f32", 64)])
def test_unit_path_of_packed_windows(oracle, L, Hq, Hkv, W, pct, dtype, d):
    """Windows that are no whole blocks of 32 query rows, up to 64 rows per kv head, in both strategies against the oracle."""
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, launched, run_gpu
    w = wl.make_workload("packed", dtype, L, 2, Hq, Hkv, d, W, [[L // 5, L // 2, L - L // 5 - L // 2 - W // 2, W // 2] if W > 1 else [L // 5, L - L // 5]], [pct])
    for theta in (-1.0, 2.0):
        print(f"L {L} heads {Hq}/{Hkv} W {W} {dtype} d {d} theta {theta}", flush=True)
        with launched() as kernels:
            gpu = run_gpu(w, theta=theta, fused=theta > 0)
        assert "unit_plan" in kernels, kernels
        for l in range(w.n_layers):
            check_layer(oracle, w, gpu, l, theta=theta)


@pytest.mark.parametrize("layers,unit", [(1, False), (32, True)])
def test_long_lists_of_few_units_leave_the_unit_path(oracle, layers, unit):
    """One workgroup per unit where there are many units or few candidates, the generic kernels otherwise."""
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, launched, run_gpu
    w = wl.make_workload("long_lists", "bf16", 1000, layers, 8, 4, 64, 16, [[200, 500, 300]], [20])
    with launched() as kernels:
        gpu = run_gpu(w, fused=True)
    assert ("unit_plan" in kernels) == unit, kernels
    check_layer(oracle, w, gpu, layers - 1)


@pytest.mark.parametrize("dtype,d,L", [("bf16", 64, 500), ("bf16", 128, 1100), ("f32", 64, 300), ("f32", 64, 700)])
def test_descriptions_in_and_beside_the_kernel_arguments(oracle, dtype, d, L):
    """One sequence of 150 spans travels in the arguments of the call's first kernel, two do not fit: both entry points against the oracle, and
    the exact ratio of the two against each alone."""
    import torch
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, run_gpu
    fb = _fb()
    step = L // 150
    one = [step] * 149 + [L - 149 * step]
    rho = []
    for n in (1, 2):
        w = wl.make_workload("spans", dtype, n * L, 2, 4, 2, d, 16, [one] * n, [10] * n)
        for fused in (False, True):
            print(f"{dtype} d {d} L {L} sequences {n} fused {fused}", flush=True)
            gpu = run_gpu(w, fused=fused, flags=fb.FLOWMM_FLAG_GENERIC_PATH)
            for l in range(w.n_layers):
                check_layer(oracle, w, gpu, l)
        gen = torch.Generator(device="cuda:0").manual_seed(3)
        K = torch.randn((2, 2, L, d), generator=gen, device="cuda:0").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
        Q = torch.randn((2, 4, L, d), generator=gen, device="cuda:0").to(K.dtype)
        bufs = fb.DeviceBuffers(fb.Params.from_workload(w))
        bufs.flow_exact(K.repeat(1, 1, n, 1), Q.repeat(1, 1, n, 1), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        rho.append(bufs.rho.cpu().numpy())
    # sums of at most L weights in another order: each is right to 1e-5 (test_flow_exact_at_tile_edges)
    assert np.allclose(rho[1], rho[0], rtol=2e-5, atol=0)


@pytest.mark.parametrize("layers,L,dtype,d", [(65, 200, "bf16", 64), (64, 200, "bf16", 64), (65, 769, "bf16", 64), (65, 768, "bf16", 128), (65, 130, "f32", 128)])
def test_unit_merge_by_units_and_lengths(oracle, layers, L, dtype, d):
    """512 and 520 units and lengths around 768, where the match and merge workgroups change their size, in both strategies and entry points."""
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, run_gpu
    w = wl.make_workload("units", dtype, L, layers, 8, 8, d, 16, [[L // 5, L // 2, L - L // 5 - L // 2]], [20])
    for theta, fused in ((-1.0, True), (2.0, True), (2.0, False)):
        print(f"layers {layers} L {L} {dtype} d {d} theta {theta} fused {fused}", flush=True)
        gpu = run_gpu(w, theta=theta, fused=fused)
        for l in (0, layers - 1):
            check_layer(oracle, w, gpu, l, theta=theta)


@pytest.mark.parametrize("layers,L,pct,dtype,d", [(72, 769, 10, "bf16", 64), (73, 769, 10, "bf16", 64), (80, 1024, 10, "bf16", 128), (128, 961, 10, "bf16", 64), (80, 800, 17, "bf16", 64),
                                                  (192, 800, 10, "bf16", 64), (80, 900, 10, "f32", 64)])
def test_unit_merge_of_long_equal_sequences(oracle, layers, L, pct, dtype, d):
    """576 to 1536 units of more than 768 tokens with few or many pivots, where the match and merge workgroups change their size, in both strategies and entry points."""
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, run_gpu
    w = wl.make_workload("units", dtype, L, layers, 8, 8, d, 16, [[L // 5, L // 2, L - L // 5 - L // 2]], [pct])
    for theta, fused in ((-1.0, False), (2.0, True)):
        print(f"layers {layers} L {L} {pct} % {dtype} d {d} theta {theta} fused {fused}", flush=True)
        gpu = run_gpu(w, theta=theta, fused=fused)
        for l in (0, layers - 1):
            check_layer(oracle, w, gpu, l, theta=theta, kv_heads=[0, 7])


@pytest.mark.parametrize("layers,L,d,W", [(32, 300, 64, 16), (33, 300, 64, 16), (33, 384, 64, 16), (33, 250, 64, 16), (33, 300, 64, 48), (64, 250, 128, 16), (63, 250, 128, 16), (128, 100, 128, 16),
                                          (64, 300, 128, 16), (64, 250, 128, 40)])
def test_unit_path_f32_by_units_and_key_tiles(oracle, layers, L, d, W):
    """Both sides of the bounds between keys split into bf16 terms and the fp32 instructions, in both strategies and entry points."""
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, launched, run_gpu
    w = wl.make_workload("units", "f32", L, layers, 8, 8, d, W, [[L // 5, L // 2, L - L // 5 - L // 2]], [50])
    for theta, fused in ((-1.0, True), (2.0, False)):
        print(f"layers {layers} L {L} d {d} W {W} theta {theta} fused {fused}", flush=True)
        with launched() as kernels:
            gpu = run_gpu(w, theta=theta, fused=fused)
        assert "unit_plan" in kernels, kernels
        for l in (0, layers - 1):
            check_layer(oracle, w, gpu, l, theta=theta, kv_heads=[0, 7])


UNIT_MERGE_EDGES = {  # lengths, q heads, kv heads, layers, head_dim, window, budgets in %, dtype, FLOWMM_FLAG_*, one launch
    "half_the_chip": ([900], 28, 4, 32, 128, 32, [5], "bf16", 0, True),
    "below_half": ([900], 28, 4, 31, 128, 32, [5], "bf16", 0, False),
    "unequal": ([1024, 130, 513, 65], 12, 4, 8, 64, 32, [20, 50, 5, 60], "bf16", 0, True),
    "weighted": ([700, 90], 12, 4, 16, 128, 32, [40, 40], "bf16", 4, True),
    "no_tokens_evicted": ([64, 300], 12, 4, 16, 64, 32, [100, 10], "bf16", 0, True),
    "longer": ([1025], 24, 8, 24, 64, 32, [20], "bf16", 0, True),
    "longer_on_few": ([1025], 24, 8, 23, 64, 32, [20], "bf16", 0, False),
    "longer_on_more": ([1025], 24, 8, 33, 64, 32, [20], "bf16", 0, False),
    "longest": ([2048], 24, 8, 32, 128, 32, [25], "bf16", 0, True),
    "longer_unequal": ([1025, 1024], 24, 8, 12, 64, 32, [20, 20], "bf16", 0, False),
    "beyond": ([2049], 24, 8, 24, 64, 32, [20], "bf16", 0, False),
    "too_many_pivots": ([900], 28, 4, 32, 64, 32, [57], "bf16", 0, False),
    "f32": ([600, 300], 12, 4, 16, 128, 32, [20, 20], "f32", 0, True),
}


@pytest.mark.parametrize("name", list(UNIT_MERGE_EDGES))
def test_generic_plans_merged_in_one_launch(oracle, name):
    """Plans of the generic kernels that one workgroup per unit merges, on either side of every bound, both entry points against the oracle."""
    from paper_2511_05534_amd import binding as fb, workloads as wl
    from parity_utils import check_layer, launched, run_gpu
    lens, Hq, Hkv, layers, d, W, pcts, dtype, extra, one = UNIT_MERGE_EDGES[name]
    w = wl.make_workload("merged", dtype, sum(lens), layers, Hq, Hkv, d, W, [[L // 5, L // 2, L - L // 5 - L // 2] for L in lens], pcts)
    flags = fb.FLOWMM_FLAG_GENERIC_PATH | extra
    got = []
    for fused in (True, False):
        print(f"{name} fused {fused}", flush=True)
        with launched() as kernels:
            gpu = run_gpu(w, fused=fused, flags=flags)
        assert ("unit_merge" in kernels) == one and ("merge_tasks" in kernels) != one, kernels
        for l in (0, layers - 1):
            check_layer(oracle, w, gpu, l, flags=flags)
        got.append(gpu)
    for field in got[0]:
        assert np.array_equal(got[0][field], got[1][field]), field


UNEQUAL_SCORES = {  # lengths, q heads, kv heads, head_dim, window, layers, one workgroup per unit
    "32_rows_many_idle": ([1000] + [150] * 8, 32, 32, 128, 32, 1, False),
    "32_rows_some_idle": ([1000, 300, 900, 200, 600, 300, 1000, 150, 400], 32, 32, 128, 32, 1, True),
    "32_rows_many_units_some_idle": ([1000, 200, 200, 400, 200, 300, 600, 150, 100], 32, 32, 128, 32, 2, True),
    "64_rows_of_64_channels": ([1000] + [150] * 8, 16, 4, 64, 16, 4, True),
    "64_rows_of_64_channels_many_units": ([1000] + [150] * 8, 16, 4, 64, 16, 16, False),
    "128_rows": ([1000, 300, 900, 200, 600, 300, 1000, 150, 400], 32, 8, 128, 32, 2, False),
}


@pytest.mark.parametrize("name", list(UNEQUAL_SCORES))
def test_score_of_unequal_sequences_by_rows_and_units(oracle, name):
    """The bounds between the score kernel that keeps a unit's keys and the streaming ones where shorter sequences leave waves without keys."""
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, launched, run_gpu
    lens, Hq, Hkv, d, W, layers, resident = UNEQUAL_SCORES[name]
    print(name, flush=True)
    w = wl.make_workload("unequal", "bf16", sum(lens), layers, Hq, Hkv, d, W, [[L // 5, L // 2, L - L // 5 - L // 2] for L in lens], [10] * len(lens))
    with launched() as kernels:
        gpu = run_gpu(w, fused=True)
    assert ("score_resident" in kernels) == resident and "unit_plan" not in kernels, kernels
    check_layer(oracle, w, gpu, layers - 1, kv_heads=[0, Hkv - 1])


def test_workspace_between_the_score_kernels():
    """224 query rows a little above 64 MiB: streamed with the workspace that flowmm_plan_sizes asks for, by the resident kernel with 64 MiB, both alike, and refused with
    less than either takes; a re-merge of such a cache the same."""
    import torch
    from parity_utils import launched
    fb = _fb()
    Lyr, Hq, Hkv, d, W, L, B = 136, 28, 4, 128, 32, 900, 90
    gen = torch.Generator(device="cuda:0").manual_seed(31)
    K, V = (torch.randn((Lyr, Hkv, L, d), generator=gen, device="cuda:0").bfloat16() for _ in range(2))
    Q = torch.randn((Lyr, Hq, W, d), generator=gen, device="cuda:0").bfloat16()
    params = fb.Params(Lyr, Hq, Hkv, d, "bf16", [L], [B], [[(0, 300, 1), (300, L, 0)]], W, -1.0, [1e9])
    bufs = fb.DeviceBuffers(params)
    asked, stream, results = bufs.workspace_bytes, torch.cuda.current_stream().cuda_stream, []
    assert asked > 64 << 20
    for size, kernel in ((asked, "score_stats"), (64 << 20, "score_resident")):
        bufs.workspace_bytes = size
        with launched() as kernels:
            bufs.plan_merge(K, V, Q, stream)
            torch.cuda.synchronize()
        assert kernel in kernels, (size, kernels)
        results.append((bufs.importance.clone(), bufs.rho.clone()))
    bufs.workspace_bytes = 48 << 20
    with pytest.raises(fb.FlowMMError) as ei:
        bufs.plan_merge(K, V, Q, stream)
    assert ei.value.status == fb.FLOWMM_EWORKSPACE and str(asked) in ei.value.message
    # weights of up to 900 keys summed over 224 rows in another order, their logits' and constants' fp32 rounding
    assert torch.allclose(results[0][0], results[1][0], rtol=1e-4, atol=1e-9) and torch.allclose(results[0][1], results[1][1], rtol=1e-4, atol=1e-9)
    cap = fb.Params(Lyr, Hq, Hkv, d, "bf16", [L], [B], [[(0, L, 0)]], W, -1.0, [1e9], q_strides=(Hq * W * d, W * d, d))
    sizes, ws = fb.flowmm_cache_remerge_sizes(cap, [0, L], 0, L)
    rows = 2 * Lyr * Hkv * B * d * 2
    space = torch.empty(ws, dtype=torch.uint8, device="cuda:0")
    for size, kernel in ((ws, "score_stats"), ((64 << 20) + rows, "score_resident")):
        Kc, Vc = K.clone(), V.clone()
        assert size <= ws
        with launched() as kernels:
            fb.flowmm_cache_remerge(cap, [0, L], [L], 0, Kc.data_ptr(), Vc.data_ptr(), Q.data_ptr(), bufs.plan_ptrs, space.data_ptr(), size, stream)
            torch.cuda.synchronize()
        assert kernel in kernels, (size, kernels)


_EXACT_SCALE = float(np.float32(0.125 / 1.4426950408889634))  # times log2(e), as the kernels take it: 2^-3


def _extreme_case(d, Hq, dtype, Lq, L, gen):
    """Queries and keys of one kv head with extreme logits: those of head 0 overflow to -inf, those of head 1 are finite and far below
    -1e30, key 5's half as far as the others', which are equal; the other heads' are ordinary.  With _EXACT_SCALE a logit is an exact
    multiple of its product, so that equal ones are equal after rounding too."""
    import torch
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K = torch.randn((1, 1, L, d), generator=gen, device="cuda:0")
    Q = torch.randn((1, Hq, Lq, d), generator=gen, device="cuda:0")
    K[..., 0] = -2.0 ** 60
    K[:, :, 5, 0] = -2.0 ** 59
    Q[..., 0] = 0.0
    Q[:, 0, :, 0], Q[:, 1, :, 0] = 3e38, 2.0 ** 50
    return K.to(tdt), Q.to(tdt)


def _extreme_weights(Q, K, h, first):
    """Attention of query rows at positions first, first + 1, .. in 64 bits."""
    n, L = Q.shape[0], K.shape[0]
    s = _EXACT_SCALE * (Q[:, 1:] @ K[:, 1:].T)
    if h == 1:
        s[:], s[:, 5] = 0.0, 1e6  # channel 0 is 2^100 times larger than what is left out here
    s[np.arange(L)[None, :] > first + np.arange(n)[:, None]] = -np.inf
    p = np.exp(s - s.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    return 0.0 * p if h == 0 else p


@pytest.mark.parametrize("d,W,image_window,dtype", [(64, 32, False, "bf16"), (64, 32, True, "bf16"), (128, 64, True, "bf16"), (128, 64, False, "bf16")])
def test_score_of_very_negative_logits(d, W, image_window, dtype):
    """A window row whose logits are all -inf weighs nothing and leaves the flow ratio a number; one whose logits are finite and
    far below all others is a row like any other."""
    import torch
    fb = _fb()
    L, Hq = 1100, 4
    print(f"d {d} W {W} image_window {image_window} {dtype}", flush=True)
    tail = W // 2 if image_window else W
    img = np.zeros(L, bool)
    img[300:L - tail] = True
    K, Q = _extreme_case(d, Hq, dtype, W, L, torch.Generator(device="cuda:0").manual_seed(8))
    params = fb.Params(1, Hq, 1, d, dtype, [L], [W + 8], [[(0, 300, 0), (300, L - tail, 1), (L - tail, L, 0)]], W, 0.25, [1.0],
                       scale=_EXACT_SCALE, flags=fb.FLOWMM_FLAG_GENERIC_PATH)
    bufs = fb.DeviceBuffers(params)
    bufs.plan(K, Q, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    Kn, Qn = K[0, 0].double().cpu().numpy(), Q[0].double().cpu().numpy()
    p = [_extreme_weights(Qn[h], Kn, h, L - W) for h in range(Hq)]
    want = sum(x.sum(axis=0) for x in p) / (Hq * W)
    cross = sum((x * (img[L - W:, None] != img[None, :])).sum() for x in p) / W / Hq
    # as for the ordinary logits: a weight carries the fp32 rounding of its logit, of its row's constant and of exp2
    assert np.allclose(bufs.importance[0, 0].cpu().numpy(), want, rtol=1e-5, atol=1e-9)
    assert abs(float(bufs.rho[0, 0]) - cross) <= 1e-5 * cross, (float(bufs.rho[0, 0]), cross)


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "f32"), (128, "f32")])
def test_flow_exact_of_very_negative_logits(d, dtype):
    import torch
    fb = _fb()
    L, Hq = 300, 3
    print(f"d {d} {dtype}", flush=True)
    img = np.zeros(L, bool)
    img[50:250] = True
    K, Q = _extreme_case(d, Hq, dtype, L, L, torch.Generator(device="cuda:0").manual_seed(9))
    params = fb.Params(1, Hq, 1, d, dtype, [L], [1], [[(0, 50, 0), (50, 250, 1), (250, L, 0)]], 1, 0.25, [1.0], scale=_EXACT_SCALE)
    bufs = fb.DeviceBuffers(params)
    bufs.flow_exact(K, Q, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    Kn, Qn = K[0, 0].double().cpu().numpy(), Q[0].double().cpu().numpy()
    want = sum((_extreme_weights(Qn[h], Kn, h, 0) * (img[:, None] != img[None, :])).sum() for h in range(Hq)) / L / Hq
    assert abs(float(bufs.rho[0, 0]) - want) <= 1e-5 * want, (float(bufs.rho[0, 0]), want)


F32_MAGNITUDES = {  # tokens, pivots, kv heads, layers, head_dim, generic kernels, a kernel that runs
    "unit_d64": (300, 60, 2, 2, 64, False, "unit_plan"),
    "unit_d128": (300, 60, 2, 2, 128, False, "unit_plan"),
    "unit_many_units_d64": (200, 60, 16, 33, 64, False, "unit_plan"),
    "unit_many_units_d128": (200, 60, 16, 33, 128, False, "unit_plan"),
    "resident_eight_d64": (300, 60, 2, 2, 64, True, "score_resident"),
    "resident_eight_d128": (250, 60, 2, 2, 128, True, "score_resident"),
    "resident_sixteen_d64": (400, 60, 2, 2, 64, True, "score_resident"),
    "resident_sixteen_d128": (400, 60, 66, 2, 128, True, "score_resident"),
    "three_kernels_d64": (700, 70, 2, 2, 64, True, "score_stats"),
    "three_kernels_d128": (700, 70, 2, 2, 128, True, "score_stats"),
    "select_match_d64": (300, 90, 2, 2, 64, True, "select_match"),
    "select_match_d128": (300, 90, 2, 2, 128, True, "select_match"),
    "match_d64": (900, 200, 2, 2, 64, True, "match"),
    "match_d128": (900, 200, 2, 2, 128, True, "match"),
}


@pytest.mark.parametrize("theta", [-1.0, 2.0])
@pytest.mark.parametrize("name", list(F32_MAGNITUDES))
def test_f32_rows_of_extreme_magnitude(name, theta):
    """Numbers that three bf16 terms do not hold, where every product and sum is a finite fp32 number: importances, flow ratio, pivots and slots against 64 bits.
    Channel 0: one kept row beyond the largest bf16 against zeros.  1 and 2: a token whose product with either of two pivots is finite and the product of its
    leading terms is not; the later pivot is the closer one.  3: a logit of that kind.
    Intra-modal layers of the unit path, which compare plain numbers: rows far below 2^-110 find their pivots."""
    import torch
    from parity_utils import launched
    fb = _fb()
    L, B, Hkv, Lyr, d, generic, kernel = F32_MAGNITUDES[name]
    W, big = 16, float(np.float32(1.84108e19))  # leads with 2^64 and has a finite square
    print(f"{name} theta {theta}", flush=True)
    gen = torch.Generator().manual_seed(17)
    K = torch.randn((Lyr, Hkv, L, d), generator=gen)
    Q = torch.randn((Lyr, Hkv, W, d), generator=gen)
    V = torch.randn(K.shape, generator=gen)
    K[..., :4] = 0.0
    Q[..., :4] = 0.0
    tok, first, second, hot = 20, L - 9, L - 7, 30
    K[:, :, L - 3, 0] = 3.4e38
    K[:, :, [tok, first, second]] = 0.0
    K[:, :, [tok, first, second], 1] = big
    K[:, :, [tok, second], 2] = 1.1e18
    K[:, :, hot, 3] = big
    Q[:, :, :3, 3] = big
    tiny = list(range(40, 60)) if theta > 0 and not generic else []
    K[:, :, tiny] *= 2.0 ** -133
    K[:, :, L // 2:L // 2 + B, 5] += 6.0  # what the window looks at (none of the rows above but the hot one)
    Q[..., 5] = 4.0
    K[:, :, :L // 2, 5] = torch.where(K[:, :, :L // 2, 5].abs() > 1e-20, torch.tensor(-3.0), K[:, :, :L // 2, 5])
    img = np.zeros(L, bool)
    img[70:L - W - 20] = True
    params = fb.Params(Lyr, Hkv, Hkv, d, "f32", [L], [B], [[(0, 70, 0), (70, L - W - 20, 1), (L - W - 20, L, 0)]], W, theta, [1e9], scale=_EXACT_SCALE,
                       flags=fb.FLOWMM_FLAG_GENERIC_PATH if generic else 0)
    bufs = fb.DeviceBuffers(params)
    stream = torch.cuda.current_stream().cuda_stream
    dev = [t.to("cuda:0") for t in (K, V, Q)]
    with launched() as kernels:
        bufs.plan_merge(*dev, stream)
        torch.cuda.synchronize()
    assert kernel in kernels, kernels
    seen = np.tril(np.ones((W, L), bool), L - W)
    for l in (0, Lyr - 1):
        cross = 0.0
        for g in range(Hkv):
            Kn, Qn = K[l, g].double().numpy(), Q[l, g].double().numpy()
            logits = np.where(seen, Qn @ Kn.T / 8.0, -np.inf)  # in powers of two
            p = np.exp2(logits - logits.max(axis=1, keepdims=True))
            p /= p.sum(axis=1, keepdims=True)
            cross += (p * (img[L - W:, None] != img[None, :])).sum() / W / Hkv
            imp = bufs.importance[l, g].cpu().numpy()
            # (the rounding of logits of up to a few hundred, of the row's constant and of exp2)
            assert np.allclose(imp, p.sum(axis=0) / W, rtol=1e-4, atol=1e-9), (l, g)
            kept = bufs.kept_idx.cpu().numpy().reshape(Lyr, Hkv, B)[l, g]
            assign = bufs.assign.cpu().numpy().reshape(Lyr, Hkv, L)[l, g]
            assert set(range(L - W, L)) | {hot} <= set(kept) and not {tok, *tiny} & set(kept)
            norm = np.linalg.norm(Kn, axis=1)
            u = Kn @ Kn[kept].T / np.maximum(norm[:, None], 1e-300) / norm[kept]
            if theta > 0:
                u[img[:, None] != img[kept][None, :]] = -np.inf
            assert kept[assign[tok]] == second, (l, g, kept[assign[tok]])
            for i in sorted(set(range(L)) - set(kept)):
                best = u[i].max()
                assert assign[i] >= 0 and (best < 1e-15 or best - u[i, assign[i]] <= 1e-3 * best), (l, g, i)
        assert abs(float(bufs.rho[l, 0]) - cross) <= 1e-4 * cross + 1e-9, (l, float(bufs.rho[l, 0]), cross)
    assert bool(torch.isfinite(bufs.K_out).all()) and bool(torch.isfinite(bufs.V_out).all())


@pytest.mark.parametrize("name,L,d,generic,kernel", [("unit", 300, 64, False, "unit_plan"), ("unit", 300, 128, False, "unit_plan"), ("resident", 250, 64, True, "score_resident"),
                                                     ("resident", 250, 128, True, "score_resident"), ("tiles", 700, 64, True, "score_stats"), ("tiles", 700, 128, True, "score_stats")])
def test_f32_products_keep_all_terms(name, L, d, generic, kernel):
    """Logits of one window row, read back from its weights: off from 64 bits by the rounding of fp32 sums and no more.
    Root mean square, for logits of spread 12: the sum of the products 2e-7 of that, the weight's exponent (below 2^7) rounded 2^-18 / sqrt(3) at the most: 4.6e-6
    together, twice that allowed.  Without the third terms the products alone would be off by 2^-18 of themselves, 4.6e-5."""
    import torch
    from parity_utils import launched
    fb = _fb()
    print(f"{name} L {L} d {d}", flush=True)
    gen = torch.Generator().manual_seed(29)
    K = torch.randn((1, 2, L, d), generator=gen)
    Q = torch.randn((1, 2, 1, d), generator=gen) * (12.0 * 8.0 / d ** 0.5)
    params = fb.Params(1, 2, 2, d, "f32", [L], [32], [[(0, L, 0)]], 1, 0.25, [1e9], scale=_EXACT_SCALE, flags=fb.FLOWMM_FLAG_GENERIC_PATH if generic else 0)
    bufs = fb.DeviceBuffers(params)
    with launched() as kernels:
        bufs.plan(K.to("cuda:0"), Q.to("cuda:0"), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    assert kernel in kernels, kernels
    for g in range(2):
        logits = K[0, g].double().numpy() @ Q[0, g, 0].double().numpy() / 8.0  # in powers of two
        got = np.log2(bufs.importance[0, g].double().cpu().numpy())
        err = got - logits
        err -= np.median(err)  # (the row's constant)
        assert np.sqrt((err ** 2).mean()) <= 9.2e-6, np.sqrt((err ** 2).mean())


@pytest.mark.parametrize("L,B,dtype,d,Lyr", [(700, 400, "bf16", 128, 16), (3000, 2500, "bf16", 128, 16), (640, 500, "bf16", 64, 16), (400, 320, "f32", 128, 16),
                                             (700, 256, "bf16", 128, 2), (600, 500, "bf16", 128, 8)])
def test_remerge_in_place_in_a_token_major_cache(L, B, dtype, d, Lyr):
    """The middle sequence of a cache stored [T][kv heads][d], at the units and budgets where the merge goes into place: its rows
    against flowmm_plan_merge of a copy of them, everything else as it was."""
    import torch
    fb = _fb()
    print(f"L {L} B {B} {dtype} d {d} layers {Lyr}", flush=True)
    W, Hq, Hkv = 20, 8, 4
    cap = [50, L + 7, 33]
    cu = [0, 50, 57 + L, 90 + L]
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda:0").manual_seed(7)
    Kc, Vc = (torch.randn((Lyr, cu[-1], Hkv, d), generator=gen, device="cuda:0").to(tdt) for _ in range(2))
    Kc[:, 60:60 + L // 2] = (0.9 * Kc[:, 100:101].float() + 0.3 * Kc[:, 60:60 + L // 2].float()).to(tdt)  # many tokens resemble one
    Q = torch.randn((Lyr, Hq, W, d), generator=gen, device="cuda:0").to(tdt)
    K, V = (t[:, 50:50 + L].permute(0, 2, 1, 3).contiguous() for t in (Kc, Vc))
    stream = torch.cuda.current_stream().cuda_stream
    beside = fb.DeviceBuffers(fb.Params(Lyr, Hq, Hkv, d, dtype, [L], [B], [[(0, L, 0)]], W, -1.0, [4.0 / B]))
    beside.plan_merge(K, V, Q, stream)
    params = fb.Params(Lyr, Hq, Hkv, d, dtype, cap, [20, B, 20], [[(0, n, 0)] for n in cap], W, 0.25, [1.0, 4.0 / B, 1.0],
                       k_strides=(cu[-1] * Hkv * d, d, Hkv * d), q_strides=(Hq * W * d, W * d, d))
    sizes, ws = fb.flowmm_cache_remerge_sizes(params, cu, 1, L)
    kinds = [torch.float32, torch.float32, torch.int32, torch.int32, torch.int32, torch.int32]
    plan = [torch.empty(s // 4, dtype=t, device="cuda:0") for s, t in zip(sizes, kinds)]
    K0, V0 = Kc.clone(), Vc.clone()
    space = torch.empty(ws, dtype=torch.uint8, device="cuda:0")
    fb.flowmm_cache_remerge(params, cu, [40, L, 33], 1, Kc.data_ptr(), Vc.data_ptr(), Q.data_ptr(), [t.data_ptr() for t in plan],
                            space.data_ptr(), ws, stream)
    torch.cuda.synchronize()
    assert torch.equal(plan[3].view_as(beside.kept_idx), beside.kept_idx) and torch.equal(plan[4].view_as(beside.assign), beside.assign)
    for got, before, want in ((Kc, K0, beside.K_out), (Vc, V0, beside.V_out)):
        assert torch.equal(got[:, :50], before[:, :50]) and torch.equal(got[:, 50 + B:], before[:, 50 + B:])
        # fp32 sums in another order (at most 3000 terms: 3000 x 2^-24 of the largest row), then one rounding to the data type
        a, b = got[:, 50:50 + B].permute(0, 2, 1, 3).double(), want.double()
        tol = 2.0 ** (-7 if dtype == "bf16" else -23) * b.abs() + 3000 * 2.0 ** -24 * before.double().abs().max()
        assert bool(((a - b).abs() <= tol).all())


IN_PLACE_PARTS = {  # rows, budget, dtype, head_dim, layers (four kv heads each), merged in place
    "whole_rows": (380, 300, "bf16", 128, 80, True),
    "two_parts": (1500, 1200, "bf16", 128, 16, True),
    "two_parts_to_fit": (3000, 2000, "bf16", 128, 16, True),
    "four_parts": (480, 400, "bf16", 128, 2, True),
    "four_parts_a_round_and_one_row": (700, 513, "bf16", 128, 2, True),
    "two_narrow_parts_d64": (480, 400, "bf16", 64, 2, True),
    "four_parts_f32": (900, 700, "f32", 128, 16, True),
    "two_parts_f32_of_long_slots": (1500, 900, "f32", 128, 16, True),
    "eight_parts_f32": (480, 400, "f32", 128, 2, True),
    "four_narrow_parts_f32_d64": (480, 400, "f32", 64, 2, True),
    "beside_few_units": (1900, 1500, "bf16", 128, 4, False),
    "beside_too_many_members": (3200, 1600, "bf16", 128, 16, False),
}


@pytest.mark.parametrize("name", list(IN_PLACE_PARTS))
def test_remerge_in_place_by_parts_of_the_rows(name):
    """The numbers of parts into which the in-place merge cuts the channels, and the sizes at which it gives way."""
    from parity_utils import launched
    *sizes, in_place = IN_PLACE_PARTS[name]
    with launched() as kernels:
        test_remerge_in_place_in_a_token_major_cache(*sizes)
    assert ("merge_in_place" in kernels) == in_place and ("cache_store_rows" in kernels) != in_place, kernels


@pytest.mark.parametrize("dtype,Lyr,B,n,parts", [("bf16", 2, 400, 2000, 4), ("bf16", 16, 400, 1119, 2), ("f32", 2, 300, 2000, 8)])
def test_remerge_in_place_of_one_long_slot(dtype, Lyr, B, n, parts):
    """All evicted rows in one slot, with values where one fp32 sum over all of them rounds up at every row: the mean of 64 bits, correctly rounded (bf16)
    or as near as sums of 128 rows come (fp32: 128 roundings, and one for each of them, of half an ulp)."""
    import torch
    from parity_utils import launched
    fb = _fb()
    Hkv, d, W, L = 4, 128, 16, B + n
    print(f"{dtype} layers {Lyr} rows {L} members {n}", flush=True)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    # pivots of 2^15 (1 + i / 128), members of 2^-9 (1 + j / 128): what is added is more than half an ulp of the sum and counts as one
    i, j = (a.ravel() for a in np.meshgrid(np.arange(128), np.arange(1, 100), indexing="ij"))
    pivot, member = 2.0 ** 15 * (1 + i / 128), 2.0 ** -9 * (1 + j / 128)
    mean = (pivot + n * member) / (n + 1)
    chain = (pivot + n * 2.0 ** -8) / (n + 1)
    slack = (128 + n / 128 + 2) * 2.0 ** -24  # relative: half an ulp of the sum for a sum of 128 rows, for each of the sums and for the quotient
    rounded = lambda x: torch.tensor(x, dtype=torch.float64).to(tdt).double().numpy()
    shows = np.flatnonzero((rounded(mean) != rounded(chain)) & ((rounded(mean * (1 + slack)) == rounded(mean)) | (dtype == "f32")))
    assert len(shows) >= d
    pick = shows[np.linspace(0, len(shows) - 1, d).astype(int)]
    gen = torch.Generator(device="cuda:0").manual_seed(23)
    K = torch.randn((Lyr, Hkv, L, d), generator=gen, device="cuda:0")
    V = torch.randn((Lyr, Hkv, L, d), generator=gen, device="cuda:0")
    Q = torch.randn((Lyr, Hkv, W, d), generator=gen, device="cuda:0")
    order = torch.randperm(L - W, generator=gen, device="cuda:0")
    kept, evicted = order[:B - W], order[B - W:]
    Q[..., 0] = 8.0
    K[..., 0] = 0.0
    K[:, :, kept, 0] = 16.0
    first = int(kept[0])
    K[:, :, evicted] = 0.125 * K[:, :, first:first + 1]
    K[:, :, evicted, 0] = 0.0  # (closer to their model than to the others all the same: 3 in 4 of its square are in the other channels)
    K[:, :, kept, 0] = 6.0
    V[:, :, first] = torch.from_numpy(pivot[pick]).to("cuda:0", torch.float32)
    V[:, :, evicted] = torch.from_numpy(member[pick]).to("cuda:0", torch.float32)
    K, V, Q = K.to(tdt), V.to(tdt), Q.to(tdt)
    params = fb.Params(Lyr, Hkv, Hkv, d, dtype, [L], [B], [[(0, L, 0)]], W, 0.25, [1e9], q_strides=(Hkv * W * d, W * d, d))
    sizes, ws = fb.flowmm_cache_remerge_sizes(params, [0, L], 0, L)
    kinds = [torch.float32, torch.float32, torch.int32, torch.int32, torch.int32, torch.int32]
    plan = [torch.empty(s // 4, dtype=t, device="cuda:0") for s, t in zip(sizes, kinds)]
    space = torch.empty(ws, dtype=torch.uint8, device="cuda:0")
    with launched() as kernels:
        fb.flowmm_cache_remerge(params, [0, L], [L], 0, K.data_ptr(), V.data_ptr(), Q.data_ptr(), [t.data_ptr() for t in plan], space.data_ptr(), ws,
                                torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    assert "merge_in_place" in kernels, kernels
    kept_idx, assign = plan[3].view(Lyr, Hkv, B).cpu().numpy(), plan[4].view(Lyr, Hkv, L).cpu().numpy()
    for l in range(Lyr):
        for g in range(Hkv):
            slot = int(np.flatnonzero(kept_idx[l, g] == first)[0])
            assert int((assign[l, g] == slot).sum()) == n + 1, (l, g)
            got = V[l, g, slot].double().cpu().numpy()
            if dtype == "bf16":
                assert (got == rounded(mean[pick])).all(), (l, g)
            else:
                assert (np.abs(got - mean[pick]) <= slack * mean[pick]).all(), (l, g)


LAYOUT_CASES = {  # lengths, q heads, kv heads, head_dim, window, dtype, layers
    "resident_eight": ([70, 512, 321], 6, 2, 128, 20, "bf16", 2),
    "resident_sixteen": ([1024, 800], 34, 34, 64, 32, "bf16", 2),
    "streamed": ([1281, 130, 700], 14, 2, 128, 32, "bf16", 2),
    "three_kernels": ([1281, 130, 700], 10, 2, 128, 32, "bf16", 2),
    "f32": ([700, 257], 4, 2, 128, 16, "f32", 2),
    "f32_unit": ([300, 257], 2, 2, 64, 16, "f32", 2),
}


@pytest.mark.parametrize("name", list(LAYOUT_CASES))
def test_token_major_layout_at_every_score_kernel(name):
    """A cache stored [T][kv heads][d] gives bit for bit what the dense one gives, whichever kernels serve the shape."""
    import torch
    fb = _fb()
    lens, Hq, Hkv, d, W, dtype, Lyr = LAYOUT_CASES[name]
    print(f"case {name}", flush=True)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    T, n = sum(lens), len(lens)
    spans = [[(0, L // 3, 0), (L // 3, L - W // 2, 1), (L - W // 2, L, 0)] for L in lens]
    budgets = [max(W, L // 5) for L in lens]
    flags = 0 if name == "f32_unit" else fb.FLOWMM_FLAG_GENERIC_PATH
    gen = torch.Generator(device="cuda:0").manual_seed(11)
    K, V = (torch.randn((Lyr, Hkv, T, d), generator=gen, device="cuda:0").to(tdt) for _ in range(2))
    Q, Qf = (torch.randn((Lyr, Hq, m, d), generator=gen, device="cuda:0").to(tdt) for m in (n * W, T))
    results = []
    for dense in (True, False):
        params = fb.Params(Lyr, Hq, Hkv, d, dtype, lens, budgets, spans, W, 0.25, [1.0] * n, flags=flags,
                           k_strides=None if dense else (T * Hkv * d, d, Hkv * d))
        Ks, Vs = (K, V) if dense else (t.permute(0, 2, 1, 3).contiguous() for t in (K, V))
        bufs = fb.DeviceBuffers(params)
        stream = torch.cuda.current_stream().cuda_stream
        bufs.plan_merge(Ks, Vs, Q, stream)
        out = [getattr(bufs, f).clone() for f in fb.PLAN_FIELDS] + [bufs.K_out.clone(), bufs.V_out.clone()]
        bufs.flow_exact(Ks, Qf, stream)
        torch.cuda.synchronize()
        results.append(out + [bufs.rho.clone()])
    for a, b in zip(*results):
        assert torch.equal(a, b)


SELECT_MATCH_EDGES = {  # lengths, budgets, q heads, kv heads, head_dim, window, dtype, tau (None: the usual gate)
    "one_token": ([97], [96], 2, 2, 128, 32, "bf16", None),
    "groups_of_tokens": ([96, 97, 65], [64, 64, 34], 4, 2, 128, 32, "bf16", None),
    "a_round_and_one_more": ([576, 577, 575], [64, 64, 64], 4, 2, 64, 32, "bf16", None),
    "tiles_of_pivots": ([300, 301, 500], [128, 129, 257], 4, 2, 128, 20, "bf16", None),
    "many_pivots": ([1060], [1000], 4, 1, 64, 33, "bf16", None),
    "last_of_the_range": ([1100, 1124], [76, 100], 6, 2, 128, 16, "bf16", None),
    "beyond_the_range": ([1125], [100], 6, 2, 128, 16, "bf16", None),
    "no_eligible_pivot": ([200, 700], [50, 90], 2, 1, 128, 16, "bf16", -1.0),
    "all_kept": ([64, 200], [64, 40], 2, 1, 64, 16, "bf16", 1.0),
    "f32": ([100, 333], [60, 64], 4, 2, 64, 16, "f32", None),
    "f32_wide": ([100, 333], [60, 64], 2, 2, 128, 16, "f32", None),
}


@pytest.mark.parametrize("name", list(SELECT_MATCH_EDGES))
def test_split_and_match_in_one_workgroup(oracle, name):
    """Short sequences through the generic kernels, in both strategies and entry points, stage by stage against the oracle."""
    from paper_2511_05534_amd import binding as fb, workloads as wl
    from parity_utils import check_layer, run_gpu
    lens, budgets, Hq, Hkv, d, W, dtype, tau = SELECT_MATCH_EDGES[name]
    spans = [[L // 5, L // 3, L - L // 5 - L // 3 - W // 2, W // 2] for L in lens]
    w = wl.make_workload("short", dtype, sum(lens), 3, Hq, Hkv, d, W, spans, [10] * len(lens), budgets=budgets)
    assert w.seqlens == lens and w.budgets == budgets
    tau = None if tau is None else [tau] * len(lens)
    for theta in (-1.0, 2.0):
        plans = []
        for fused in (True, False):
            print(f"{name} theta {theta} fused {fused}", flush=True)
            gpu = run_gpu(w, theta=theta, tau=tau, fused=fused, flags=fb.FLOWMM_FLAG_GENERIC_PATH)
            for l in range(w.n_layers):
                check_layer(oracle, w, gpu, l, theta=theta, tau=tau)
            plans.append(gpu)
        for field in plans[0]:
            assert np.array_equal(plans[0][field], plans[1][field]), field


@pytest.mark.parametrize("name", list(SELECT_MATCH_EDGES))
def test_split_and_match_edges_take_the_kernel_they_are_for(name):
    from paper_2511_05534_amd import binding as fb, workloads as wl
    from parity_utils import launched, run_gpu
    lens, budgets, Hq, Hkv, d, W, dtype, _ = SELECT_MATCH_EDGES[name]
    w = wl.make_workload("short", dtype, sum(lens), 3, Hq, Hkv, d, W, [[L] for L in lens], [10] * len(lens), budgets=budgets)
    with launched() as kernels:
        run_gpu(w, fused=True, flags=fb.FLOWMM_FLAG_GENERIC_PATH)
    one = name != "beyond_the_range"
    assert ("select_match" in kernels) == one and ("match" in kernels) != one, kernels


NEAR_TIES = {  # dtype, head_dim, tokens to be matched, pivots, how the pivots' keys resemble each other
    "bf16": ("bf16", 128, 900, 232, "scaled"),
    "bf16_d64": ("bf16", 64, 900, 300, "scaled"),
    "f32": ("f32", 128, 200, 140, "scaled"),
    "f32_d64": ("f32", 64, 230, 130, "scaled"),
    "bf16_other_order": ("bf16", 128, 900, 232, "permuted"),
    "bf16_d64_other_order": ("bf16", 64, 900, 300, "permuted"),
    "f32_other_order": ("f32", 128, 200, 140, "permuted"),
    "f32_d64_other_order": ("f32", 64, 230, 130, "permuted"),
}


@pytest.mark.parametrize("name", list(NEAR_TIES))
def test_near_ties_fall_alike_in_both_match_kernels(name):
    """Pivots whose cosines to a token are equal but for rounding (keys that are multiples of one another; keys of the same channels in
    another order): a sequence alone, which one workgroup splits and matches, and beside a long one, which takes it to the kernels of
    their own, gets the same pivots."""
    import torch
    from parity_utils import launched
    fb = _fb()
    dtype, d, E, B, how = NEAR_TIES[name]
    print(f"case {name}", flush=True)
    W, Hkv, Lyr, mate = 16, 2, 2, 4200
    L = E + B
    rng = np.random.default_rng(21)
    K = np.zeros((Lyr, Hkv, L, d))
    pivot = np.zeros(L, bool)
    pivot[L - W:] = True
    pivot[rng.permutation(L - W)[:B - W]] = True
    for l in range(Lyr):
        for g in range(Hkv):
            if how == "scaled":  # small integers: every product and sum of a cosine is exact, up to the norm
                base = rng.integers(-2, 3, (6, d))
                base[:, 0] = 4
                K[l, g, pivot] = base[rng.integers(0, 6, B)] * rng.integers(1, 32, B)[:, None]
                K[l, g, ~pivot] = rng.integers(-2, 3, (E, d))
            else:
                row, sign = rng.standard_normal(d), rng.choice([-1.0, 1.0], (4, d))
                K[l, g, pivot] = sign[rng.integers(0, 4, B)] * np.stack([np.abs(rng.permutation(row)) for _ in range(B)])
                K[l, g, pivot, 0] = 4.0
                K[l, g, ~pivot] = sign[rng.integers(0, 4, E)] * rng.uniform(0.5, 2.0, E)[:, None]
            K[l, g, ~pivot, 0] = 0.0  # the window queries see channel 0 only: the pivots stand out
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda:0").manual_seed(22)
    K = torch.from_numpy(K).to("cuda:0").to(tdt)
    long = torch.randn((Lyr, Hkv, mate, d), generator=gen, device="cuda:0").to(tdt)
    Q = torch.zeros((Lyr, Hkv, 2 * W, d), dtype=tdt, device="cuda:0")
    Q[..., 0] = 1.0
    results = []
    for alone in (True, False):
        lens, budgets = ([L], [B]) if alone else ([L, mate], [B, 64])
        n = len(lens)
        params = fb.Params(Lyr, Hkv, Hkv, d, dtype, lens, budgets, [[(0, m, 0)] for m in lens], W, -1.0, [1.0] * n, flags=fb.FLOWMM_FLAG_GENERIC_PATH)
        bufs = fb.DeviceBuffers(params)
        with launched() as kernels:
            bufs.plan(K if alone else torch.cat([K, long], 2).contiguous(), Q[:, :, :n * W].contiguous(), torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
        assert ({"select_match"} if alone else {"select", "match"}) <= kernels and ("select_match" in kernels) == alone, kernels
        results.append((bufs.kept_idx[:, :, :B].cpu().numpy(), bufs.assign[:, :, :L].cpu().numpy()))
    assert (results[0][0] == np.flatnonzero(pivot)).all() and (results[1][0] == results[0][0]).all()
    differ = (results[0][1] != results[1][1]).sum()
    assert differ == 0, f"{differ} of {Lyr * Hkv * E} tokens"


SELECT_MATCH_ROUTES = {  # tokens to be matched, pivots, units, dtype, and whether one workgroup splits and matches
    "few_units": (1024, 292, 8, "bf16", True), "few_units_many_candidates": (1024, 293, 8, "bf16", False), "more_than_1024_on_few_units": (1025, 64, 152, "bf16", False),
    "units_from_96_on": (1024, 900, 96, "bf16", True), "up_to_2048_from_160_units_on": (2048, 64, 160, "bf16", True), "more_than_2048": (2049, 64, 160, "bf16", False),
    "up_to_2048_at_512_units": (1025, 40, 512, "bf16", True), "more_units": (1025, 40, 520, "bf16", False), "longest": (600, 3496, 104, "bf16", True),
    "longer": (600, 3497, 104, "bf16", False), "f32": (500, 60, 8, "f32", True), "f32_many_candidates": (500, 61, 8, "f32", False),
    "f32_many_tokens": (513, 40, 8, "f32", False),
}


@pytest.mark.parametrize("name", list(SELECT_MATCH_ROUTES))
def test_routes_of_split_and_match(oracle, name):
    """Both sides of every bound of the rule that sends short sequences to one workgroup: the kernels that run, and the first and the last layer's results."""
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, launched, run_gpu
    E, B, units, dtype, one = SELECT_MATCH_ROUTES[name]
    L = E + B
    w = wl.make_workload("route", dtype, 17, units // 8, 8, 8, 64, 16, [[L // 5, L // 3, L - L // 5 - L // 3]], [10], budgets=[B])
    assert w.seqlens == [L] and w.budgets == [B]
    for fused in (True, False):
        print(f"{name} fused {fused}", flush=True)
        with launched() as kernels:
            gpu = run_gpu(w, fused=fused, flags=1)
        assert ("select_match" in kernels) == one and ("match" in kernels) != one and ("merge_csr" in kernels) == (not (one and fused)), kernels
        for l in {0, w.n_layers - 1}:
            check_layer(oracle, w, gpu, l)


MERGE_COUNTS = [0, 1, 2, 3, 4, 5, 0, 12, 15, 16, 17, 0, 19, 20, 21, 31, 32, 33, 0, 63, 64, 65]  # members of the slots
MERGE_GROUPS = {  # members of the slots, dtype, head_dim, generic kernels, token stride (elements, 0: dense), weighted
    "generic": (MERGE_COUNTS + [127, 128, 129, 255, 256, 257, 1000], "bf16", 128, True, 0, False),
    "generic_d64_weighted": (MERGE_COUNTS + [129, 257], "bf16", 64, True, 0, True),
    "generic_f32": (MERGE_COUNTS + [128, 129, 300], "f32", 128, True, 0, False),
    "generic_f32_d64": (MERGE_COUNTS + [128, 129], "f32", 64, True, 0, False),
    "generic_weighted": (MERGE_COUNTS + [128, 129], "bf16", 128, True, 0, True),
    "generic_split_slots_only": ([129] * 16, "bf16", 64, True, 0, False),  # as many partial sums as that many members can make
    "generic_split_slots_only_weighted": ([129] * 16, "bf16", 128, True, 0, True),
    "generic_slots_of_many_tasks": (MERGE_COUNTS + [129, 640, 1100, 2600], "bf16", 64, True, 0, False),  # more partial sums than a lane group has in flight
    "generic_slots_of_many_tasks_f32_weighted": (MERGE_COUNTS + [129, 640, 1100, 2600], "f32", 128, True, 0, True),
    "rows_beyond_4GiB": (MERGE_COUNTS + [129], "bf16", 128, True, 4 << 20, False),
    "rows_beyond_4GiB_weighted": (MERGE_COUNTS + [129], "bf16", 128, True, 4 << 20, True),
    "rows_up_to_4GiB": (MERGE_COUNTS + [129], "bf16", 128, True, 7 << 19, False),
    "unit": (MERGE_COUNTS + [129], "bf16", 128, False, 0, False),
    "unit_weighted": (MERGE_COUNTS + [129], "bf16", 128, False, 0, True),
    "unit_f32_d64": (MERGE_COUNTS[:18], "f32", 64, False, 0, False),
    "unit_many": (MERGE_COUNTS + [129], "bf16", 64, False, 0, False),
}


@pytest.mark.parametrize("name", list(MERGE_GROUPS))
def test_merge_of_given_groups(name):
    """flowmm_merge on a plan whose slots have as many members as the loads of a trip, of a task, one less and one more; the K and V
    rows of a sequence behind another one's, a slot without members a bit copy of its pivot (zeros of either sign too)."""
    import torch
    fb = _fb()
    counts, dtype, d, generic, stride, weighted = MERGE_GROUPS[name]
    print(f"case {name}", flush=True)
    rng = np.random.default_rng(12)
    B, lead, Lyr, Hkv = len(counts), 40, 130 if name == "unit_many" else 1, 4 if name == "unit_many" else 1
    L = B + sum(counts) + 7  # seven tokens go nowhere
    perm = rng.permutation(L)
    kept = np.sort(perm[:B])
    assign = np.full(L, -1, np.int64)
    assign[kept] = np.arange(B)
    at = B
    for slot, n in zip(rng.permutation(B), counts):
        assign[perm[at:at + n]] = slot
        at += n
    tdt, bits = (torch.bfloat16, torch.int16) if dtype == "bf16" else (torch.float32, torch.int32)
    T, stride = lead + L, stride or d
    gen = torch.Generator(device="cuda:0").manual_seed(13)
    K, V = (torch.empty(((Lyr * Hkv - 1) * T * d if stride == d else 0) + (T - 1) * stride + d, dtype=tdt, device="cuda:0") for _ in range(2))
    rows = [torch.as_strided(t, (Lyr, Hkv, T, d), (Hkv * T * d, T * d, stride, 1)) for t in (K, V)]
    for t in rows:
        t.copy_(torch.randn((Lyr, Hkv, T, d), generator=gen, device="cuda:0"))
        t[:, :, lead + kept[0], ::3] = -0.0
    flags = (fb.FLOWMM_FLAG_GENERIC_PATH if generic else 0) | (fb.FLOWMM_FLAG_WEIGHTED_MERGE if weighted else 0)
    params = fb.Params(Lyr, Hkv, Hkv, d, dtype, [lead, L], [lead, B], [[(0, lead, 0)], [(0, L, 0)]], 16, 0.25, [1.0, 1.0], flags=flags,
                       k_strides=(Hkv * T * d, T * d, stride), q_strides=(Hkv * 32 * d, 32 * d, d))
    bufs = fb.DeviceBuffers(params)
    first = torch.arange(lead, dtype=torch.int32)
    bufs.kept_idx[:] = torch.cat([first, torch.from_numpy(kept.astype(np.int32))]).cuda()
    bufs.assign[:] = torch.cat([first, torch.from_numpy(assign.astype(np.int32))]).cuda()
    bufs.mode[:], bufs.rho[:] = 0, 0.0
    bufs.merge(K, V, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    members = torch.from_numpy((assign[None, :] == np.arange(B)[:, None]) & (np.arange(L)[None, :] != kept[:, None])).double()
    n = members.sum(1)
    for l, h in ((0, 0), (Lyr - 1, Hkv - 1)):
        Kd, Vd = (t[l, h, lead:].double().cpu() for t in rows)
        w = members
        if weighted:
            unit = Kd / Kd.norm(dim=1, keepdim=True)
            w = members * (unit[kept] @ unit.T).clamp(min=0.0)
        for got, rows_d, src in ((bufs.K_out[l, h], Kd, rows[0]), (bufs.V_out[l, h], Vd, rows[1])):
            assert torch.equal(got[:lead].view(bits), src[l, h, :lead].contiguous().view(bits))
            alone = torch.nonzero(n == 0)[:, 0]
            assert torch.equal(got[lead:].cpu()[alone].view(bits), src[l, h, lead:].cpu()[torch.from_numpy(kept)][alone].contiguous().view(bits))
            want = (rows_d[kept] + w @ rows_d) / (1.0 + w.sum(1, keepdim=True))
            # sums of n + 1 fp32 terms (the weights of a weighted one carry d terms more), divided, rounded to the data type once
            terms = (n[:, None] + 2 + (d if weighted else 0)) * rows_d.abs().max()
            tol = (2.0 ** -8 if dtype == "bf16" else 2.0 ** -23) * want.abs() * 1.01 + terms * 2.0 ** -24
            assert bool(((got[lead:].double().cpu() - want).abs() <= tol).all()), (l, h)


@pytest.mark.parametrize("lens,heads,layers,d", [
    ([200, 97, 300, 150, 299], (8, 4, 16), 13, 64),     # one workgroup per unit scores, splits, matches and groups
    ([1300, 97, 2500, 1301], (8, 8, 16), 9, 64),        # kernels of their own, with folds of split slots
    ([64] * 3 + [65] * 70, (2, 2, 16), 2, 64),          # metadata of more than one block
])
def test_sequences_by_length(oracle, lens, heads, layers, d):
    """More (sequence, kv head, layer) workgroups than compute units, of unequal sequences: every one of them is taken once."""
    from paper_2511_05534_amd import workloads as wl
    from parity_utils import check_layer, run_gpu
    hq, hkv, W = heads
    print(f"lens {lens[:6]} heads {heads} layers {layers} d {d}", flush=True)
    assert layers * hkv * len(lens) > 256 and len(set(lens)) > 1
    spans = [[L // 4, L // 2, L - L // 4 - L // 2] for L in lens]
    w = wl.make_workload("", "bf16", 11, layers, hq, hkv, d, W, spans, [20] * len(lens), budgets=[W + L // 8 for L in lens])
    for fused in (False, True):
        gpu = run_gpu(w, fused=fused, flags=1)
        for l in (0, layers // 2, layers - 1):
            check_layer(oracle, w, gpu, l, flags=1)
