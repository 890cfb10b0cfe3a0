"""Kernel variants that a rule on sizes picks: each at the edges of its range, against the CPU oracle, bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

import haq_inputs as hi
import oracle
import paper_2508_07329_amd as haq
from paper_2508_07329_amd.binding import lib
from tests import offline
from tests.gpu_util import bits_equal, dev, diff_report, host
from tests.test_gpu_parity import _check_moe, _check_moe_asym
from tests.tile_sizes import DENSE_TILES, STREAM_ROWS, TALL_GROUPS

pytestmark = pytest.mark.gpu


def _linear_both_codes(T, K, N, act):
    """The dense linear in symmetric and in asymmetric codes, with and without the accumulator dump."""
    X, _, _ = hi.hidden_states(T + K + N, T, K, n_outlier=max(1, K // 200))
    s, Wq, sw = offline.quantize_linear(X, hi.gaussian_weight(T + K + N, 0, K, N))
    x, s_d, wq = dev(X), dev(s), dev(Wq)
    wp, sw_d, cs, a = haq.haq_pack_weight(wq), dev(sw), haq.haq_weight_colsum(wq), oracle.ACT[act]
    y_ref, acc_ref, _, _ = oracle.w8a8_linear(X, s, Wq, sw, act, full=True)
    y, acc, _, _ = haq.haq_w8a8_linear(x, s_d, wp, sw_d, N, a, debug=True)
    assert bits_equal(host(acc), acc_ref), diff_report(host(acc), acc_ref)
    assert bits_equal(host(y), y_ref)
    wide = torch.full((T, N + 24), 7.0, dtype=torch.float16, device=x.device)   # rows with a gap between them
    haq.haq_w8a8_linear(x, s_d, wp, sw_d, N, a, out=wide[:, :N])
    assert bits_equal(host(wide[:, :N]).copy(), y_ref) and bool((wide[:, N:] == 7.0).all())
    if K <= 16384:
        y_ref, acc_ref, _, _, _ = oracle.w8a8_linear_asym(X, s, Wq, sw, act, full=True)
        y, acc, _, _, _ = haq.haq_w8a8_linear_asym(x, s_d, wp, sw_d, cs, N, a, debug=True)
        assert bits_equal(host(acc), acc_ref), diff_report(host(acc), acc_ref)
        assert bits_equal(host(y), y_ref)
        assert bits_equal(host(haq.haq_w8a8_linear_asym(x, s_d, wp, sw_d, cs, N, a)), y_ref)


@pytest.mark.parametrize("T,K,N,act", [
    (1, 16, 16, "none"), (15, 80, 48, "relu"), (16, 448, 272, "none"), (17, 512, 16, "relu"), (32, 1040, 528, "none"),
    (33, 2064, 80, "relu"), (64, 3584, 48, "none"), (65, 960, 112, "relu"), (96, 2560, 16, "none"), (97, 2112, 64, "none"),
    (128, 4112, 272, "relu"), (129, 528, 272, "none"),
    # 128 units of 64 channels and more: four channel blocks per work-group, the last unit partly past the last channel
    (1, 64, 8192, "relu"), (16, 592, 8208, "none"), (31, 208, 8240, "relu"), (64, 1344, 8224, "none"), (90, 912, 8192, "relu"),
    (90, 912, 8208, "relu"), (128, 1104, 8208, "none"), (90, 1040, 8208, "relu"), (128, 1168, 8208, "none"),
    # wide layers of few K-steps: the tiled kernel, most of its rows past the last one
    (40, 80, 24592, "none"), (128, 272, 8224, "relu")])
def test_short_batch_linear_at_the_edges_of_its_variants(T, K, N, act):
    """Row blocks of 16 (1, 2, 4, 6, 8 of them; 129 rows take several row tiles), K-steps that do and do not divide among
    the eight waves and the prefetch depth, a last partial K-step, channel units past the last channel."""
    _linear_both_codes(T, K, N, act)


@pytest.mark.parametrize("T,K,N,act", [
    # row tiles of the streaming kernel, of 64 (the second ends in one row; one round, and many tiles) and of 96 rows; many rows
    (129, 1040, 528, "none"), (257, 592, 16, "relu"), (1030, 1104, 272, "none"), (333, 1040, 4096, "relu"), (500, 1088, 4080, "none"),
    # tiles of 128 and 256 rows, and many of them
    (300, 80, 2064, "relu"), (513, 80, 10240, "none"), (2049, 48, 14352, "none")])
def test_dense_linear_at_the_edges_of_its_tile_shapes(T, K, N, act):
    _linear_both_codes(T, K, N, act)


@pytest.mark.parametrize("T,K,N,act", [
    # K-steps: one to six, the last one partial, in the streaming kernel and (with the accumulator dump) 128 x 256 tiles
    (300, 16, 272, "relu"), (300, 208, 272, "none"), (257, 256, 400, "none"), (300, 272, 2064, "relu"), (300, 336, 2064, "none"),
    # 192-row tiles (one tile and a row; a row short of one) and others, the last channel tile in 16 channels
    (385, 1040, 8208, "relu"), (191, 592, 16400, "none"), (513, 1040, 16400, "none"), (385, 400, 16400, "relu")])
def test_dense_linear_at_the_edges_of_its_rings_and_tiles(T, K, N, act):
    _linear_both_codes(T, K, N, act)


@pytest.mark.parametrize("T,K,N", [size for shapes in (DENSE_TILES, STREAM_ROWS) for sizes in shapes.values() for size in sizes])
def test_dense_linear_on_each_tile_shape(T, K, N):
    """Both codes; the accumulator dump takes 128 x 256 tiles, the calls without it the tiles that the size is listed under."""
    _linear_both_codes(T, K, N, "relu" if T % 2 else "none")


@pytest.mark.parametrize("T,N", [(130, 4_000_016), (4_000_016, 32)])
def test_tiled_linear_on_operands_past_4_gb(T, N):
    """Byte offsets that need more than 32 bits: in the weights, then in the codes.  Every output of the rows or channels
    checked (the first, the last, those on both sides of an offset of 2^32) is an exact sum and two roundings."""
    K, g = 1088, torch.Generator("cuda").manual_seed(T)
    code = lambda n: torch.randint(-127, 128, (n,), dtype=torch.int8, device="cuda", generator=g)
    q, w = code(haq.haq_packed_act_bytes(T, K)), code(haq.haq_packed_bytes(K, N))
    assert max(q.numel(), w.numel()) > 2 ** 32
    sx, sw = (torch.rand(n, device="cuda", generator=g) * 1e-3 + 1e-3 for n in (T, N))
    y = haq.haq_gemm_w8a8_packed(q, sx, w, sw, T, K, N)

    def some(n):
        near = 2 ** 32 // K  # the offset of row i in the last chunk is near i * K
        return torch.tensor(sorted({i for i in [0, 1, n - 2, n - 1, *range(near - 40, near + 300)] if 0 <= i < n} if n > 200 else range(n)))

    t, n = some(T), some(N)
    rows = lambda p, i: p.view(K // 16, -1, 16)[:, i.to(p.device)].permute(1, 0, 2).reshape(len(i), K).cpu().double()
    acc = rows(q, t) @ rows(w, n).T  # below 2^53: exact in any order
    ref = ((acc.float() * sx.cpu()[t, None]) * sw.cpu()[None, n]).half()
    assert torch.equal(y[t.to(y.device)][:, n.to(y.device)].cpu().view(torch.int16), ref.view(torch.int16))


@pytest.mark.parametrize("T,K", [(256, 816), (257, 80), (511, 4112), (1024, 528), (1025, 336), (256, 16384), (257, 8208), (1030, 1040)])
def test_short_batch_quantisers_at_the_edges_of_their_row_split(T, K):
    """One, two and eight rows per work-group (the line lies at one and at four rows per compute unit, 256 of them)."""
    X, _, _ = hi.hidden_states(T + K, T, K, n_outlier=max(1, K // 200))
    X[T // 2] = 0
    W = hi.gaussian_weight(T + K, 0, K, 16)
    s, Wq, sw = offline.quantize_linear(X, W)
    q_ref, sx_ref = oracle.w8a8_linear(X, s, Wq, sw, "none", full=True)[2:]
    q, sx = haq.haq_smooth_quant_act(dev(X), dev(s))
    assert bits_equal(host(q), q_ref) and bits_equal(host(sx), sx_ref)
    qp, sx = haq.haq_quant_act_packed(dev(X), dev(s))
    rows = host(qp).reshape(-1, haq.haq_packed_act_rows(T), 16)[:K // 16, :T]
    assert np.array_equal(rows.transpose(1, 0, 2).reshape(T, K), q_ref) and bits_equal(host(sx), sx_ref)
    wq = dev(Wq)
    y_ref, _, q_ref, sx_ref, zp_ref = oracle.w8a8_linear_asym(X, s, Wq, sw, "none", full=True)
    y, _, q, sx, zp = haq.haq_w8a8_linear_asym(dev(X), dev(s), haq.haq_pack_weight(wq), dev(sw), haq.haq_weight_colsum(wq), 16, debug=True)
    assert bits_equal(host(q), q_ref) and bits_equal(host(sx), sx_ref) and bits_equal(host(zp), zp_ref)
    assert bits_equal(host(y), y_ref)


@pytest.mark.parametrize("T", [257, 1030, 4100])
@pytest.mark.parametrize("K", [16, 32, 48])
def test_quantisers_on_rows_of_fewer_chunks_than_a_thread_has_rows(T, K):
    """Two or four rows to a thread and one to three chunks of 16 channels to a row: every row's scale is written."""
    _linear_both_codes(T, K, 16, "none")


@pytest.mark.parametrize("T,K,N,n_e", [(40, 64, 16, 37), (33, 128, 272, 16), (24, 192, 528, 17)])
def test_smoothing_search_on_more_candidates_than_one_pass_over_the_weights_takes(T, K, N, n_e):
    """16 candidates to a pass: one, one and a single one, two and a rest; a channel of zeros, one below the range in which a
    code is formed by the scale's reciprocal, one of which only a single weight is not zero."""
    X, _, _ = hi.hidden_states(T + K, T, K, n_outlier=2)
    W = hi.gaussian_weight(T + K, 0, K, N)
    W[:, 3], W[:, 5], W[:, 7] = 0.0, W[:, 5] * np.float32(2.0 ** -110), 0.0
    W[K - 1, 7] = -0.75
    grid = [i / (n_e - 1) for i in range(n_e)]
    losses_ref, best_ref, s_ref = oracle.smoothing_search(X, W, grid, True)
    losses, best, s = haq.haq_smoothing_search(dev(X), dev(W), grid, True)
    assert np.array_equal(np.asarray(losses), losses_ref), diff_report(np.asarray(losses), losses_ref)
    assert best == best_ref and bits_equal(host(s), s_ref)


@pytest.mark.parametrize("T,K,N", [(17, 63, 17), (80, 65, 130), (40, 128, 9), (33, 257, 66), (64, 330, 1000), (100, 448, 208), (70, 700, 81)])
def test_layer_quantiser_at_the_edges_of_its_blocks(T, K, N):
    """Panels and blocks of 64 with one row less and more, k chunks of 16 with a remainder, a second stretch of 256
    channels, errors kept in the freed matrices (700 x 81) and, where they do not fit there, block by block (330 x 1000)."""
    rng = np.random.default_rng(T + K + N)
    X = (rng.standard_normal((T, 12)) @ rng.standard_normal((12, K)) + 0.1 * rng.standard_normal((T, K))).astype(np.float16)
    W = hi.gaussian_weight(T + K, 0, K, N)
    W[3, :] = -0.0
    s = oracle.smoothing_vector(oracle.col_absmax_f16(X), oracle.row_absmax_f32(W), 0.5)
    for sv in (None, s):
        H_ref = oracle.hessian(X, sv, 0.01)
        H = haq.haq_hessian_f64(dev(X), None if sv is None else dev(sv), 0.01)
        assert bits_equal(host(H), H_ref), diff_report(host(H), H_ref)
        U_ref = oracle.inverse_cholesky_upper(H_ref)
        U = haq.haq_inverse_cholesky_upper_f64(H)
        assert bits_equal(host(U), U_ref), diff_report(host(U), U_ref)
        Wq_ref, sw_ref = oracle.gptq(W, sv, U_ref)
        Wq, sw = haq.haq_hessian_quant_weight(dev(X), dev(W), None if sv is None else dev(sv), 0.01)
        assert bits_equal(host(sw), sw_ref) and bits_equal(host(Wq), Wq_ref)


def test_an_indefinite_hessian_leaves_plain_rounding():
    """Equal channels without damping: the second pivot is exactly zero."""
    K, N = 64, 48
    x, W = torch.ones(4, K, dtype=torch.float16, device="cuda"), hi.gaussian_weight(5, 0, K, N)
    w, wq, sw = dev(W), torch.full((K, N), 85, dtype=torch.int8, device="cuda"), torch.empty(N, device="cuda")
    ws = torch.empty(int(lib().haq_hessian_quant_workspace_bytes(K, N)), dtype=torch.uint8, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    rc = lib().haq_hessian_quant_weight(p(x), ctypes.c_int64(K), 4, p(w), None, K, N, ctypes.c_double(0.0), p(wq), p(sw), p(ws),
                                        ctypes.c_size_t(ws.numel()), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == -1 and b"not positive definite" in lib().haq_last_error()
    Wq_ref, sw_ref = oracle.quant_weight(W, None)
    assert bits_equal(host(wq), Wq_ref) and bits_equal(host(sw), sw_ref)


@pytest.mark.parametrize("rows,cols", [(33, 40), (70, 16)])
def test_binary64_products_at_strides_past_32_bits(rows, cols):
    """A tile's offsets from its first element exceed 2^32 elements: rows of x 2^27 apart (reference product), tokens 2^29
    apart (Hessian), and a weight row of 2^29 values.  What lies between the rows is never read."""
    rng = np.random.default_rng(rows)
    X, W = rng.standard_normal((rows, cols)).astype(np.float16), rng.standard_normal((cols, 24)).astype(np.float32)
    far = lambda n, ld: torch.empty((n - 1) * ld + cols, dtype=torch.float16, device="cuda").as_strided((n, cols), (ld, 1))
    x = far(rows, 2 ** 27)
    x.copy_(dev(X))
    assert bits_equal(host(haq.haq_reference_matmul_f64(x, dev(W))), oracle.matmul_f64(X, W))
    del x
    x = far(17, 2 ** 29)
    x.copy_(dev(X[:17]))
    assert bits_equal(host(haq.haq_hessian_f64(x, None, 0.01)), oracle.hessian(X[:17], None, 0.01))
    del x
    n, k = 2 ** 29, 9
    w = torch.zeros(k, n, dtype=torch.float32, device="cuda")
    w[:, -100:] = dev(W[:k, :1])
    y = haq.haq_reference_matmul_f64(dev(X[:1, :k]), w)
    assert bits_equal(host(y[:, -100:]), oracle.matmul_f64(X[:1, :k], np.repeat(W[:k, :1], 100, axis=1))) and not bool(y[:, :-100].any())

@pytest.mark.parametrize("H,I,first,second,E", [
    # few channels: the down projection streams in tiles of 32, 64, 96 and 128 rows (and one row more, and groups of two and
    # three tiles, which share their weights); the gate/up projection takes the tiled kernel's form for few rows; groups
    # with one row tile, one row more, two tiles, one row, none
    (192, 448, (129, 97, 65, 33, 17, 1), (128, 96, 64, 32, 16, 6), 16),
    (64, 64, (257, 2), (130, 128, 1), 12),
    (320, 448, (129, 64, 65, 84), (256, 1, 0, 85), 8),
    (128, 704, (100, 28), (127, 1), 4),
    # 80 rows on average and 512 units of 64 channels: the down projection in 128 x 128 tiles
    (4096, 64, (129, 64, 65, 62), (256, 1, 0, 63), 8),
    # 56 rows on average and more channel tiles than CUs: the form for few rows in both projections; channel tiles that are
    # no multiple of 8 (the count goes on from group to group)
    (4096, 64, (300, 148), (1, 447), 16),
    (2624, 192, (130, 70, 1, 199), (128, 129, 0, 143), 16),
    # 192 x 256 tiles of the down projection
    *[(H, I, first, second, len(first) + len(second)) for H, I, first, second in TALL_GROUPS]])
def test_routed_experts_at_the_edges_of_their_row_tiles(H, I, first, second, E):
    """Group sizes are set through the logits: every token has one expert of `first` and one of `second`."""
    T = sum(first)
    assert T == sum(second) and len(first) + len(second) <= E
    m = offline.small_moe(seed=T + H, T=T, H=H, I=I, E=E)
    logits = np.full((T, E), -4.0, np.float16)
    logits[np.arange(T), np.repeat(np.arange(len(first)), first)] = 2.0
    logits[np.arange(T), len(first) + np.repeat(np.arange(len(second)), second)[::-1]] = 1.5
    m["logits"] = logits + (np.arange(T)[:, None] % 7 * 0.0625).astype(np.float16)
    _check_moe(m)
    counts = _check_moe_asym(m)
    assert tuple(counts[:len(first) + len(second)]) == (*first, *second)


@pytest.mark.parametrize("T,H,I,E", [(1, 64, 64, 2), (63, 2048, 64, 32), (64, 2112, 128, 3), (65, 192, 128, 8), (33, 16384, 64, 4)])
def test_asymmetric_tokens_and_routing_in_one_launch(T, H, I, E):
    """Work-groups of as many threads as pairs need, as chunks of 16 channels need, one chunk more than whole waves, and the
    largest; one token more than the launch takes; all 32 experts."""
    _check_moe_asym(offline.small_moe(seed=T + H, T=T, H=H, I=I, E=E))


@pytest.mark.parametrize("H,I,E,rows", [(256, 192, 4, 300), (128, 64, 8, 500), (4096, 64, 8, 257)])
def test_large_expert_groups(H, I, E, rows):
    """More than 128 rows per expert on average, several row tiles of 128 rows to a group, the last group the longest."""
    T = E * rows // 2
    m = offline.small_moe(seed=rows + H, T=T, H=H, I=I, E=E)
    first, second = np.arange(T) % E, (np.arange(T) // E) % E
    second = np.where(second == first, (first + 1) % E, second)
    for e, n in enumerate((193, 129)):  # tokens past these go to the last expert
        first[np.flatnonzero(first == e)[n:]] = E - 1
    second = np.where(second == first, (first + 1) % E, second)
    logits = np.full((T, E), -4.0, np.float16)
    logits[np.arange(T), second] = 1.5
    logits[np.arange(T), first] = 2.0
    m["logits"] = logits
    _check_moe(m)
    _check_moe_asym(m)


@pytest.mark.parametrize("T,K,N,act", [
    # one, two, four and eight waves to a row: the most rows and channels of each, one row and one channel chunk more
    (16, 1024, 48, "relu"), (17, 1024, 16, "none"), (8, 1040, 272, "none"), (8, 2048, 16, "relu"), (9, 2048, 32, "none"), (4, 2064, 80, "none"),
    (4, 4096, 16, "relu"), (2, 4112, 144, "none"), (2, 8192, 16, "relu"), (3, 8192, 16, "none"), (1, 8208, 16, "none"), (1, 16, 16, "relu"),
    # units of 64 channels, the last one partly past the last channel
    (16, 592, 8208, "none"), (5, 1552, 8224, "relu"), (3, 4096, 8240, "none"), (1, 6160, 8192, "none")])
def test_few_rows_of_short_k_in_one_launch(T, K, N, act):
    """The calls without debug outputs; those with them take the two launches."""
    _linear_both_codes(T, K, N, act)


@pytest.mark.parametrize("T,K", [(16, 1008), (7, 2048), (4, 3088), (2, 8192)])
def test_one_launch_linear_without_smoothing_on_odd_rows_and_in_place(T, K):
    """No smoothing vector; entries whose reciprocal is not used; a row of zeros, one of tiny and one of large values; rows
    with a gap between them; and outputs over the inputs, which only the two launches allow."""
    X, _, _ = hi.hidden_states(T + K, T, K, n_outlier=2)
    X[0] = 0
    X[T - 1] *= np.float16(2.0 ** -12)
    s, Wq, sw = offline.quantize_linear(X, hi.gaussian_weight(T + K, 0, K, K))
    s[3], s[K - 1] = 2.0 ** 50, 2.0 ** -45
    wp, sw_d = haq.haq_pack_weight(dev(Wq)), dev(sw)
    for sv in (None, s):
        ref = oracle.w8a8_linear(X, sv if sv is not None else np.ones(K, np.float32), Wq, sw, "none")
        sd = dev(sv) if sv is not None else None
        x = torch.full((T, K + 8), 3.0, dtype=torch.float16, device="cuda")
        x[:, :K] = dev(X)
        assert bits_equal(host(haq.haq_w8a8_linear(x[:, :K], sd, wp, sw_d, K)), ref)
        both = dev(X)
        assert bits_equal(host(haq.haq_w8a8_linear(both, sd, wp, sw_d, K, out=both)), ref)


@pytest.mark.parametrize("T,K,N", [(16, 1008, 48), (7, 2048, 16), (4, 3088, 80), (2, 8192, 16)])
def test_one_launch_linear_on_infinities_and_nan(T, K, N):
    """The same bits as the two launches, which the calls with debug outputs take: rows with an infinity of either sign, with a
    NaN, with both, with nothing else; a zero, an infinite and a NaN entry of the smoothing vector."""
    rng = np.random.default_rng(T + K)
    X = rng.standard_normal((T, K)).astype(np.float16)
    X[0, [1, 40]], X[0, 7] = np.inf, -np.inf
    X[1, [3, K - 1]] = np.nan
    if T > 2:
        X[2, 5], X[2, 6], X[3] = np.nan, -np.inf, np.nan
    _, Wq, sw = offline.quantize_linear(np.ones((1, K), np.float16), hi.gaussian_weight(T + K, 0, K, N))
    s = (rng.random(K) + 0.5).astype(np.float32)
    wp, sw_d, x = haq.haq_pack_weight(dev(Wq)), dev(sw), dev(X)
    for bad in (None, 0.0, np.inf, np.nan):
        if bad is not None:
            s[K // 2] = bad
        for sv in (dev(s), None):
            y = haq.haq_w8a8_linear(x, sv, wp, sw_d, N)
            two = haq.haq_w8a8_linear(x, sv, wp, sw_d, N, debug=True)[0]
            assert bool((y.view(torch.int16) == two.view(torch.int16)).all())


def test_ffn_of_few_rows_in_two_launches():
    for T, K, F, N in ((16, 320, 1024, 80), (8, 1024, 2048, 1024), (2, 2048, 8192, 2048), (4, 1024, 8192, 512)):
        X, _, _ = hi.hidden_states(T + K, T, K, n_outlier=2)
        s1, W1, sw1 = offline.quantize_linear(X, hi.gaussian_weight(T + K, 0, K, F))
        h = oracle.w8a8_linear(X, s1, W1, sw1, "relu")
        s2, W2, sw2 = offline.quantize_linear(h, hi.gaussian_weight(T + K, 1, F, N))
        y = haq.haq_w8a8_ffn(dev(X), dev(s1), haq.haq_pack_weight(dev(W1)), dev(sw1), F, oracle.ACT["relu"], dev(s2), haq.haq_pack_weight(dev(W2)), dev(sw2), N)
        assert bits_equal(host(y), oracle.w8a8_linear(h, s2, W2, sw2, "none"))
