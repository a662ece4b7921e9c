"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded
inputs.  Decoded weights are bit-exact; GEMM within 1e-3 * sum|a w| + 1e-6 per element."""
import numpy as np
import pytest

import oracle
from paper_2603_17435_amd import binding, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


# --------------------------------------------------------------------------- decode
@pytest.mark.parametrize("kind,N,K", [("gauss", 64, 64), ("gauss", 192, 320), ("rowscale", 256, 192),
                                       ("student_t", 128, 448), ("outliers", 320, 128), ("specials", 256, 256)])
def test_decompress_bit_exact_small(gu, kind, N, K):
    W = inputs.make_weights(kind, N, K, seed=inputs.seed_for(3, 0, 1))
    out = gu.gpu_decompress(W)
    assert np.array_equal(out, oracle.decode(oracle.encode(W)))
    assert np.array_equal(out, W)


@pytest.mark.parametrize("pad", [0, 8, 40, 64])
def test_decompress_rows_and_padding(gu, pad):
    """Every element differs from its neighbours in row and column (a swapped lane, row or half shows),
    and the columns between the rows stay as they were."""
    import torch
    N, K = 320, 192
    W = (np.arange(N, dtype=np.uint32)[:, None] * 131 + np.arange(K, dtype=np.uint32) * 7 + 0x3A00).astype(np.uint16)
    blob, d = binding.zs_encode(W)
    out = torch.full((N, K + pad), 0x5A5A, dtype=torch.int16, device="cuda")
    binding.zs_decompress(d, gu.upload_blob(blob), out, ldw=K + pad)
    got = out.cpu().numpy().view(np.uint16)
    assert np.array_equal(got[:, :K], W) and (got[:, K:] == 0x5A5A).all()


@pytest.mark.parametrize("N,K,pad", [(3840, 4096, 0), (3904, 4096, 8), (4608, 4096, 0), (4672, 4096, 24)])
@pytest.mark.parametrize("kind", ["gauss", "rowscale", "spread"])
def test_decompress_half_and_whole_lines(gu, kind, N, K, pad):
    """Sizes on both sides of the change from stores of half cache lines to whole ones (15 BlockTiles for
    every compute unit, 18 with many fallbacks), with each of the three decoders."""
    import torch
    rng = np.random.default_rng(57)
    if kind == "spread":                        # 5 % of the weights outside the window, evenly
        W = (rng.integers(0, 1 << 16, (N, K)) & 0x807F | 0x3F80).astype(np.uint16)
        W[rng.random((N, K)) < 0.05] &= 0x9FFF
    else:
        W = inputs.make_weights(kind, N, K, seed=58)
    blob, d = binding.zs_encode(W)
    out = torch.full((N, K + pad), 0x5A5A, dtype=torch.int16, device="cuda")
    binding.zs_decompress(d, gu.upload_blob(blob), out, ldw=K + pad)
    got = out.cpu().numpy().view(np.uint16)
    assert np.array_equal(got[:, :K], W) and (got[:, K:] == 0x5A5A).all()


def test_decompress_all_bit_patterns(gu):
    W = np.random.default_rng(0).permutation(np.arange(65536, dtype=np.uint16)).reshape(256, 256)
    assert np.array_equal(gu.gpu_decompress(W), W)
    W = np.arange(65536, dtype=np.uint16).reshape(256, 256)
    assert np.array_equal(gu.gpu_decompress(W), W)


@pytest.mark.parametrize("case", ["zeros", "neg_zero_mix", "inf", "all_fallback_blocks", "window_at_top"])
def test_decompress_degenerate(gu, case):
    rng = np.random.default_rng(4)
    if case == "zeros":
        W = np.zeros((64, 128), dtype=np.uint16)                      # base_exp = -1
    elif case == "neg_zero_mix":
        W = rng.choice(np.array([0x0000, 0x8000, 0x0001, 0x807F, 0x0080, 0x8123], dtype=np.uint16), (128, 64))
    elif case == "inf":
        W = rng.choice(np.array([0x7F80, 0xFF80, 0x7FC0, 0xFFFF, 0x7F00], dtype=np.uint16), (64, 64))
    elif case == "all_fallback_blocks":
        W = inputs.gaussian_weights(128, 128, 8)
        W[:64, 64:] = inputs.f32_to_bf16(rng.standard_normal((64, 64)).astype(np.float32) * 1e5)
        W[64:, :64] = rng.integers(0, 65536, (64, 64)).astype(np.uint16)
    else:
        W = ((rng.integers(249, 256, (64, 64)) << 7) | rng.integers(0, 128, (64, 64))).astype(np.uint16)
    assert np.array_equal(gu.gpu_decompress(W), W)


def test_decompress_config1_full(gu):
    W = inputs.gaussian_weights(4096, 4096, inputs.seed_for(1))
    assert np.array_equal(gu.gpu_decompress(W), W)


# --------------------------------------------------------------------------- GEMM
@pytest.mark.parametrize("M", [1, 3, 8, 16, 17, 32, 33, 64, 100])
def test_gemm_small_all_M(gu, M):
    W = inputs.gaussian_weights(192, 320, inputs.seed_for(2, 1))
    A = inputs.activations(M, 320, inputs.seed_for(2, 1, 1))
    gu.check_gemm(W, A)


@pytest.mark.parametrize("kind", ["rowscale", "student_t", "outliers"])
@pytest.mark.parametrize("M", [1, 16])
def test_gemm_adversarial_small(gu, kind, M):
    W = inputs.make_weights(kind, 256, 512, seed=inputs.seed_for(3, 2))
    A = inputs.activations(M, 512, inputs.seed_for(3, 2, 1))
    gu.check_gemm(W, A)


@pytest.mark.parametrize("per_row", [2, 3, 5, 7, 8, None])
def test_rows_with_many_fallbacks(gu, per_row):
    """FragTile rows with a given number of out-of-window elements at random places (None: any number
    from 0 to 8 by turns), in a matrix that has enough of them for the long L window."""
    rng = np.random.default_rng(50 + (per_row or 0))
    W = inputs.gaussian_weights(192, 448, 51)
    rows = W.reshape(-1, 8)                     # eight consecutive k = one FragTile row
    hit = rng.random(len(rows)) < 0.4
    count = rng.integers(0, 9, len(rows)) if per_row is None else np.full(len(rows), per_row)
    place = rng.random(rows.shape).argsort(1) < np.where(hit, count, 0)[:, None]
    far = (rng.integers(0, 1 << 16, rows.shape) & 0x80FF) | (rng.integers(1, 60, rows.shape) << 8)
    W = np.where(place, far.astype(np.uint16), rows).reshape(W.shape).astype(np.uint16)
    _, d = binding.zs_encode(W)
    assert 2 * d.n_fallback / (3 * 7) > 256     # bytes per BlockTile: beyond the short window
    assert np.array_equal(gu.gpu_decompress(W), W)
    for M in (5, 31, 40, 77):                   # every kernel that decodes
        gu.check_gemm(W, inputs.activations(M, 448, 52 + M))


@pytest.mark.parametrize("share,rows,loop", [(0.05, 1.0, True), (0.0545, 1.0, True), (0.056, 1.0, False), (0.05, 0.1, False)])
def test_careful_decoder_choice(gu, share, rows, loop):
    """The long L window with few fallbacks that lie evenly (rows of three and more one at a time) and
    with more of them, or with as many in a tenth of the rows (register by register)."""
    rng = np.random.default_rng(54)
    N, K = 1024, 448
    W = inputs.gaussian_weights(N, K, 55) & 0x807F | 0x3F80      # one exponent, so nothing else falls out
    chosen = rng.permutation(N)[:int(N * rows)]
    pick = np.zeros((N, K), dtype=bool)
    flat = rng.permutation(chosen.size * K)[:round(N * K * share)]
    pick[chosen[flat // K], flat % K] = True
    W = np.where(pick, (W & 0x807F) | (rng.integers(1, 60, W.shape) << 7), W).astype(np.uint16)
    _, d = binding.zs_encode(W)
    n_bt = (N // 64) * (K // 64)
    assert d.n_fallback == round(N * K * share) and 2 * d.n_fallback / n_bt > 256
    assert (18 * d.n_fallback <= N * K and d.max_l_units * 16 * n_bt <= 3 * d.n_fallback) == loop
    assert np.array_equal(gu.gpu_decompress(W), W)
    for M in (5, 31, 40, 77, 150):              # every kernel that decodes
        gu.check_gemm(W, inputs.activations(M, K, 56 + M))


def test_gemm_specials(gu):
    """Finite specials: numeric check.  Inf/NaN: class check (NaN <-> NaN, Inf same sign)."""
    A = inputs.activations(16, 256, 9)
    W = inputs.special_weights(256, 256, 10, finite_only=True)
    gu.check_gemm(W, A)
    W = inputs.special_weights(256, 256, 11, finite_only=False)
    gu.check_gemm(W, A)


@pytest.mark.parametrize("M", [70, 128, 150, 256, 300])
def test_gemm_shared_decode_specials(gu, M):
    """Infinities and NaN through the producer / consumer kernel: weights of all kinds, then an activation
    row of each kind at the first, an inner and the last token (beyond 256 in the second launch); the
    rows beside them stay as they are."""
    A = inputs.activations(M, 256, 64)
    gu.check_gemm(inputs.special_weights(256, 256, 65, finite_only=True), A)
    gu.check_gemm(inputs.special_weights(256, 256, 66, finite_only=False), A)
    A = A.copy()
    A[0, 3], A[M // 2, 17], A[M - 1, 255] = 0x7F80, 0xFF80, 0x7FC0      # +Inf, -Inf, NaN
    C = gu.check_gemm(inputs.gaussian_weights(256, 256, 67), A)
    assert not np.isfinite(C[[0, M // 2, M - 1]]).any()
    assert np.isfinite(np.delete(C, [0, M // 2, M - 1], axis=0)).all()


def test_gemm_every_config_small(gu):
    W = inputs.gaussian_weights(256, 1024, 12)
    for cfg, name in binding.zs_gemm_configs().items():
        M = int(name[1:name.index("_")])  # tokens per launch
        for m in (M, M - 5):
            A = inputs.activations(m, 1024, 13 + m)
            gu.check_gemm(W, A, config=cfg)


def test_gemm_workgroup_counts(gu):
    """Forced workgroup counts: ranges that cut strips anywhere, many tasks per workgroup,
    one workgroup for everything, more workgroups asked for than there are BlockTiles."""
    W = inputs.gaussian_weights(448, 320, 30)  # 7 strips x 5 BlockTiles
    A = inputs.activations(16, 320, 31)
    for wgs in (1, 2, 3, 6, 7, 11, 35, 200):
        gu.check_gemm(W, A, config=1 + 256 * wgs)
    names = {v: k for k, v in binding.zs_gemm_configs().items()}
    A = inputs.activations(41, 320, 34)  # producer / consumer kernel, three consumers, ragged M
    for wgs in (1, 3, 7, 35):
        gu.check_gemm(W, A, config=names["p64_l0_w7"] + 256 * wgs)
    W = inputs.gaussian_weights(1024, 64, 32)  # one BlockTile per strip: every tile is a task
    A = inputs.activations(7, 64, 33)
    for wgs in (1, 3, 16):
        gu.check_gemm(W, A, config=256 * wgs)


@pytest.mark.parametrize("M", [1, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("contributors", [2, 4, 5, 6, 7, 8, 9, 10, 17, 18, 40])
def test_gemm_exchange_batches(gu, contributors, M):
    """One strip summed from several workgroups, around the number of partial tiles that are read at a
    time (4; from five on 16, 8 or 4 for up to 16, 32 and 64 tokens); the scratch buffer is zero again afterwards."""
    import torch
    K = 64 * contributors                       # one BlockTile, so one workgroup, per contributor
    W, A = inputs.gaussian_weights(64, K, 70), inputs.activations(M, K, 71 + M)
    C_ref, S = oracle.gemm(A, W)
    blob, d = binding.zs_encode(W)
    dev, a = gu.upload_blob(blob), torch.from_numpy(A.view(np.int16)).cuda()
    ws = torch.zeros(max(binding.zs_gemm_workspace(d, M), 256), dtype=torch.uint8, device="cuda")
    for _ in range(3):
        c = torch.full((M, 64), float("nan"), dtype=torch.float32, device="cuda")
        binding.zs_gemm(d, dev, a, c, M, workspace_dev=ws, workspace_bytes=ws.numel())
        gu.assert_gemm_matches(c.cpu().numpy(), C_ref, S)
        assert not ws.any()


@pytest.mark.parametrize("config", ["m16_l0_w8", "m16_l0_w11", "m32_l0_w7", "m32_l0_w10", "m64_l0_w7", "m16_l4_w7", "m32_l4_w6", "m64_l4_w5"])
def test_gemm_tasks_of_a_workgroup(gu, config):
    """Ranges of one, two and many strip parts, whole and shared, first ones through the writer wave and the last one
    through all waves, with every number of rows of four tokens; with sums in tiles of their own and in tiles
    under a lock.  Every call is repeated and leaves the scratch buffer at zero."""
    import torch
    names = {v: k for k, v in binding.zs_gemm_configs().items()}
    law = "gauss" if "_l0_" in config else "rowscale"
    W = inputs.gaussian_weights(448, 1344, 90) if law == "gauss" else inputs.make_weights(law, 448, 1344, seed=91)
    W_dec = oracle.decode(oracle.encode(W))
    blob, d = binding.zs_encode(W)
    dev = gu.upload_blob(blob)                  # 7 strips x 21 BlockTiles
    tokens = int(config[1:3])
    for M in sorted({1, 4, 5, tokens // 2 + 1, tokens - 3, tokens}):
        A = inputs.activations(M, 1344, 92 + M)
        C_ref, S = oracle.gemm(A, W_dec)
        a = torch.from_numpy(A.view(np.int16)).cuda()
        for wgs in (1, 2, 5, 7, 10, 17, 30, 147):
            number = names[config] + 256 * wgs
            ws = torch.zeros(binding.zs_gemm_workspace(d, M, number), dtype=torch.uint8, device="cuda")
            for _ in range(2):
                c = torch.full((M, 448), float("nan"), dtype=torch.float32, device="cuda")
                binding.zs_gemm(d, dev, a, c, M, workspace_dev=ws, workspace_bytes=ws.numel(), config=number)
                gu.assert_gemm_matches(c.cpu().numpy(), C_ref, S)
            assert not ws.any()


@pytest.mark.parametrize("law", ["gauss", "rowscale"])
@pytest.mark.parametrize("M", [65, 97, 127, 128, 129, 193, 255, 256, 257])
def test_gemm_shared_decode_edges(gu, M, law):
    """Producer / consumer kernel at the edges of its consumers and launches (257: a second panel), over
    ranges that cut strips anywhere (forced workgroup counts: one tile each, a few, all of them) and
    hold fewer and more tiles than the ring of decoded tiles."""
    W = inputs.gaussian_weights(320, 448, 60) if law == "gauss" else inputs.make_weights(law, 320, 448, seed=61)
    A = inputs.activations(M, 448, 62 + M)
    _, d = binding.zs_encode(W)
    pick = binding.zs_gemm_pick_config(d, M)
    for wgs in (0, 1, 3, 8):                    # 5 strips x 7 BlockTiles: 1, 35, 11 or 12, 4 or 5 to a workgroup
        gu.check_gemm(W, A, config=pick + 256 * wgs)


def test_gemm_shared_strips_with_and_without_scratch(gu):
    """Strips cut between workgroups: with scratch memory the partial tiles are parked there and
    summed by the last workgroup to arrive, and the whole buffer is left at zero for the next
    call, whatever matrix it is for; without it the fallback (cleared C + FP32 atomics) is used."""
    import torch
    W1 = inputs.gaussian_weights(448, 320, 40)   # 7 strips x 5 BlockTiles
    W2 = inputs.gaussian_weights(192, 1024, 41)  # 3 strips x 16 BlockTiles
    W3 = inputs.gaussian_weights(8192, 128, 43)  # 128 strips x 2 BlockTiles
    ws = torch.zeros(1 << 22, dtype=torch.uint8, device="cuda")
    for M in (5, 16, 27):
        runs = {}
        for name, W in (("w1", W1), ("w2", W2), ("w3", W3)):
            A = inputs.activations(M, W.shape[1], 42 + M)
            blob, d = binding.zs_encode(W)
            dev = gu.upload_blob(blob)
            a = torch.from_numpy(A.view(np.int16)).cuda()
            C_ref, S = oracle.gemm(A, W)
            for wgs in (3, 11, 100, 0):
                outs = []
                for rep in range(3):  # same scratch for every call, never cleared again
                    c = torch.full((M, d.N), float("nan"), dtype=torch.float32, device="cuda")
                    binding.zs_gemm(d, dev, a, c, M, workspace_dev=ws, workspace_bytes=ws.numel(), config=256 * wgs)
                    torch.cuda.synchronize()
                    outs.append(c.cpu().numpy())
                for out in outs:
                    gu.assert_gemm_matches(out, C_ref, S)
                c = torch.full((M, d.N), float("nan"), dtype=torch.float32, device="cuda")
                binding.zs_gemm(d, dev, a, c, M, workspace_dev=None, workspace_bytes=0, config=256 * wgs)
                torch.cuda.synchronize()
                gu.assert_gemm_matches(c.cpu().numpy(), C_ref, S)
                runs[(name, wgs)] = outs[0]
    assert not ws.cpu().numpy().any()  # counters and slots are back at zero
    # scratch that cannot be used (too small, or not 256-byte aligned) is ignored, not an error
    W, M = W1, 9
    A = inputs.activations(M, W.shape[1], 50)
    blob, d = binding.zs_encode(W)
    dev = gu.upload_blob(blob)
    a = torch.from_numpy(A.view(np.int16)).cuda()
    C_ref, S = oracle.gemm(A, W)
    need = binding.zs_gemm_workspace(d, M, 256 * 3)
    for buf, nbytes in ((ws, need - 1), (ws[16:], ws.numel() - 16)):
        c = torch.full((M, d.N), float("nan"), dtype=torch.float32, device="cuda")
        binding.zs_gemm(d, dev, a, c, M, workspace_dev=buf, workspace_bytes=nbytes, config=256 * 3)
        torch.cuda.synchronize()
        gu.assert_gemm_matches(c.cpu().numpy(), C_ref, S)
    assert not ws.cpu().numpy().any()
    # all-zero weights through shared strips: partial tiles of exact zeros
    Wz = np.zeros((128, 1024), dtype=np.uint16)
    blob, d = binding.zs_encode(Wz)
    dev = gu.upload_blob(blob)
    A = inputs.activations(16, 1024, 51)
    a = torch.from_numpy(A.view(np.int16)).cuda()
    for rep in range(2):
        c = torch.full((16, 128), float("nan"), dtype=torch.float32, device="cuda")
        binding.zs_gemm(d, dev, a, c, 16, workspace_dev=ws, workspace_bytes=ws.numel(), config=256 * 5)
        torch.cuda.synchronize()
        assert not c.cpu().numpy().any()
    assert not ws.cpu().numpy().any()


def test_gemm_one_hot_reads_weights(gu):
    """Identity activations read single weights back: pins operand layout and k order."""
    W = inputs.gaussian_weights(64, 64, 14)
    A = np.zeros((64, 64), dtype=np.uint16)
    A[np.arange(64), np.arange(64)] = 0x3F80
    C = gu.gpu_gemm(W, A)
    assert np.array_equal(C, inputs.bf16_to_f32(W).T)


def test_gemm_config1_full(gu):
    """Config 1: 4096 x 4096 N(0, 0.02), M = 8, every output element against the oracle."""
    W = inputs.gaussian_weights(4096, 4096, inputs.seed_for(1))
    A = inputs.activations(8, 4096, inputs.seed_for(1, 0, 1))
    gu.check_gemm(W, A)


def test_dense_gemm_matches_oracle(gu):
    """zs_dense_gemm (hipBLASLt on uncompressed weights): every algorithm the heuristic offers."""
    import torch
    for (M, N, K) in ((5, 192, 320), (130, 256, 512)):
        W = inputs.gaussian_weights(N, K, 60 + M)
        A = inputs.activations(M, K, 61 + M)
        C_ref, S = oracle.gemm(A, W)
        w = torch.from_numpy(W.view(np.int16)).cuda()
        a = torch.from_numpy(A.view(np.int16)).cuda()
        ws = torch.empty(binding.ZS_DENSE_WORKSPACE_BYTES, dtype=torch.uint8, device="cuda")
        n = binding.zs_dense_gemm_algos(M, N, K, ws.numel())
        assert n >= 1
        for algo in range(min(n, 4)):
            c = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
            binding.zs_dense_gemm(a, w, c, M, N, K, workspace_dev=ws, workspace_bytes=ws.numel(), algo=algo)
            torch.cuda.synchronize()
            gu.assert_gemm_matches(c.cpu().numpy(), C_ref, S)
        with pytest.raises(binding.ZsError):
            binding.zs_dense_gemm(a, w, c, M, N, K, algo=99)


@pytest.mark.parametrize("kind", ["gauss", "rowscale"])
def test_linear_both_sides_of_the_crossover(gu, kind):
    """zs_linear against the oracle for token counts on both sides of the switch from the fused
    kernels to zs_decompress + dense GEMM (Section 4.4), through one workspace."""
    import torch
    W = inputs.make_weights(kind, 320, 448, seed=70)
    blob, d = binding.zs_encode(W)
    dev = gu.upload_blob(blob)
    W_dec = oracle.decode(oracle.encode(W))
    Ms = (1, 32, 100, 127, 128, 129, 300)  # a small layer: the decoupled pipeline takes over at 128 tokens
    ws = torch.zeros(max(binding.zs_linear_workspace(d, M) for M in Ms), dtype=torch.uint8, device="cuda")
    paths = set()
    for M in Ms:
        A = inputs.activations(M, 448, 71 + M)
        a = torch.from_numpy(A.view(np.int16)).cuda()
        c = torch.full((M, 320), float("nan"), dtype=torch.float32, device="cuda")
        paths.add(binding.zs_linear_path(d, M))
        if binding.zs_linear_path(d, M) == binding.ZS_PATH_FUSED:
            ws.zero_()  # the fused path wants its scratch all zero; the decoupled one scribbles over it
        binding.zs_linear(d, dev, a, c, M, workspace_dev=ws, workspace_bytes=ws.numel())
        torch.cuda.synchronize()
        C_ref, S = oracle.gemm(A, W_dec)
        gu.assert_gemm_matches(c.cpu().numpy(), C_ref, S)
    assert paths == {binding.ZS_PATH_FUSED, binding.ZS_PATH_DECOUPLED}
    # the decoupled path needs its workspace
    a = torch.zeros((200, 448), dtype=torch.int16, device="cuda")
    c = torch.zeros((200, 320), dtype=torch.float32, device="cuda")
    with pytest.raises(binding.ZsError):
        binding.zs_linear(d, dev, a, c, 200, workspace_dev=ws, workspace_bytes=1024)
    with pytest.raises(binding.ZsError):
        binding.zs_linear(d, dev, a, c, 200, workspace_dev=None, workspace_bytes=0)


def desc_fields(d):
    return {name: getattr(d, name) for name, _ in binding.ZsDesc._fields_}


@pytest.mark.parametrize("kind,N,K,pad", [("gauss", 64, 64, 0), ("gauss", 320, 448, 0), ("rowscale", 192, 128, 8),
                                          ("specials", 256, 256, 0), ("student_t", 128, 256, 24), ("outliers", 448, 320, 0),
                                          ("patterns", 256, 256, 0), ("allfallback", 128, 128, 0)])
def test_encode_device_equals_host_encoder(kind, N, K, pad):
    """zs_encode_device writes the blob zs_encode writes, byte for byte, and the same descriptor
    (the host packer is itself pinned to the oracle's arrays); memory beyond the blob stays untouched."""
    import torch
    if kind == "patterns":
        W = np.random.default_rng(3).permutation(np.arange(65536, dtype=np.uint16)).reshape(256, 256)
    elif kind == "allfallback":  # exponents spread so that no window holds more than a few elements
        W = ((np.arange(N * K, dtype=np.uint32) * 37 % 256) << 7).astype(np.uint16).reshape(N, K)
    else:
        W = inputs.make_weights(kind, N, K, seed=90)
    blob, d = binding.zs_encode(W)
    host = np.zeros((N, K + pad), dtype=np.uint16)
    host[:, :K] = W
    host[:, K:] = 0x7FC0  # never read
    w_dev = torch.from_numpy(host.view(np.int16)).cuda()
    cap = binding.zs_encode_bound(N, K)
    out = torch.full((cap + 512,), 0xA5, dtype=torch.uint8, device="cuda")
    ws = torch.full((binding.ZS_ENCODE_WORKSPACE_BYTES,), 0xFF, dtype=torch.uint8, device="cuda")
    d_dev = binding.zs_encode_device(w_dev, N, K, out, cap, ws, ldw=K + pad)
    torch.cuda.synchronize()
    assert desc_fields(d_dev) == desc_fields(d)
    got = out.cpu().numpy()
    assert np.array_equal(got[:d.total_bytes], blob)
    assert (got[d.total_bytes:] == 0xA5).all()
    assert binding.zs_desc_validate(d_dev) == 0
    with pytest.raises(binding.ZsError):
        binding.zs_encode_device(w_dev, N, K, out, cap - 1, ws, ldw=K + pad)


@pytest.mark.parametrize("n_threads", [3, 20])
def test_encode_device_from_threads(n_threads):
    """Calls under way at the same time, each on its own thread and stream, get their own totals: fewer than there are slots of
    pinned memory for them, and more.  (Whether more than sixteen meet is up to the threads; that those beyond copy is what
    tests/test_encode_host.py makes happen.)"""
    import threading

    import torch
    shapes = [(64 * (1 + t % 5), 64 * (1 + t % 3)) for t in range(n_threads)]
    kinds = ["gauss", "student_t", "rowscale"]
    W = [inputs.make_weights(kinds[t % 3], *shapes[t], seed=200 + t) for t in range(n_threads)]
    w_dev = [torch.from_numpy(w.view(np.int16)).cuda() for w in W]
    torch.cuda.synchronize()
    got, start = [None] * n_threads, threading.Barrier(n_threads, timeout=60)

    def work(t):
        N, K = shapes[t]
        cap, stream = binding.zs_encode_bound(N, K), torch.cuda.Stream()
        with torch.cuda.stream(stream):
            out = torch.empty(cap, dtype=torch.uint8, device="cuda")
            ws = torch.empty(binding.ZS_ENCODE_WORKSPACE_BYTES, dtype=torch.uint8, device="cuda")
            start.wait()
            results = []
            for _ in range(8):
                d = binding.zs_encode_device(w_dev[t], N, K, out, cap, ws, stream=stream.cuda_stream)
                results.append((desc_fields(d), out[:d.total_bytes].cpu().numpy()))
        got[t] = results

    threads = [threading.Thread(target=work, args=(t,)) for t in range(n_threads)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    for t in range(n_threads):
        blob, d = binding.zs_encode(W[t])
        assert got[t] is not None
        for fields, b in got[t]:
            assert fields == desc_fields(d) and np.array_equal(b, blob)


@pytest.mark.parametrize("M", [1, 16, 31, 64, 150])
def test_gemm_bf16_output(gu, M):
    """zs_gemm_bf16: the FP32 result rounded once to BF16.  Bound per element: the GEMM tolerance
    plus half a BF16 unit in the last place of the reference (2^-9 relative, taken as 2^-8 to
    cover a result that the FP32 error moved across a rounding boundary)."""
    import torch
    W = inputs.make_weights("rowscale", 320, 448, seed=80)  # 5 strips x 7 BlockTiles: shared strips at any workgroup count
    A = inputs.activations(M, 448, 81 + M)
    blob, d = binding.zs_encode(W)
    dev = gu.upload_blob(blob)
    C_ref, S = oracle.gemm(A, oracle.decode(oracle.encode(W)))
    a = torch.from_numpy(A.view(np.int16)).cuda()
    need = binding.zs_gemm_workspace(d, min(M, 64))
    ws = torch.zeros(max(need, 256), dtype=torch.uint8, device="cuda")
    ldc = 324  # a row stride wider than N
    for rep in range(2):  # the second call reuses the scratch the first one left
        c = torch.full((M, ldc), 0x7FC1, dtype=torch.int16, device="cuda")
        binding.zs_gemm_bf16(d, dev, a, c, M, ldc=ldc, workspace_dev=ws, workspace_bytes=ws.numel())
        torch.cuda.synchronize()
        out = c.cpu().numpy().view(np.uint16)
        assert (out[:, 320:] == 0x7FC1).all()  # nothing written beyond N
        got = inputs.bf16_to_f32(out[:, :320]).astype(np.float64)
        bound = 1e-3 * S + 1e-6 + 2.0 ** -8 * np.abs(C_ref)
        assert (np.abs(got - C_ref) <= bound).all()
        # and it is the rounding of an FP32 result within the GEMM tolerance: at most one BF16 step from RNE(reference)
        ref16 = inputs.f32_to_bf16(C_ref.astype(np.float32)).astype(np.int64)
        near = np.abs(C_ref) > 64 * (1e-3 * S + 1e-6)  # where the GEMM tolerance is far below a BF16 step
        assert (np.abs(out[:, :320].astype(np.int64) - ref16)[near] <= 1).all()
    if need:
        with pytest.raises(binding.ZsError):
            binding.zs_gemm_bf16(d, dev, a, c, M, ldc=ldc, workspace_dev=None, workspace_bytes=0)


def test_gemm_strided_operands(gu):
    import torch
    W = inputs.gaussian_weights(128, 192, 15)
    A = inputs.activations(5, 192, 16)
    blob, d = binding.zs_encode(W)
    dev = gu.upload_blob(blob)
    a = torch.zeros((5, 256), dtype=torch.int16, device="cuda")
    a[:, :192] = torch.from_numpy(A.view(np.int16)).cuda()
    c = torch.full((5, 160), 7.0, dtype=torch.float32, device="cuda")
    binding.zs_gemm(d, dev, a, c, 5, lda=256, ldc=160)
    torch.cuda.synchronize()
    C_ref, S = oracle.gemm(A, W)
    out = c.cpu().numpy()
    gu.assert_gemm_matches(out[:, :128], C_ref, S)
    assert (out[:, 128:] == 7.0).all()


@pytest.mark.parametrize("M", [66, 128, 200, 256, 300])
@pytest.mark.parametrize("wgs", [0, 1, 3])
def test_gemm_shared_decode_strided_operands(gu, wgs, M):
    """Row strides wider than the rows for the producer / consumer kernel, whole strips (one workgroup)
    and shared ones; what lies between the rows is neither used nor written."""
    import torch
    N, K, lda, ldc = 192, 320, 376, 212
    W, A = inputs.gaussian_weights(N, K, 18), inputs.activations(M, K, 19 + M)
    blob, d = binding.zs_encode(W)
    a = torch.full((M, lda), 0x7FC0, dtype=torch.int16, device="cuda")    # NaN between the rows
    a[:, :K] = torch.from_numpy(A.view(np.int16)).cuda()
    c = torch.full((M, ldc), 7.0, dtype=torch.float32, device="cuda")
    binding.zs_gemm(d, gu.upload_blob(blob), a, c, M, lda=lda, ldc=ldc, config=binding.zs_gemm_pick_config(d, M) + 256 * wgs)
    C_ref, S = oracle.gemm(A, W)
    out = c.cpu().numpy()
    gu.assert_gemm_matches(out[:, :N], C_ref, S)
    assert (out[:, N:] == 7.0).all()


def test_error_paths(gu):
    import torch
    W = inputs.gaussian_weights(64, 64, 17)
    blob, d = binding.zs_encode(W)
    dev = gu.upload_blob(blob)
    a = torch.zeros((4, 64), dtype=torch.int16, device="cuda")
    c = torch.zeros((4, 64), dtype=torch.float32, device="cuda")
    assert binding.zs_gemm_workspace(d, 4) > 0      # shared-strip sums of the skinny kernel
    assert binding.zs_gemm_workspace(d, 100) == 0   # the producer / consumer kernel uses none
    kw = dict(workspace_dev=None, workspace_bytes=0)  # scratch is optional
    binding.zs_gemm(d, dev, a, c, 4, **kw)
    with pytest.raises(binding.ZsError):
        binding.zs_gemm(d, dev, a, c, 0, **kw)
    with pytest.raises(binding.ZsError):
        binding.zs_gemm(d, dev, a, c, 4, config=99, **kw)
    with pytest.raises(binding.ZsError):
        binding.zs_gemm(d, dev.data_ptr() + 16, a, c, 4, **kw)
    with pytest.raises(binding.ZsError):
        binding.zs_gemm(d, dev, a, c, 4, lda=32, **kw)
    with pytest.raises(binding.ZsError):
        binding.zs_decompress(d, dev, None)


@pytest.mark.parametrize("strips,k_blocks", [(63, 65), (64, 64), (17, 241), (3, 2731)])
def test_encode_device_scan_workgroups(strips, k_blocks):
    """Numbers of BlockTiles around a workgroup's share of the prefix sum: 4095, 4096, 4097, 8193."""
    import torch
    N, K = 64 * strips, 64 * k_blocks
    W = inputs.make_weights("student_t", N, K, seed=92)
    blob, d = binding.zs_encode(W)
    cap = binding.zs_encode_bound(N, K)
    out = torch.full((cap,), 0xA5, dtype=torch.uint8, device="cuda")
    ws = torch.full((binding.ZS_ENCODE_WORKSPACE_BYTES,), 0xFF, dtype=torch.uint8, device="cuda")
    d_dev = binding.zs_encode_device(torch.from_numpy(W.view(np.int16)).cuda(), N, K, out, cap, ws)
    assert desc_fields(d_dev) == desc_fields(d)
    assert np.array_equal(out.cpu().numpy()[:d.total_bytes], blob)


def tied_windows(N, K):
    """Exponents 100..115 in equal shares: every window inside covers the same, the smallest start
    wins, and a prediction from a part of the weights has no reason to agree.  (Every BlockTile holds the
    same number of weights in any of them: the counts that a wrong prediction left are right by chance.)"""
    return (((np.arange(N * K, dtype=np.uint32) % 16 + 100) << 7) | (np.arange(N * K, dtype=np.uint32) // 16 % 128)).astype(np.uint16).reshape(N, K)


@pytest.mark.parametrize("kind,N,K", [("tied", 128, 192), ("tied", 1024, 1088), ("gauss", 192, 64 * 2732), ("student_t", 64, 576)])
def test_encode_device_prediction_and_scan_edges(kind, N, K):
    """Tied windows, and numbers of BlockTiles that leave a part of a thread's four in the prefix sum: 8196
    (two workgroups of 4096 and one thread of a third) and 9 (two threads and a quarter of one)."""
    import torch
    W = tied_windows(N, K) if kind == "tied" else inputs.make_weights(kind, N, K, seed=91)
    blob, d = binding.zs_encode(W)
    assert kind != "tied" or d.base_exp == 99
    cap = binding.zs_encode_bound(N, K)
    out = torch.full((cap,), 0xA5, dtype=torch.uint8, device="cuda")
    ws = torch.full((binding.ZS_ENCODE_WORKSPACE_BYTES,), 0xFF, dtype=torch.uint8, device="cuda")
    d_dev = binding.zs_encode_device(torch.from_numpy(W.view(np.int16)).cuda(), N, K, out, cap, ws)
    assert desc_fields(d_dev) == desc_fields(d)
    got = out.cpu().numpy()
    assert np.array_equal(got[:d.total_bytes], blob)
    assert (got[d.total_bytes:] == 0xA5).all()


def sampled_units(N, K):
    """The 16-byte units of a row-major N x K matrix that the GPU packer predicts the window from."""
    h = np.arange(2048, dtype=np.uint64) * 0x9E3779B1 & 0xFFFFFFFF
    return (h * np.uint64(N * K // 8) >> np.uint64(32)).astype(np.int64)


def best_window(exponents):
    hist = np.bincount(exponents.ravel(), minlength=256)
    return int(np.argmax(np.convolve(hist, np.ones(7, dtype=np.int64), "valid")))   # the first maximum


@pytest.mark.parametrize("strips,k_blocks,a_strips", [(4, 4, 3), (16, 17, 9), (92, 90, 50)])
def test_encode_device_wrong_prediction(strips, k_blocks, a_strips):
    """Most strips hold exponents 100..106, the others and every sampled unit 110..116, and a tenth of all
    weights lie outside both: the predicted window is 110, the right one 100, and with the one's counts a
    BlockTile's segments would have the other's sizes.  92 x 90 BlockTiles are more than the waves of
    a pass over them (16 in each of two workgroups on 256 compute units)."""
    import torch
    N, K = 64 * strips, 64 * k_blocks
    rng = np.random.default_rng(93)
    base = np.full((N, K), 110, dtype=np.uint16)
    base[:64 * a_strips] = 100
    base.reshape(-1, 8)[sampled_units(N, K)] = 110
    exponent = base + rng.integers(0, 7, (N, K), dtype=np.uint16)
    exponent[rng.random((N, K)) < 0.1] = 200
    W = (exponent << 7 | rng.integers(0, 2, (N, K), dtype=np.uint16) << 15 | rng.integers(0, 128, (N, K), dtype=np.uint16)).astype(np.uint16)
    assert best_window(exponent.reshape(-1, 8)[sampled_units(N, K)]) == 110 and best_window(exponent) == 100
    tiles = exponent.reshape(strips, 64, k_blocks, 64)
    units = [-(-((tiles >= lo) & (tiles < lo + 7)).sum((1, 3)) // 16) for lo in (100, 110)]
    assert (units[0] != units[1]).mean() > 0.9
    blob, d = binding.zs_encode(W)
    assert d.base_exp == 99
    cap = binding.zs_encode_bound(N, K)
    out = torch.full((cap,), 0xA5, dtype=torch.uint8, device="cuda")
    ws = torch.full((binding.ZS_ENCODE_WORKSPACE_BYTES,), 0xFF, dtype=torch.uint8, device="cuda")
    d_dev = binding.zs_encode_device(torch.from_numpy(W.view(np.int16)).cuda(), N, K, out, cap, ws)
    assert desc_fields(d_dev) == desc_fields(d)
    assert np.array_equal(out.cpu().numpy()[:d.total_bytes], blob)
