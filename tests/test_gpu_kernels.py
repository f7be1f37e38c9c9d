"""GPU parity of single kernels through the C ABI: the bf16 MFMA GEMM against a float64 matmul of
the same bf16 values (several tile shapes, ragged tails), and the plain f32 GEMM."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _rand_bf16(shape, seed, std=1.0):
    a = np.empty(int(np.prod(shape)), dtype=np.uint16)
    synth.weights.fill_normal(a, seed, 77, std=std)
    return a.reshape(shape)


# row counts that land on every accumulator height of the MFMA kernel (32 ... 256 rows, with ragged
# last 16-row tiles), column counts off the 256 grid, K of one slab; (50, 30, 64) has a column count
# that is not a multiple of 4 and takes the plain kernel
@pytest.mark.parametrize("M,N,K", [(256, 256, 64), (2304, 512, 256), (300, 1000, 128), (1, 256, 4096),
                                   (129, 384, 192), (577, 256, 1024), (64, 32000, 256),
                                   (17, 260, 128), (33, 256, 128), (95, 256, 192), (161, 516, 128),
                                   (224, 256, 128), (255, 256, 128), (257, 256, 128), (513, 772, 256),
                                   (700, 256, 128), (4608, 256, 64), (50, 30, 64)])
def test_gemm_bf16_mfma(M, N, K):
    import torch
    import paper_2505_10259_amd as P
    from gpu_common import dev
    A = _rand_bf16((M, K), 1)
    W = _rand_bf16((N, K), 2, std=0.05)
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    P.spec_gemm(dev(A), dev(W), C, M, N, K, P.SPEC_BF16)
    torch.cuda.synchronize()
    ref = synth.bf16_bits_to_f32(A).astype(np.float64) @ synth.bf16_bits_to_f32(W).astype(np.float64).T
    got = C.cpu().numpy()
    assert np.isfinite(got).all()
    scale = np.sqrt(K) * 0.05
    assert np.abs(got - ref).max() < 2e-5 * scale * 10, np.abs(got - ref).max()
    # and the plain kernel agrees too
    C2 = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    P.spec_gemm(dev(A), dev(W), C2, M, N, K, P.SPEC_BF16, P.SPEC_FLAG_SIMPLE_KERNELS)
    torch.cuda.synchronize()
    assert np.abs(C2.cpu().numpy() - ref).max() < 2e-5 * scale * 10


@pytest.mark.parametrize("tile_cols", [128, 256])
@pytest.mark.parametrize("tile_rows", [32, 64, 96, 128, 160, 192, 224, 256])
def test_gemm_bf16_mfma_every_tile_variant(tile_rows, tile_cols):
    """Every accumulator height of the MFMA kernel at both tile widths (the launcher's own choice visits
    only some of the combinations at any given shape): two full row tiles and a ragged third, a column
    count off the tile grid, K long enough for the steady-state loop and its tail."""
    import torch
    import paper_2505_10259_amd as P
    from gpu_common import dev
    M, N, K = 2 * tile_rows + 17, 3 * tile_cols // 2 + 20, 1152
    A = _rand_bf16((M, K), 3)
    W = _rand_bf16((N, K), 4, std=0.05)
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    P.spec_debug_gemm(dev(A), dev(W), C, M, N, K, tile_rows, tile_cols)
    torch.cuda.synchronize()
    ref = synth.bf16_bits_to_f32(A).astype(np.float64) @ synth.bf16_bits_to_f32(W).astype(np.float64).T
    got = C.cpu().numpy()
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() < 2e-4 * np.sqrt(K) * 0.05, np.abs(got - ref).max()


# products whose own tiles are narrower than 256 columns (32, 64 and 128 columns; one row tile and several; a
# ragged last row and column tile; as many slabs as stages, fewer, more) and, the last two, 256-column tiles
@pytest.mark.parametrize("M,N,K", [(1, 4096, 64), (5, 4096, 1024), (33, 6144, 512), (33, 4100, 1088), (64, 2048, 2048),
                                   (100, 4096, 320), (128, 6144, 1152), (230, 4096, 960), (320, 6144, 256),
                                   (513, 4096, 448), (900, 8192, 128), (2304, 4096, 128), (40, 65536, 64)])
def test_gemm_bf16_tile_choice_changes_no_bit(M, N, K):
    """Every output is one sum over K in ascending order whatever the tiles: the launcher's choice and forced
    256-column tiles agree bit for bit (and the forced ones are checked against float64 above)."""
    import torch
    import paper_2505_10259_amd as P
    from gpu_common import dev
    A, W = dev(_rand_bf16((M, K), 5)), dev(_rand_bf16((N, K), 6, std=0.05))
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    D = torch.zeros_like(C)
    P.spec_gemm(A, W, C, M, N, K, P.SPEC_BF16)
    P.spec_debug_gemm(A, W, D, M, N, K, 256, 256)
    torch.cuda.synchronize()
    assert torch.equal(C, D)
    rows = slice(0, min(M, 64))
    ref = A.view(torch.bfloat16)[rows].double() @ W.view(torch.bfloat16).double().t()
    # f32 sums of K products: error below K * 2^-24 of the sum of magnitudes, far less for random signs
    assert ((C[rows].double() - ref).abs().max() < 2e-4 * np.sqrt(K) * 0.05).item()


# heights of one, three, five and eight 32-row units; contractions of one slab, two, one short of a tile's LDS stages, as
# many, one more, and two rounds of them and one
@pytest.mark.parametrize("tile_rows", [32, 96, 160, 256])
@pytest.mark.parametrize("epilogue,tile_cols", [("add", 32), ("add", 64), ("add", 128), ("store", 32), ("store", 64), ("store", 128),
                                                ("swiglu", 128)])
def test_gemm_narrow_tiles_with_every_epilogue_change_no_bit(tile_rows, epilogue, tile_cols):
    """Narrow tiles at ragged rows and columns against 256-column tiles, bit for bit, and those against float64."""
    import torch
    import paper_2505_10259_amd as P
    epi = {"store": P.SPEC_GEMM_STORE, "add": P.SPEC_GEMM_ADD, "swiglu": P.SPEC_GEMM_SWIGLU}[epilogue]
    g = torch.Generator("cuda").manual_seed(tile_rows + tile_cols)
    mi, ni = tile_rows // 32, tile_cols // 32
    stages = min(16, max(3, 160 * 1024 // ((32 * mi + 32 * ni) * 128)))
    for slabs in sorted({1, 2, stages - 1, stages, stages + 1, 2 * stages + 1}):
        M, N, K = 2 * tile_rows + 17, 2 * 256 + tile_cols // 2 + 12, 64 * slabs
        A = torch.randn(M, K, device="cuda", generator=g).bfloat16()
        W = (torch.randn(2, N, K, device="cuda", generator=g) * 0.05).bfloat16()
        W3 = W[1] if epilogue == "swiglu" else None
        out = []
        for rows, cols in ((tile_rows, tile_cols), (256, 256)):
            C = torch.full((M, N), 0.25, device="cuda", dtype=torch.bfloat16 if epilogue == "swiglu" else torch.float32)
            P.spec_debug_gemm_epilogue(A, W[0], W3, C, None, 0, M, N, K, epi, rows, cols)
            torch.cuda.synchronize()
            out.append(C)
        assert torch.equal(out[0], out[1]), slabs
        x = A.double() @ W[0].double().t()
        if epilogue == "swiglu":
            x = torch.nn.functional.silu(x) * (A.double() @ W[1].double().t())
            assert ((out[1].double() - x).abs() <= 2.0 ** -8 * x.abs() + 2e-4 * np.sqrt(K)).all()       # one bf16 rounding
        else:
            x = x + (0.25 if epilogue == "add" else 0.0)
            # f32 sums of K products: error below K * 2^-24 of the sum of magnitudes, far less for random signs
            assert (out[1].double() - x).abs().max().item() < 2e-4 * np.sqrt(K) * 0.05 + 2.0 ** -22


# few rows that reach few of the groups: narrower tiles than for all groups
@pytest.mark.parametrize("epilogue", ["store", "swiglu"])
@pytest.mark.parametrize("sizes", [(0, 1, 0, 0, 0, 0, 0, 1), (1, 0, 0, 1, 0, 2, 0, 0), (0, 0, 0, 3, 0, 0, 0, 3), (2, 1, 1, 0, 2, 0, 1, 1)])
def test_gemm_few_live_groups_change_no_bit(epilogue, sizes):
    import torch
    import paper_2505_10259_amd as P
    epi = {"store": P.SPEC_GEMM_STORE, "swiglu": P.SPEC_GEMM_SWIGLU}[epilogue]
    g = torch.Generator("cuda").manual_seed(sum(sizes))
    N, M, K, G = 4096 + 40, sum(sizes), 320, len(sizes)
    A = torch.randn(M, K, device="cuda", generator=g).bfloat16()
    W = (torch.randn(2, G, N, K, device="cuda", generator=g) * 0.05).bfloat16()
    W3 = W[1] if epilogue == "swiglu" else None
    off = torch.tensor([0] + list(np.cumsum(sizes)), dtype=torch.int32, device="cuda")
    C = torch.full((M, N), 0.25, device="cuda", dtype=torch.bfloat16 if epilogue == "swiglu" else torch.float32)
    D = C.clone()
    P.spec_debug_gemm_epilogue(A, W[0], W3, C, off, G, M, N, K, epi, 0, 0)
    b = 0
    for i, n in enumerate(sizes):
        if n:
            P.spec_debug_gemm_epilogue(A[b:b + n], W[0, i], W[1, i] if W3 is not None else None, D[b:b + n], None, 0, n, N, K, epi, 256, 256)
        b += n
    torch.cuda.synchronize()
    assert torch.equal(C, D)


# 36 column tiles for each of the groups that have rows: an XCD's list is longer than its 32 units by a few tiles, which are cut
# into column halves where one row tile reads the weights; the last column tile is ragged on either side of its middle
@pytest.mark.parametrize("epilogue", ["store", "add", "swiglu"])
@pytest.mark.parametrize("short_by", [32, 160])
@pytest.mark.parametrize("sizes", [(80, 80, 80, 80, 80, 80, 80, 80), (5, 128, 0, 97, 64, 17, 33, 96),
                                   (131, 110, 128, 97, 125, 140, 118, 127)])
def test_gemm_column_halves_change_no_bit(epilogue, short_by, sizes):
    """Groups of at most 128 rows (some without any) in one launch against every group by itself; groups on either side of
    128 rows as the launcher cuts them."""
    import torch
    import paper_2505_10259_amd as P
    epi = {"store": P.SPEC_GEMM_STORE, "add": P.SPEC_GEMM_ADD, "swiglu": P.SPEC_GEMM_SWIGLU}[epilogue]
    g = torch.Generator("cuda").manual_seed(short_by)
    live = sum(1 for n in sizes if n)
    cols = 128 if epilogue == "swiglu" else 256                # outputs per tile
    N = -(-36 * 8 // live) * cols - (short_by // 2 if epilogue == "swiglu" else short_by)
    M, K, G = sum(sizes), 192, len(sizes)
    A = torch.randn(M, K, device="cuda", generator=g).bfloat16()
    W = (torch.randn(2, G, N, K, device="cuda", generator=g) * 0.05).bfloat16()
    W3 = W[1] if epilogue == "swiglu" else None
    off = torch.tensor([0] + list(np.cumsum(sizes)), dtype=torch.int32, device="cuda")
    C = torch.full((M, N), 0.25, device="cuda", dtype=torch.bfloat16 if epilogue == "swiglu" else torch.float32)
    D = C.clone()
    forced = (128, 256) if max(sizes) <= 128 else (0, 0)
    P.spec_debug_gemm_epilogue(A, W[0], W3, C, off, G, M, N, K, epi, *forced)
    b = 0
    for i, n in enumerate(sizes):
        if n:
            P.spec_debug_gemm_epilogue(A[b:b + n], W[0, i], W[1, i] if W3 is not None else None, D[b:b + n], None, 0, n, N, K, epi, 256, 256)
        b += n
    torch.cuda.synchronize()
    assert torch.equal(C, D)


# panels of 4 rows (K up to 4096) and of 8, one to two hundred slabs, ragged column tiles; sizes that stay as rows
@pytest.mark.parametrize("epilogue", ["store", "add", "swiglu"])
@pytest.mark.parametrize("N,K,rows", [(8, 64, 4), (264, 1024, 4), (520, 4096, 4), (136, 4160, 8), (40, 16384, 8), (36, 256, 1),
                                      (64, 16448, 1)])
def test_gemm_weight_panels_change_no_bit(epilogue, N, K, rows):
    """Weights turned into panels: the matrix itself against the layout written out, and the products against those of the rows."""
    import torch
    import paper_2505_10259_amd as P
    G, sizes = 3, [5, 0, 70]
    epi = {"store": P.SPEC_GEMM_STORE, "add": P.SPEC_GEMM_ADD, "swiglu": P.SPEC_GEMM_SWIGLU}[epilogue]
    g = torch.Generator("cuda").manual_seed(N + K)
    W = (torch.randn(2, G, N, K, device="cuda", generator=g) * 0.05).bfloat16()
    A = torch.randn(sum(sizes), K, device="cuda", generator=g).bfloat16()
    off = torch.tensor(np.cumsum([0] + sizes), dtype=torch.int32, device="cuda")
    V = W.clone()
    for i in range(2):
        for e in range(G):
            assert P.spec_debug_weight_panels(V[i, e], N, K) == rows
    torch.cuda.synchronize()
    if rows > 1:
        assert torch.equal(V.reshape(2, G, N // rows, K // 64, rows, 64), W.reshape(2, G, N // rows, rows, K // 64, 64).transpose(4, 3))
    else:
        assert torch.equal(V, W)

    def call(groups, plain, panels):
        C = torch.full((len(A), N), 0.25, device="cuda", dtype=torch.bfloat16 if epilogue == "swiglu" else torch.float32)
        w = V if panels else W
        w = w if groups else w[:, 2]
        args = (A, w[0], w[1] if epilogue == "swiglu" else None, C, off if groups else None, G if groups else 0, len(A), N, K, epi)
        if panels:
            P.spec_debug_gemm_panels(*args, plain)
        else:
            P.spec_debug_gemm_epilogue(*args, 0, 0)
        torch.cuda.synchronize()
        return C

    for groups in (False, True):
        rows_out = call(groups, 0, False)
        assert torch.equal(call(groups, 0, True), rows_out)
        plain = call(groups, 1, True).float()
        # the plain kernel sums in another order: K products of about 0.05 each way, and one bf16 rounding of a SwiGLU result
        tol = 2e-5 * np.sqrt(K) + (2.0 ** -7 * rows_out.float().abs() if epilogue == "swiglu" else 0.0)
        assert ((plain - rows_out.float()).abs() <= tol).all()


@pytest.mark.parametrize("M,N,K", [(5, 4096, 4096), (9, 40, 64), (20, 264, 320), (3, 520, 8256), (64, 8192, 128)])
def test_plain_kernels_on_panels(M, N, K):
    """The plain kernels on panels (a bf16 product onto an output off 16 bytes) have the bits of those on rows, and their tiles: small
    ones where 64 x 64 tiles leave most compute units idle (the first size: 4 to 8 times as fast)."""
    import torch
    import paper_2505_10259_amd as P
    g = torch.Generator("cuda").manual_seed(K)
    A = torch.randn(M + 1, K, device="cuda", generator=g).bfloat16().reshape(-1)
    W = (torch.randn(N, K, device="cuda", generator=g) * 0.05).bfloat16()
    V = W.clone()
    assert P.spec_debug_weight_panels(V, N, K) > 1
    for a in (A[:M * K], A[1:M * K + 1]):                       # operand rows on 16 bytes and off
        C, D = torch.full((M, N), 7.0, device="cuda"), torch.full((M, N), 9.0, device="cuda")
        rows = lambda: P.spec_gemm(a, W, C, M, N, K, P.SPEC_BF16, P.SPEC_FLAG_SIMPLE_KERNELS)
        panels = lambda: P.spec_debug_gemm_panels(a, V, None, D, None, 0, M, N, K, P.SPEC_GEMM_STORE, 1)
        us = []
        for f in (rows, panels):
            best = float("inf")
            for _ in range(3):
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                for _ in range(20):
                    f()
                e1.record()
                e1.synchronize()
                best = min(best, e0.elapsed_time(e1) * 50)
            us.append(best)
        assert torch.equal(C, D)
        assert us[1] < 2.5 * us[0], us


# small plain tiles (8 x 32, steps of 256) with ragged rows, columns and contractions, unaligned rows (K odd), and
# the sizes on either side of the line to the 64 x 64 tiles
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (8, 32, 128), (9, 33, 129), (20, 768, 256), (4, 256, 1024), (7, 100, 255), (3, 40, 257),
                                   (64, 8128, 64), (64, 8192, 64), (65, 4033, 96)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_gemm_plain_small_and_large_tiles(M, N, K, dtype):
    import torch
    import paper_2505_10259_amd as P
    g = torch.Generator("cuda").manual_seed(M + N + K)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    A = torch.randn(M, K, device="cuda", generator=g).to(t)
    W = torch.randn(N, K, device="cuda", generator=g).to(t)
    C = torch.full((M, N), float("nan"), device="cuda")
    P.spec_gemm(A, W, C, M, N, K, P.SPEC_F32 if dtype == "f32" else P.SPEC_BF16, P.SPEC_FLAG_SIMPLE_KERNELS)
    torch.cuda.synchronize()
    ref = A.double() @ W.double().t()
    # a chain of K fused multiply-adds: error at most K * 2^-24 * sum |a w|, about K * E|a w| = 0.64 K
    assert (C.double() - ref).abs().max().item() < max(2, K) * 2.0 ** -24 * 2 * K


# one piece of 4, a tail of less than 16, one block of 256 and on either side of it, three blocks; 1 to 20 rows, ragged columns
@pytest.mark.parametrize("M,N,K", [(1, 16, 4), (20, 48, 100), (16, 40, 256), (17, 33, 264), (4, 64, 600), (20, 100, 1024)])
@pytest.mark.parametrize("values", ["ordinary", "subnormal", "special"])
def test_gemm_f32_same_bits_on_every_kernel(M, N, K, values):
    """f32 products of few tiles run on the matrix cores, which must give the chain of fused multiply-adds of the other kernels bit
    for bit (a prefill's bits may not depend on its group's rows): against 8 x 32 tiles (operands off 16 bytes; the
    plain-kernel flag) and 64 x 64 tiles (the same rows inside a matrix of 8200)."""
    import torch
    import paper_2505_10259_amd as P
    g = torch.Generator("cuda").manual_seed(M * K + N)
    A = torch.randn(8200, K, device="cuda", generator=g)
    W = torch.randn(N, K, device="cuda", generator=g)
    if values == "subnormal":              # operands, products and sums on both sides of 2^-126
        A *= 2.0 ** -70
        A[:, ::2] *= 2.0 ** -62
        W *= 2.0 ** -56
        W[:, ::2] *= 2.0 ** 66
    elif values == "special":
        A[torch.rand(A.shape, device="cuda", generator=g) < 0.3] = -0.0
        W[torch.rand(W.shape, device="cuda", generator=g) < 0.3] = 0.0
        A[0, K // 2] = float("inf")
        if M > 4:
            A[3, 1], W[5, 2], A[1, K - 1] = float("nan"), float("-inf"), 3.0e38

    def call(a, w, rows, flags=0):
        C = torch.full((rows, N), 7.0, device="cuda")
        P.spec_gemm(a, w, C, rows, N, K, P.SPEC_F32, flags)
        torch.cuda.synchronize()
        return C[:M]

    def off(t):
        b = torch.empty(t.numel() + 1, device="cuda")
        b[1:] = t.reshape(-1)
        return b[1:]

    ref = call(A, W, 8200)
    if values == "subnormal":
        assert ((ref != 0) & (ref.abs() < 2.0 ** -126)).any()
    for name, C in (("matrix cores", call(A[:M], W, M)), ("off 16 bytes", call(off(A[:M]), W, M)),
                    ("weights off 16 bytes", call(A[:M], off(W), M)), ("plain", call(A[:M], W, M, P.SPEC_FLAG_SIMPLE_KERNELS))):
        nan = torch.isnan(ref)
        assert torch.equal(torch.isnan(C), nan), name
        assert torch.equal(C.view(torch.int32)[~nan], ref.view(torch.int32)[~nan]), name


# segments of 16 k, empty and ragged ones, pieces of 8 and of 16 on either side of a fold; the three in front of the last are tiles enough for
# one wavefront each (127 of 64 x 64 at most, more than 512 of 16 x 16); the last is 128 of 64 x 64
@pytest.mark.parametrize("M,N,K", [(3, 24, 16), (16, 40, 68), (16, 40, 132), (5, 33, 1028), (20, 64, 2052),
                                   (64, 8064, 260), (64, 8100, 1028), (33, 8100, 2064), (33, 8192, 2064)])
def test_gemm_f32_four_segments(M, N, K):
    """An f32 sum is four chains over consecutive segments of the contraction, added in ascending order, whichever kernel makes it: the
    matrix cores with a wavefront per segment or for all four, 8 x 32 tiles (operands off 16 bytes) and 64 x 64 tiles (the same rows
    inside 1024) agree bit for bit, and the error is that of chains of a quarter of K."""
    import torch
    import paper_2505_10259_amd as P
    g = torch.Generator("cuda").manual_seed(M + N + K)
    A = torch.randn(1024, K, device="cuda", generator=g)
    W = torch.randn(N, K, device="cuda", generator=g)

    def call(a, w, rows):
        C = torch.full((rows, N), 7.0, device="cuda")
        P.spec_gemm(a, w, C, rows, N, K, P.SPEC_F32)
        torch.cuda.synchronize()
        return C[:M]

    off = torch.empty(M * K + 1, device="cuda")
    off[1:] = A[:M].reshape(-1)
    W_all = torch.cat([W, torch.zeros(max(0, 1024 - N), K, device="cuda")])        # (1024 rows and columns are 256 tiles of 64 x 64)
    C_all = torch.empty(1024, W_all.shape[0], device="cuda")
    P.spec_gemm(A, W_all, C_all, 1024, W_all.shape[0], K, P.SPEC_F32)
    torch.cuda.synchronize()
    ref = C_all[:M, :N]
    assert torch.equal(call(A[:M], W, M), ref)
    assert torch.equal(call(off[1:], W, M), ref)
    seg = (K + 63) // 64 * 16
    terms = A[:M].double().abs() @ W.double().abs().t()
    # a segment's chain rounds seg times, the sum of four three times more
    assert ((ref.double() - A[:M].double() @ W.double().t()).abs() <= 1.01 * (seg + 3) * 2.0 ** -24 * terms).all()


def test_gemm_f32_plain():
    import torch
    import paper_2505_10259_amd as P
    from gpu_common import dev
    rng = np.random.default_rng(0)
    M, N, K = 70, 130, 100
    A = rng.standard_normal((M, K)).astype(np.float32)
    W = rng.standard_normal((N, K)).astype(np.float32)
    C = torch.zeros((M, N), dtype=torch.float32, device="cuda")
    P.spec_gemm(dev(A), dev(W), C, M, N, K, P.SPEC_F32)
    torch.cuda.synchronize()
    assert np.abs(C.cpu().numpy() - A.astype(np.float64) @ W.astype(np.float64).T).max() < 1e-4
