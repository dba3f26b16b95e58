"""The GEMMs at the sizes where their tiles change, against float64 products of the same operands.  Bound per element: one
rounding of the result to its type plus K roundings of float on the sum of the absolute products."""
import pytest
import torch

from paper_2603_05035_amd import binding as g

pytestmark = pytest.mark.gpu


def check(m, k, n, dtype):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + 7 * k + 31 * n)
    U = torch.randn((m, k), generator=gen, device="cuda").to(dtype)
    W = torch.randn((k, n), generator=gen, device="cuda").to(dtype)
    Y = torch.full((m + 2, n), float("nan"), device="cuda", dtype=dtype)
    ctx = g.gelo_create(0, 1)
    g.gelo_project(ctx, U, W, Y[1:m + 1])
    torch.cuda.synchronize()
    g.gelo_destroy(ctx)
    assert torch.isnan(Y[0]).all() and torch.isnan(Y[-1]).all()
    ref, size = U.double() @ W.double(), U.double().abs() @ W.double().abs()
    # rounding to nearest with p significant bits errs by at most 2^-p of the value; bfloat16 has 8 (7 stored), float 24
    half_unit = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -24
    assert bool(((Y[1:m + 1].double() - ref).abs() <= half_unit * 1.01 * ref.abs() + k * 2.0 ** -24 * size).all())


# whole 256-row tiles and up to 128 rows more: those as tiles of 128 rows behind wide, narrow or both kinds of whole tiles
# (1, 102 and 128 rows left), 129 left (a whole tile again); widths that fill no tile
@pytest.mark.parametrize("m,n", [(2150, 22016), (2049, 22008), (2176, 21768), (2177, 22016), (2150, 12288), (384, 49152), (257, 33800),
                                 (1100, 16392), (1152, 11008), (4301, 12288), (640, 22016)])
@pytest.mark.parametrize("k", [64, 192])
def test_bf16_rows_behind_the_last_whole_tile(m, n, k):
    check(m, k, n, torch.bfloat16)



# the same rows in mix and un-mix: B in two segments (data rows, then shield rows) that meet inside a K step, and a K that fills no
# step (572 + 28 rows: 600 = 9 x 64 + 24).  The operands are the library's own, read back: A and A^-1 rounded as it rounds them,
# the shield rows as they are stored
@pytest.mark.parametrize("width", [16384, 22016])
def test_bf16_rows_behind_the_last_whole_tile_of_a_mix(width):
    n_data, k = 572, 28
    n = n_data + k
    gen = torch.Generator(device="cuda")
    gen.manual_seed(width)
    H = torch.randn((n_data, width), generator=gen, device="cuda").to(torch.bfloat16)
    Y = torch.randn((n, width), generator=gen, device="cuda").to(torch.bfloat16)
    U, Z = torch.full((n + 2, width), float("nan"), device="cuda", dtype=torch.bfloat16), torch.full((n_data + 2, width), float("nan"), device="cuda", dtype=torch.bfloat16)
    ctx = g.gelo_create(0, 1)
    m = g.gelo_sample_mixing(ctx, g.GELO_REFLECTOR_PRODUCT, n_data, k, width, g.GELO_BF16, batch_id=1)
    g.gelo_mix(ctx, m, H, U[1:n + 1])
    g.gelo_unmix(ctx, m, Y, Z[1:n_data + 1])
    A, A_inv, S, _, _ = g.gelo_mixing_export(ctx, m, n, k, width)
    torch.cuda.synchronize()
    g.gelo_mixing_free(ctx, m)
    g.gelo_destroy(ctx)
    for out, rows, left, right in ((U, n, A, torch.cat([H.double(), S.double()])), (Z, n_data, A_inv[:n_data], Y.double())):
        left = left.to(torch.bfloat16).double()
        assert torch.isnan(out[0]).all() and torch.isnan(out[-1]).all()
        ref, size = left @ right, left.abs() @ right.abs()
        assert bool(((out[1:rows + 1].double() - ref).abs() <= 2.0 ** -8 * 1.01 * ref.abs() + n * 2.0 ** -24 * size).all())


# one, two and three K steps and more (what is fetched ahead ends differently), in both widths of a whole tile (192: as few rounds as with 256; 256: 3900 x
# 4088 is one round of them and two of the others)
@pytest.mark.parametrize("m,n", [(300, 520), (2048, 12288), (3900, 4088)])
@pytest.mark.parametrize("k", [64, 128, 192, 320])
def test_bf16_few_steps(m, n, k):
    check(m, k, n, torch.bfloat16)


# B in two segments of different pitch: they meet between two steps, on a step's first and last row; shield rows that fill no step, one
# step, two; in tiles of 192 columns and, where those are one more round than tiles of 256, in these
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("n_data,k", [(128, 1), (129, 0), (128, 64), (191, 65), (193, 64), (192, 128), (256, 130), (319, 66)])
def test_bf16_segments_of_a_mix(n_data, k, wide):
    n = n_data + k
    width = (49160 if n <= 384 else 24584) if wide else 520
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_data + k)
    H = torch.full((n_data, width + 24), float("nan"), device="cuda", dtype=torch.bfloat16)[:, :width]
    H.copy_(torch.randn((n_data, width), generator=gen, device="cuda"))
    U = torch.full((n + 2, width), float("nan"), device="cuda", dtype=torch.bfloat16)
    ctx = g.gelo_create(0, 1)
    m = g.gelo_sample_mixing(ctx, g.GELO_ORTHOGONAL, n_data, k, width, g.GELO_BF16, batch_id=1)
    g.gelo_mix(ctx, m, H, U[1:n + 1])
    A, _, S, _, _ = g.gelo_mixing_export(ctx, m, n, k, width)
    torch.cuda.synchronize()
    g.gelo_mixing_free(ctx, m)
    g.gelo_destroy(ctx)
    left, right = A.to(torch.bfloat16).double(), torch.cat([H.double(), S.double()]) if k else H.double()
    ref, size = left @ right, left.abs() @ right.abs()
    assert torch.isnan(U[0]).all() and torch.isnan(U[-1]).all()
    assert bool(((U[1:n + 1].double() - ref).abs() <= 2.0 ** -8 * 1.01 * ref.abs() + n * 2.0 ** -24 * size).all())


# 64 x 64 tiles below one round (256) of 128 x 128 ones, large tiles taken apart into bf16 values from there on (2048 x 40 x 2048 is one
# round); broken tiles, and K that fills no step
@pytest.mark.parametrize("m,k,n", [(1, 136, 8), (63, 136, 72), (64, 264, 64), (65, 136, 200), (543, 776, 1544), (1000, 64, 776),
                                   (2048, 40, 2048), (2049, 40, 2048), (2048, 40, 2056), (129, 512, 2304)])
def test_float_tiles(m, k, n):
    check(m, k, n, torch.float32)


# A result that takes its operand's place: one tile has to read all of it before it stores.  Up to 128 rows of B (un-mix into Y,
# mix into the buffer of H, with and without shield rows), up to 96 columns of A (projection into U); the same bits as elsewhere
@pytest.mark.parametrize("n_data,k", [(64, 0), (65, 0), (100, 0), (121, 6), (127, 0), (128, 0)])
@pytest.mark.parametrize("p", [8, 72, 1000])
def test_float_results_in_place_of_their_operands(n_data, k, p):
    n = n_data + k
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_data + p)
    ctx = g.gelo_create(0, 1, allow_batch_reuse=True)
    m = g.gelo_sample_mixing(ctx, g.GELO_CONDITIONED, n_data, k, p, g.GELO_F32, batch_id=1)
    H = torch.randn((n_data, p), generator=gen, device="cuda")
    U, Z = torch.empty((n, p), device="cuda"), torch.empty((n_data, p), device="cuda")
    g.gelo_mix(ctx, m, H, U)
    g.gelo_unmix(ctx, m, U, Z)
    buf = torch.zeros((n, p), device="cuda")
    buf[:n_data] = H
    g.gelo_mix(ctx, m, buf[:n_data], buf)
    torch.cuda.synchronize()
    assert torch.equal(buf, U)
    g.gelo_unmix(ctx, m, buf, buf[:n_data])
    torch.cuda.synchronize()
    assert torch.equal(buf[:n_data], Z)
    g.gelo_mixing_free(ctx, m)
    if p <= 96:
        X = torch.randn((300, p), generator=gen, device="cuda")
        W, Y = torch.randn((p, p), generator=gen, device="cuda"), torch.empty((300, p), device="cuda")
        g.gelo_project(ctx, X, W, Y)
        g.gelo_project(ctx, X, W, X)
        torch.cuda.synchronize()
        assert torch.equal(X, Y)
    g.gelo_destroy(ctx)


# the same projection of at most 128 rows and columns, one tile too: narrower ones would each read all of A
@pytest.mark.parametrize("rows", [1, 5, 64, 128])
@pytest.mark.parametrize("p", [16, 40, 48, 64, 96, 128])
def test_float_projection_of_few_rows_into_its_operand(rows, p):
    gen = torch.Generator(device="cuda").manual_seed(rows + p)
    X, W, Y = torch.randn((rows, p), generator=gen, device="cuda"), torch.randn((p, p), generator=gen, device="cuda"), torch.empty((rows, p), device="cuda")
    ctx = g.gelo_create(0, 1)
    g.gelo_project(ctx, X, W, Y)
    g.gelo_project(ctx, X, W, X)
    torch.cuda.synchronize()
    g.gelo_destroy(ctx)
    assert torch.equal(X, Y)


# float products taken apart into bf16 values (256 tiles of 128 x 128 and more; one tile less beside them): rows, columns and K that
# fill no tile, fragment or step, the fewest k
@pytest.mark.parametrize("m,k,n", [(2048, 32, 2048), (2047, 40, 2040), (2033, 8, 2048), (1921, 104, 2056), (513, 264, 8200), (130, 1000, 16392), (2048, 64, 1920)])
def test_float_tiles_taken_apart(m, k, n):
    check(m, k, n, torch.float32)


# the same in mix and un-mix: segments of B that meet inside a K step and inside a thread's eight rows (1021 + 51 rows), K = 1072
def test_float_tiles_taken_apart_in_a_mix():
    n_data, k, width = 1021, 51, 4104
    n = n_data + k
    gen = torch.Generator(device="cuda").manual_seed(3)
    H = torch.randn((n_data, width), generator=gen, device="cuda")
    Y = torch.randn((n, width), generator=gen, device="cuda")
    U, Z = torch.empty((n, width), device="cuda"), torch.empty((n_data, width), device="cuda")
    ctx = g.gelo_create(0, 1)
    m = g.gelo_sample_mixing(ctx, g.GELO_REFLECTOR_PRODUCT, n_data, k, width, g.GELO_F32, batch_id=1)
    g.gelo_mix(ctx, m, H, U)
    g.gelo_unmix(ctx, m, Y, Z)
    A, A_inv, S, _, _ = g.gelo_mixing_export(ctx, m, n, k, width)
    torch.cuda.synchronize()
    g.gelo_mixing_free(ctx, m)
    g.gelo_destroy(ctx)
    for out, left, right in ((U, A.double(), torch.cat([H.double(), S.double()])), (Z, A_inv[:n_data].double(), Y.double())):
        bound = (n + 1) * 2.0 ** -24 * (left.abs() @ right.abs()) * 1.01
        assert bool(((out.double() - left @ right).abs() <= bound).all())


# operands below 2^-110, whose last bits bf16 has no exponent for: everywhere, a row, a column, a K step or a single one of them, among zeros,
# in the first and the last K step, in steps behind each other and apart.  The other operand is large, so that results are normal
@pytest.mark.parametrize("k,at", [(40, slice(None)), (200, slice(None)), (200, slice(3, 4)), (200, slice(64, 96)), (200, slice(31, 65)), (200, slice(199, 200)), (200, slice(0, 200, 64))])
@pytest.mark.parametrize("left", [True, False])
def test_float_tiles_taken_apart_with_small_operands(k, at, left):
    gen = torch.Generator(device="cuda").manual_seed(k)
    U, W = torch.randn((2048, k), generator=gen, device="cuda"), torch.randn((k, 2048), generator=gen, device="cuda")
    small, large = (U, W.t()) if left else (W.t(), U)        # (K is the second dimension of either)
    small[:, at] *= 2.0 ** -123
    large *= 2.0 ** 30
    small[100:200] *= torch.rand((100, k), generator=gen, device="cuda") < 0.5
    small[300] = 0.0                                          # nothing else in these rows: no larger product hides what one loses
    small[300, at] = 1.2345678e-37
    small[301] = 0.0
    small[301, k - 1] = -1.2345678e-36
    Y = torch.empty((2048, 2048), device="cuda")
    ctx = g.gelo_create(0, 1)
    g.gelo_project(ctx, U, W, Y)
    torch.cuda.synchronize()
    g.gelo_destroy(ctx)
    ref, size = U.double() @ W.double(), U.double().abs() @ W.double().abs()
    assert bool(((Y.double() - ref).abs() <= 2.0 ** -24 * 1.01 * ref.abs() + k * 2.0 ** -24 * size).all())


# infinities, NaN and sums past the largest float come out as float products give them: an infinity times a finite number is an
# infinity, and the rest of the result is what it is without them
def test_float_tiles_taken_apart_with_infinities():
    gen = torch.Generator(device="cuda").manual_seed(4)
    U = torch.randn((2048, 64), generator=gen, device="cuda")
    W = torch.randn((64, 2048), generator=gen, device="cuda")
    U[3, 5], U[700, 1], U[1500, 60], W[10, 1999] = float("inf"), float("nan"), 3.3e38, -float("inf")
    Y = torch.empty((2048, 2048), device="cuda")
    ctx = g.gelo_create(0, 1)
    g.gelo_project(ctx, U, W, Y)
    torch.cuda.synchronize()
    g.gelo_destroy(ctx)
    ref = U.double() @ W.double()
    size = U.double().abs() @ W.double().abs()
    past = ref.abs() > 3.402823466e38
    want = torch.where(past, ref.sign() * float("inf"), ref)
    assert torch.equal(torch.isnan(Y), torch.isnan(ref))
    sure = ~torch.isnan(ref) & ((ref.abs() > 3.5e38) | (size < 3.3e38))      # (in between a partial sum may or may not pass it)
    assert torch.equal(torch.isinf(Y) & sure, torch.isinf(want) & sure)
    fine = sure & torch.isfinite(want)
    assert bool(((Y.double() - ref).abs()[fine] <= (65 * 2.0 ** -24 * size)[fine] * 1.01).all())


# A value that is not finite changes what it meets and nothing else, to the bit: the results without it elsewhere, in tiles that are computed
# again for its sake as well.  One value, a column of K, whole K steps, the last k, more than the 1024 steps that are told apart; with operands
# large enough for a sum to pass 2^96 too
@pytest.mark.parametrize("value", [float("inf"), -float("inf"), float("nan")])
@pytest.mark.parametrize("k,at", [(40, slice(39, 40)), (104, slice(7, 8)), (104, slice(32, 64)), (200, slice(0, 200, 33)), (33000, slice(20000, 20001))])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** 40])
def test_float_tiles_taken_apart_keep_the_bits_beside_values_not_finite(value, k, at, scale):
    gen = torch.Generator(device="cuda").manual_seed(k)
    U, W = torch.randn((2048, k), generator=gen, device="cuda") * scale, torch.randn((k, 2048), generator=gen, device="cuda") * scale
    Y, Y0 = torch.empty((2048, 2048), device="cuda"), torch.empty((2048, 2048), device="cuda")
    ctx = g.gelo_create(0, 1)
    g.gelo_project(ctx, U, W, Y0)
    U[130, at], U[2047, at], W[at, 777] = value, value, value
    g.gelo_project(ctx, U, W, Y)
    torch.cuda.synchronize()
    g.gelo_destroy(ctx)
    ref = U.double() @ W.double()
    met = torch.zeros((2048, 2048), dtype=torch.bool, device="cuda")
    met[130], met[2047], met[:, 777] = True, True, True
    assert torch.equal(Y[~met], Y0[~met])
    assert torch.equal(Y[met].double().nan_to_num(nan=7.0), ref[met].nan_to_num(nan=7.0))


# operands and sums that leave the range of the operands taken apart (2^112, 2^96) but not that of float, among others in it
def test_float_tiles_taken_apart_with_large_operands():
    gen = torch.Generator(device="cuda").manual_seed(5)
    U, W = torch.randn((2048, 72), generator=gen, device="cuda"), torch.randn((72, 2048), generator=gen, device="cuda")
    U[5], U[700, 3], U[1500] = U[5] * 2.0 ** 120, 1.5 * 2.0 ** 125, U[1500] * 2.0 ** 60
    W[:, 30] *= 2.0 ** 50
    W[:, 31] *= 2.0 ** -30
    W[3] = W[3] * 2.0 ** -6
    Y = torch.empty((2048, 2048), device="cuda")
    ctx = g.gelo_create(0, 1)
    g.gelo_project(ctx, U, W, Y)
    torch.cuda.synchronize()
    g.gelo_destroy(ctx)
    ref, size = U.double() @ W.double(), U.double().abs() @ W.double().abs()
    sure = size < 3.3e38                                     # (beyond, a partial sum may pass the largest float)
    assert int((~sure).sum()) == 2
    assert bool(((Y.double() - ref).abs() <= 2.0 ** -24 * 1.01 * ref.abs() + 72 * 2.0 ** -24 * size)[sure].all())


# The same product with its result in place of an operand (128 rows of B, so many columns that it is taken apart), and with operands and
# result as slices of the columns of one buffer: the same bits
@pytest.mark.parametrize("n_data,k", [(128, 0), (100, 28), (121, 6)])
def test_float_tiles_taken_apart_in_place_of_their_operands(n_data, k):
    n, p = n_data + k, 32776
    gen = torch.Generator(device="cuda").manual_seed(n_data)
    ctx = g.gelo_create(0, 1, allow_batch_reuse=True)
    m = g.gelo_sample_mixing(ctx, g.GELO_CONDITIONED, n_data, k, p, g.GELO_F32, batch_id=1)
    H = torch.randn((n_data, p), generator=gen, device="cuda")
    H[3, 7], H[5, 9000] = float("inf"), float("nan")             # (computed again behind the loop, still before anything is stored)
    U, Z = torch.empty((n, p), device="cuda"), torch.empty((n_data, p), device="cuda")
    g.gelo_mix(ctx, m, H, U)
    g.gelo_unmix(ctx, m, U, Z)
    buf = torch.zeros((n, p), device="cuda")
    buf[:n_data] = H
    g.gelo_mix(ctx, m, buf[:n_data], buf)
    torch.cuda.synchronize()
    assert torch.equal(buf.view(torch.int32), U.view(torch.int32))
    g.gelo_unmix(ctx, m, buf, buf[:n_data])
    torch.cuda.synchronize()
    assert torch.equal(buf[:n_data].view(torch.int32), Z.view(torch.int32))
    g.gelo_mixing_free(ctx, m)
    g.gelo_destroy(ctx)


@pytest.mark.parametrize("m,k,n", [(2048, 104, 2056), (2048, 2048, 2048), (300, 104, 200)])
def test_float_slices_of_one_buffer(m, k, n):
    gen = torch.Generator(device="cuda").manual_seed(m + n)
    wide = torch.randn((max(m, k), k + 2 * n), generator=gen, device="cuda")
    U, W, Y = wide[:m, :k], wide[:k, k:k + n], wide[:m, k + n:]
    apart = torch.empty((m, n), device="cuda")
    ctx = g.gelo_create(0, 1)
    g.gelo_project(ctx, U.contiguous(), W.contiguous(), apart)
    before = wide[:, :k + n].clone()
    g.gelo_project(ctx, U, W, Y)
    torch.cuda.synchronize()
    g.gelo_destroy(ctx)
    assert torch.equal(Y, apart) and torch.equal(wide[:, :k + n], before)
