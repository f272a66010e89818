"""GPU checks of the library's device primitives against NumPy: exclusive scan, stable radix
sort (bit-exact), and the MFMA tile routine (the lane layout of the matrix instruction)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1705_07860_amd import binding as ob
    c = ob.Context(arena_bytes=256 << 20)
    yield c
    c.close()


@pytest.mark.parametrize("n", [0, 1, 255, 1024, 1025, 4095, 4096, 4097, 5000, 300001])
def test_scan(ctx, n):
    rng = np.random.default_rng(n)
    a = rng.integers(0, 1000, size=n).astype(np.uint32)
    out, tot = ctx.test_scan(a)
    ref = np.concatenate([[0], np.cumsum(a.astype(np.uint64))[:-1]]).astype(np.uint32) if n else a
    assert np.array_equal(out, ref)
    assert tot == int(a.sum())


@pytest.mark.parametrize("n,lo,bits", [(1, 0, 8), (2, 0, 1), (64, 0, 8), (1000, 0, 18), (1023, 5, 26), (1025, 32, 10),
                                       (4097, 0, 5), (4097, 0, 26), (8192, 0, 24), (8192, 7, 17), (8193, 0, 9),
                                       (240000, 0, 18), (240000, 32, 18), (196608, 0, 12), (196609, 3, 12), (80000, 0, 17),
                                       (262144, 0, 9), (262145, 0, 16), (700001, 4, 12)])
def test_radix_sort_is_stable_and_exact(ctx, n, lo, bits):
    rng = np.random.default_rng(n + lo)
    keys = rng.integers(0, 1 << 62, size=n, dtype=np.uint64)
    keys[::3] = keys[0]                      # many duplicates to exercise stability
    vals = np.arange(n, dtype=np.uint32)
    ko, vo = ctx.test_sort(keys, vals, lo, bits)
    field = (keys >> np.uint64(lo)) & np.uint64((1 << bits) - 1)
    order = np.argsort(field, kind="stable")
    assert np.array_equal(vo, vals[order])
    assert np.array_equal(ko, keys[order])


def _two_fields(n, lo, hi):
    """n pairs; the order by the field of `hi` bits at bit 32, then by that of `lo` bits at bit 3, then as they come."""
    rng = np.random.default_rng(n + 100 * lo + hi)
    a, b = rng.integers(0, 1 << lo, size=n, dtype=np.uint64), rng.integers(0, 1 << hi, size=n, dtype=np.uint64)
    b[: n // 2] = b[0]            # half the pairs share the upper field
    keys = (b << np.uint64(32)) | (a << np.uint64(3)) | rng.integers(0, 8, size=n, dtype=np.uint64)
    return keys, np.arange(n, dtype=np.uint32)[::-1].copy(), np.lexsort((np.arange(n), a, b))


@pytest.mark.parametrize("lo,hi", [(8, 8), (16, 10), (17, 17), (9, 5), (5, 0), (0, 9)])   # 2, 4, 6, 3, 1 and 2 passes
@pytest.mark.parametrize("n", [1, 2, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 50000, 524288, 524289])
def test_two_field_sort_matches_lexicographic_order(ctx, n, lo, hi):
    """The schedule's sort: both fields in one call, the less significant one first."""
    keys, vals, order = _two_fields(n, lo, hi)
    ko, vo = ctx.test_sort_fields(keys, vals, 3, lo, 32, hi)
    assert np.array_equal(ko, keys[order]) and np.array_equal(vo, vals[order])
    if n <= 8193:                 # one field after the other gives the same
        k1, v1 = ctx.test_sort(keys, vals, 3, lo)
        k2, v2 = ctx.test_sort(k1, v1, 32, hi)
        assert np.array_equal(k2, ko) and np.array_equal(v2, vo)


@pytest.mark.parametrize("n", [1024, 1025, 2049, 4097, 8192])
@pytest.mark.parametrize("count", [0, 1, 1000, -1, None])
def test_sort_of_a_length_known_on_the_device(ctx, n, count):
    """The pairs from the count on carry the largest key and stay where they are, whichever width of the one-workgroup
    sort the count selects."""
    m = n if count is None else (n - 1 if count < 0 else count)
    keys, vals, order = _two_fields(n, 13, 13)
    keys[m:] = 0xffffffffffffffff
    order = np.concatenate([np.lexsort((np.arange(m), (keys[:m] >> np.uint64(3)) & np.uint64(0x1fff),
                                        (keys[:m] >> np.uint64(32)) & np.uint64(0x1fff))), np.arange(m, n)]).astype(np.int64)
    ko, vo = ctx.test_sort_fields(keys, vals, 3, 13, 32, 13, count=m)
    assert np.array_equal(ko, keys[order]) and np.array_equal(vo, vals[order])


# one workgroup with 1, 2, 4 and 8 keys per lane; blocks of 2048, whose counts the scatter adds up itself up to 256 blocks
@pytest.mark.parametrize("n", [63, 65, 1024, 1025, 2048, 2049, 4096, 5000, 8191, 8193, 10240, 10241, 524288, 524289])
@pytest.mark.parametrize("kind", ["equal", "falling", "random"])
def test_radix_sort_at_the_edges_of_its_tiles(ctx, n, kind):
    rng = np.random.default_rng(n)
    keys = {"equal": np.full(n, (1 << 40) | 0x5a5a5), "falling": np.arange(n)[::-1] << 3,
            "random": rng.integers(0, 1 << 40, size=n)}[kind].astype(np.uint64)
    vals = np.arange(n, dtype=np.uint32)[::-1].copy()
    ko, vo = ctx.test_sort(keys, vals, 2, 17)
    order = np.argsort((keys >> np.uint64(2)) & np.uint64((1 << 17) - 1), kind="stable")
    assert np.array_equal(ko, keys[order]) and np.array_equal(vo, vals[order])


@pytest.mark.parametrize("M,N,K", [(32, 32, 8), (64, 1024, 256), (1, 5, 256), (33, 50, 512), (70, 35, 7),
                                   (3, 3, 1), (128, 96, 36)])
def test_mfma_tile_gemm(ctx, M, N, K):
    rng = np.random.default_rng(M * 1000 + N + K)
    A = rng.standard_normal((M, K)).astype(np.float32)
    B = rng.standard_normal((N, K)).astype(np.float32)
    C = ctx.test_gemm(A, B)
    ref = A.astype(np.float64) @ B.astype(np.float64).T
    err = np.max(np.abs(C - ref)) / max(np.max(np.abs(ref)), 1e-30)
    assert err < 1e-5, err
