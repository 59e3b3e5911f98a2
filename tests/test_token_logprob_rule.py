"""Into how many parts the token statistics cut a row, by the host-side rule alone (no GPU), read off the workspace query."""
import pytest

from paper_2512_21450_amd import binding as B


def splits(n, V, dtype=B.RLDA_BF16, ref=False):
    ds = B.make_token_logprob_desc(dtype, n, V, -(-V // 8) * 8, 1.0, ref_logits=1 << 20 if ref else None)
    need = B.rl_token_logprob_workspace_bytes(ds)
    assert need % (24 * n) == 0
    return max(1, need // (24 * n))


@pytest.mark.parametrize("dtype,size", [(B.RLDA_F32, 4), (B.RLDA_BF16, 2)])
@pytest.mark.parametrize("V", [16384, 32000, 50257, 151936, 256000, 1000000])
def test_few_rows_leave_a_thread_no_long_chain_of_loads(V, dtype, size):
    """256 threads read 16 KB of a row in one round of loads: one round where the compute units hold it, two at most, but for
    what the merge's 64 splits leave (1024 threads then)."""
    for n in (1, 2, 8, 16) if V < 1000000 else (1, 2, 8):
        s = splits(n, V, dtype)
        assert s == 64 or V * size / s <= (16 if n <= 8 else 32) * 1024 * 1.1, (n, V, s)


@pytest.mark.parametrize("V", [1, 4096, 8192, 9000, 16383])
def test_short_rows_are_not_split(V):
    """Two splits and their merge: 6.8 us, one workgroup a row: 5.4 (48 rows of 9000 logits)."""
    for n in (1, 48, 191, 300, 600):
        for ref in (False, True):
            assert splits(n, V, ref=ref) == splits(n, V, B.RLDA_F32, ref) == 1, (n, V)


@pytest.mark.parametrize("n,V,dtype,ref", [(257, 32000, 1, False), (352, 32000, 1, False), (352, 32000, 0, False), (400, 65536, 1, False),
                                           (448, 65536, 0, True), (448, 151936, 1, False), (448, 151936, 0, True), (513, 65536, 0, False),
                                           (576, 151936, 0, False), (640, 65536, 1, False), (640, 65536, 0, True), (192, 151936, 1, True),
                                           (256, 151936, 0, True), (641, 151936, 1, True), (4096, 151936, 1, True)])
def test_rows_that_lose_by_splits_are_not_split(n, V, dtype, ref):
    assert splits(n, V, dtype, ref) == 1


@pytest.mark.parametrize("n,V,dtype,ref", [(257, 32000, 1, True), (300, 151936, 1, True), (300, 151936, 0, False), (376, 151936, 1, False),
                                           (448, 151936, 1, True), (513, 65536, 1, True), (576, 151936, 1, False), (600, 65536, 0, True)])
def test_rows_that_gain_are(n, V, dtype, ref):
    assert splits(n, V, dtype, ref) > 1


def test_a_workspace_of_the_fallback_is_never_larger_than_what_is_asked_for():
    """A caller with less than the query's bytes gets min(ceil(256 / n), vocab / 8192, 64) splits, so that what suffices for them
    is never refused for being too little of something larger, nor the query below it."""
    for n in list(range(1, 200)) + [256, 257, 300, 512, 600]:
        for V in (8191, 8192, 16383, 16384, 20000, 32000, 49152, 151936, 524288, 1 << 30):
            less = min(-(-256 // n), V // 8192, 64) if n < 192 else 1
            for dtype in (B.RLDA_F32, B.RLDA_BF16):
                assert splits(n, V, dtype) >= less, (n, V, dtype)
