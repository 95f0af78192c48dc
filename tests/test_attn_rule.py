"""What fs_beam_decode_step_noalloc refuses depends on the sizes alone: fewer
than 128 rows of more than two chunks whose split-KV records exceed the
scratch array, whichever decomposition the size rule takes for them.  The
calls stop at the check (no GPU, no pointer is read)."""
import pytest

from paper_2106_04718_amd import _native as N

FAKE = [(i + 1) << 32 for i in range(7)]


def status(B, k, H, S, D, dtype):
    q, K, V, ln, out, tok, lg = FAKE
    # out of line of every allowed call: the logits overlap the queries, so a
    # call that is not refused for its records ends as an invalid argument
    return N.lib().fs_beam_decode_step_noalloc(q, K, V, ln, out, B, k, H, S, D, dtype, tok, 8, 8, 3, q, 100, None)


@pytest.mark.parametrize("B,k,H,S,D,dtype,refused", [
    (1, 8, 127, 1024, 64, N.FS_BF16, True),     # 127 rows x 16 tiles x 8 beams: 8.6 MB of records
    (1, 8, 127, 512, 64, N.FS_BF16, False),     # two chunks
    (1, 8, 128, 1024, 64, N.FS_BF16, False),    # 128 rows: never split
    (1, 4, 127, 1024, 64, N.FS_BF16, False),    # half the beams: 4.3 MB
    (4, 8, 16, 2048, 128, N.FS_BF16, True),
    (1, 8, 16, 2048, 128, N.FS_F32, True),
])
def test_noalloc_refusal_depends_on_sizes_only(B, k, H, S, D, dtype, refused):
    st = status(B, k, H, S, D, dtype)
    if refused:
        assert st == N.FS_ERR_UNSUPPORTED and "scratch array" in N.last_error()
    else:
        assert st == N.FS_ERR_INVALID_ARG and "overlap" in N.last_error()
