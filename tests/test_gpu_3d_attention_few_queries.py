"""GPU parity of attention with few queries, on both sides of the rules that pick its workgroups (one tile of 64 keys; 32, 64 or
128 queries; head dims 64 and 128) and at the edges of their tiles.  The check of test_gpu_3_components.py."""
import pytest

from test_gpu_3_components import test_attention_matches_oracle as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("H,B,k,L", [
    (3, 2, 1, 1), (2, 1, 5, 63), (2, 2, 129, 64),                               # one tile of 64 keys
    (2, 1, 1, 65), (2, 2, 32, 127), (3, 1, 33, 128), (2, 1, 64, 129), (1, 3, 65, 257), (16, 1, 352, 521),
    (16, 1, 353, 384),                                                          # 176 / 192 workgroups of 32 queries
    (16, 4, 200, 300), (16, 4, 257, 512), (16, 2, 128, 513), (32, 2, 250, 140)])   # 256 workgroups of 64 queries and more
def test_attention_few_queries(H, dh, B, k, L):
    check(H, dh, B, k, L, (L + 7) // 8 * 8)


@pytest.mark.parametrize("H,B,k,L", [
    (16, 1, 100, 641), (2, 1, 33, 768), (2, 2, 1, 769), (3, 1, 32, 1023),       # tiles of 256 keys over 32 queries
    (16, 1, 257, 897), (16, 1, 300, 1024), (8, 2, 513, 1025), (30, 1, 270, 2055)])   # over 64
def test_attention_key_tiles_in_four(H, B, k, L):
    """Head dim 64, a tile's keys between four waves: last tiles of one key, of a slice and less, of all but one key, and whole."""
    check(H, 64, B, k, L, (L + 7) // 8 * 8)
