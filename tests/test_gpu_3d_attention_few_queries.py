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
