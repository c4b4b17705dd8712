"""GPU parity of the selection where its launch configuration changes: token counts at the edges of the top-k's
register classes (1024 * 2^i tokens), maps whose scores crowd into one histogram bin (the radix select has to cut a
bin again), row chunks of the column sums that are not full, and widths around the 512-column groups.
Same bar as test_gpu_1_select.py: index sets bit-exact, scores within one fp32 rounding."""
import numpy as np
import pytest
import torch

from paper_2503_23367_amd import binding as fb
from paper_2503_23367_amd import synth
from gpu_util import DEV, empty_ws
from test_gpu_1_select import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 2, 31, 33, 1023, 1024, 1025, 2048, 2049, 4097, 8192, 8193, 16385, 32767])
def test_token_count_edges(N):
    D = 64 if N > 4097 else 200
    x = synth.token_map(7, 1, 1, N, D)
    for k in sorted({1, N // 3, N - 1, N} - {0}):
        check_against_oracle(x, 1, N, k, f"N{N}_k{k}")


@pytest.mark.parametrize("N", [900, 3000, 12000])
def test_scores_crowded_into_one_bin(N):
    """One token far out sets the range of the keys; all the others differ by a few ulps or not at all, so a single
    bin of the first histogram holds nearly every token."""
    rng = np.random.default_rng(N)
    x = np.ones((1, N, 64), np.float32)
    x[0, :, 0] = rng.choice(np.float32([1.0, 1.0078125, 1.015625, 0.9921875]), size=N)
    x[0, :, 1] = rng.choice(np.float32([1.0, 1.0078125, 1.015625]), size=N)
    x[0, N // 2] = 300.0
    for k in (1, 2, 255, N // 2, N - 2):
        check_against_oracle(x, 1, N, k, f"crowded_N{N}_k{k}")


@pytest.mark.parametrize("D", [8, 504, 512, 1032, 2056, 4104])
def test_width_edges(D):
    x = synth.token_map(13, 2, 9, 23, D)
    check_against_oracle(x, 9, 23, 71, f"D{D}")


@pytest.mark.parametrize("B,h,w,D", [(8, 32, 32, 1920), (3, 40, 40, 2048), (5, 16, 16, 1024), (2, 64, 64, 512)])
def test_scores_of_a_sample_do_not_depend_on_its_batch(B, h, w, D):
    """Bit for bit, on maps whose column sums depend on the order they are added in: eight columns hold 2^80 and -2^80 at two
    rows, which swallow what the sums had gathered."""
    N, k = h * w, h * w // 3
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B)
    x = torch.randn(B, N, D, generator=gen, device=DEV)
    for b in range(B):
        for c in range(0, D, D // 8):
            x[b, torch.randperm(N, generator=gen, device=DEV)[:2], c] = torch.tensor([2.0 ** 80, -2.0 ** 80], device=DEV)
    x = x.to(torch.bfloat16)

    def scores(maps):
        n = maps.shape[0]
        score = torch.full((n, N), float("nan"), device=DEV)
        idx = torch.empty(n, k, dtype=torch.int32, device=DEV)
        fb.fastvar_select_pivotal(maps, n, h, w, D, k, idx, None, score,
                                  empty_ws(fb.fastvar_select_workspace_bytes(n, N, D)))
        return torch.cat([score.view(torch.int32), idx], dim=1)

    whole = scores(x)
    alone = torch.cat([scores(x[b:b + 1].contiguous()) for b in range(B)])
    torch.cuda.synchronize()
    assert torch.equal(whole, alone)
