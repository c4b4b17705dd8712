"""GPU parity: fastvar_restore vs the CPU oracle (Sec. 3.3, Eq. 6 + scatter).

Bar: kept slots carry the kept outputs bit for bit; every other slot equals
the oracle's fp64 bilinear resample to within one bf16 rounding of an fp32
evaluation (|err| <= 2^-8 |ref| + 2e-6, far inside the 2e-2 max-relative
bar; the tighter bound is what is asserted).
"""
import numpy as np
import pytest
import torch

from oracle import fastvar_oracle as O
from paper_2503_23367_amd import binding as fb
from paper_2503_23367_amd import synth
from gpu_util import DEV, empty_ws, from_dev_bf16, max_rel, to_dev_bf16, upload_weights

pytestmark = pytest.mark.gpu


def run_restore(yk_np, idx_np, cache_np, hc, wc, h, w, use_rank):
    B, Nc, D = cache_np.shape
    k = idx_np.shape[1]
    N = h * w
    yk = to_dev_bf16(yk_np) if k > 0 else None
    idx = torch.from_numpy(idx_np.astype(np.int32)).to(DEV) if k > 0 else None
    rank = None
    if use_rank and k > 0:
        r = np.full((B, N), -1, np.int32)
        for b in range(B):
            r[b, idx_np[b]] = np.arange(k, dtype=np.int32)
        rank = torch.from_numpy(r).to(DEV)
    cache = to_dev_bf16(cache_np)
    y = torch.full((B, N, D), float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = empty_ws(fb.fastvar_restore_workspace_bytes(B, N))
    fb.fastvar_restore(yk, idx, rank, B, k, cache, hc, wc, h, w, D, y, ws)
    torch.cuda.synchronize()
    return from_dev_bf16(y), (None if yk is None else from_dev_bf16(yk))


def check(name, B, hc, wc, h, w, D, k, use_rank=True, seed=0):
    print(f"[restore] {name} B={B} cache={hc}x{wc} map={h}x{w} D={D} k={k} rank={'given' if use_rank else 'rebuilt'}",
          flush=True)
    rng = np.random.default_rng(seed)
    N = h * w
    cache = synth.cached_map(seed, B, hc, wc, D)
    yk = synth.round_bf16(rng.standard_normal((B, k, D)).astype(np.float32))
    idx = np.stack([np.sort(rng.permutation(N)[:k]) for _ in range(B)]).astype(np.int32).reshape(B, k)
    got, _ = run_restore(yk, idx, cache, hc, wc, h, w, use_rank)
    ref = O.restore(yk, idx, cache, hc, wc, h, w)
    assert not np.isnan(got).any(), name
    for b in range(B):
        kept = np.zeros(N, bool)
        kept[idx[b]] = True
        # layout: kept slots bit-exact
        np.testing.assert_array_equal(got[b, idx[b]], yk[b], err_msg=name)
        # pruned slots: fp32 lerp rounded to bf16 vs fp64 lerp
        g, r = got[b, ~kept].astype(np.float64), ref[b, ~kept]
        if g.size:
            # one bf16 rounding (half an ulp <= 2^-8 |v|) plus fp32 evaluation noise
            assert np.all(np.abs(g - r) <= 2.0 ** -8 * 1.001 * np.abs(r) + 2e-6), name
    assert max_rel(got, ref) <= 2e-2


CASES = [
    ("d16_13_to_16", 1, 13, 13, 16, 16, 1024, 128),
    ("d30_18_to_24_b8", 8, 18, 18, 24, 24, 1920, 346),
    ("d30_18_to_32_b8", 8, 18, 18, 32, 32, 1920, 410),
    ("inf2b_32_to_64", 1, 32, 32, 64, 64, 2048, 2048),
    ("inf2b_32_to_48_b4", 4, 32, 32, 48, 48, 2048, 1152),
    ("inf2b_2k_64_to_128", 1, 64, 64, 128, 128, 2048, 4096),
    ("skip_step_k0", 2, 8, 8, 12, 12, 256, 0),
    ("keep_all", 2, 8, 8, 12, 12, 256, 144),
    ("ragged_rect_D200", 3, 3, 5, 7, 6, 200, 11),
    ("from_1x1", 2, 1, 1, 5, 3, 64, 4),
    ("same_size", 1, 6, 6, 6, 6, 128, 10),
    ("downsample_allowed", 1, 9, 9, 4, 4, 64, 3),
]


@pytest.mark.parametrize("name,B,hc,wc,h,w,D,k", CASES, ids=[c[0] for c in CASES])
def test_restore_matches_oracle(name, B, hc, wc, h, w, D, k):
    check(name, B, hc, wc, h, w, D, k, use_rank=True, seed=3)


@pytest.mark.parametrize("name,B,hc,wc,h,w,D,k", [CASES[0], CASES[3], CASES[8]], ids=["d16", "inf2b", "ragged"])
def test_restore_rebuilds_rank_from_idx(name, B, hc, wc, h, w, D, k):
    check(name, B, hc, wc, h, w, D, k, use_rank=False, seed=4)


@pytest.mark.parametrize("B,hc,wc,h,w,D,k", [(1, 21, 40, 67, 65, 64, 1300), (3, 9, 21, 37, 41, 456, 700), (1, 30, 31, 70, 62, 1288, 4340),
                                             (1, 17, 5, 4301, 1, 8, 0)])
def test_restore_two_rows_a_wave(B, hc, wc, h, w, D, k):
    """Maps of more rows than the chip has waves for: a pair a wave, an odd row and a part-filled workgroup at the end."""
    check("pair", B, hc, wc, h, w, D, k, use_rank=True, seed=5)


@pytest.mark.parametrize("B,h,w", [(3, 1, 3), (9, 1, 1), (2, 18, 14), (2, 11, 23), (3, 16, 16), (2, 257, 1), (1, 75, 70), (1, 80, 86),
                                   (9, 13, 20), (3, 20, 33), (2, 70, 63), (1, 40, 128), (2, 39, 61)])
def test_restore_shares_around_the_xcds(B, h, w):
    """Workgroups in numbers that eight does and does not divide, samples that end inside one; two on both sides of where wide rows go from
    one to two a wave; runs that move on more than a round of samples, and shares dealt in turn, of one row a wave and of a pair."""
    D = 1288 if h > 40 else 72
    check("shares", B, max(1, h // 2), max(1, w // 2), h, w, D, h * w // 3, use_rank=True, seed=6)


@pytest.mark.parametrize("B,h,w", [(9, 13, 20), (3, 16, 32), (2, 20, 33), (1, 24, 48), (1, 5, 65), (2, 3, 7)])
def test_fill_of_a_step_equals_the_restoration(B, h, w):
    """A step fills its pruned rows inside the gather's launch, by the restoration's code: the same map, bit for bit."""
    dims, N, hc, wc = synth.BlockDims(D=64, H=1, dh=64, F=64), h * w, max(1, h // 2), max(1, w // 2)
    k, L_cap = max(1, N // 3), (N // 3 + 15) // 8 * 8
    print(f"[fill] B={B} map={h}x{w} k={k}", flush=True)
    _, weights = upload_weights(synth.block_weights(3, dims))
    cache, x = to_dev_bf16(synth.cached_map(3, B, hc, wc, 64)), to_dev_bf16(synth.token_map(3, B, h, w, 64))
    kc, vc = (torch.zeros((B, 1, a, b), dtype=torch.bfloat16, device=DEV) for a, b in ((L_cap, 64), (64, L_cap)))
    y = torch.full((B, N, 64), float("nan"), dtype=torch.bfloat16, device=DEV)
    idx = torch.empty((B, k), dtype=torch.int32, device=DEV)
    d = fb.make_dims(64, 1, 64, 64)
    fb.fastvar_step(x, [hc, h], [wc, w], 1, 0, B, k, d, weights, kc, vc, 0, L_cap, cache, y, idx,
                    empty_ws(fb.fastvar_step_workspace_bytes(d, B, N, k)))
    kept = torch.gather(y, 1, idx.long()[..., None].expand(B, k, 64)).contiguous()
    ref = torch.full_like(y, float("nan"))
    fb.fastvar_restore(kept, idx, None, B, k, cache, hc, wc, h, w, 64, ref, empty_ws(fb.fastvar_restore_workspace_bytes(B, N)))
    assert not torch.isnan(y).any()
    assert torch.equal(y.view(torch.int16), ref.view(torch.int16))


def test_restore_special_cases_exact():
    print("[restore] exact special cases", flush=True)
    # same size: identity on pruned slots; constant cache: constant; 2x of a bf16-exact ramp
    c = synth.cached_map(1, 1, 6, 6, 128)
    got, _ = run_restore(np.zeros((1, 0, 128), np.float32), np.zeros((1, 0), np.int32), c, 6, 6, 6, 6, True)
    np.testing.assert_array_equal(got, c)
    c = np.full((1, 16, 64), 1.5, np.float32)
    got, _ = run_restore(np.zeros((1, 0, 64), np.float32), np.zeros((1, 0), np.int32), c, 4, 4, 9, 7, True)
    assert np.all(got == 1.5)
    # integer ramp upsampled 2x: results are multiples of 1/16, exact in bf16 for small values
    ii, jj = np.meshgrid(np.arange(4), np.arange(4), indexing="ij")
    c = np.repeat((2.0 * ii + 1.0 * jj).reshape(1, 16, 1), 8, axis=2).astype(np.float32)
    got, _ = run_restore(np.zeros((1, 0, 8), np.float32), np.zeros((1, 0), np.int32), c, 4, 4, 8, 8, True)
    ref = O.upsample_bilinear(c, 4, 4, 8, 8)
    np.testing.assert_array_equal(got.astype(np.float64), ref)


def test_restore_argument_errors():
    print("[restore] error paths", flush=True)
    c = to_dev_bf16(synth.cached_map(1, 1, 2, 2, 64))
    y = torch.zeros((1, 16, 64), dtype=torch.bfloat16, device=DEV)
    L = fb.lib()
    st = torch.cuda.current_stream().cuda_stream
    assert L.fastvar_restore(None, None, None, 1, 0, None, 2, 2, 4, 4, 64, y.data_ptr(), None, 0, st) == fb.FASTVAR_EINVAL
    assert L.fastvar_restore(None, None, None, 1, 3, c.data_ptr(), 2, 2, 4, 4, 64, y.data_ptr(), None, 0, st) == fb.FASTVAR_EINVAL
    assert L.fastvar_restore(None, None, None, 1, 0, c.data_ptr(), 2, 2, 4, 4, 64, c.data_ptr(), None, 0, st) == fb.FASTVAR_EINVAL
    assert L.fastvar_restore(None, None, None, 1, 0, c.data_ptr(), 2, 2, 4, 4, 60, y.data_ptr(), None, 0, st) == fb.FASTVAR_EALIGN
    yk = torch.zeros((1, 3, 64), dtype=torch.bfloat16, device=DEV)
    idx = torch.tensor([[0, 5, 9]], dtype=torch.int32, device=DEV)
    assert L.fastvar_restore(yk.data_ptr(), idx.data_ptr(), None, 1, 3, c.data_ptr(), 2, 2, 4, 4, 64, y.data_ptr(), None, 0, st) == fb.FASTVAR_EWORKSPACE
    torch.cuda.synchronize()
    assert torch.all(y == 0)
