"""GPU parity of the products of few rows (up to 16: a workgroup owns 8 or 16 output columns and its waves share K),
at the edges of the row group (16), column tiles and K turns (64 wide, an odd number of them, more than one
round), with and without the LayerNorm in front (every token kept, up to 2048 columns).
Same bars as test_gpu_3_components.py and test_gpu_4_block.py."""
import numpy as np
import pytest
import torch

from oracle import fastvar_oracle as O
from paper_2503_23367_amd import binding as fb
from paper_2503_23367_amd import synth
from gpu_util import DEV, cache_rows, empty_ws, from_dev_bf16, make_caches, max_rel, to_dev_bf16, upload_weights
from test_gpu_3_components import rnd
from test_gpu_4_block import branch_error
from test_gpu_9_rope import check_block_rope

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 15, 16, 17, 32, 33])
@pytest.mark.parametrize("N,K", [(64, 64), (72, 192), (200, 2048), (136, 2112), (72, 8256), (4112, 576), (4104, 1088)])
@pytest.mark.parametrize("epi", [fb.EPI_BIAS_RES, fb.EPI_BIAS_GELU])
def test_gemm_few_rows(M, N, K, epi):
    rng = np.random.default_rng(M * 7 + N * 3 + K + epi)
    A, W = rnd(rng, M, K), rnd(rng, N, K, scale=0.2)
    bias, res = rnd(rng, N), rnd(rng, M, N)
    guard = 4096   # untouched elements behind the output
    out = torch.full((M * N + guard,), float("nan"), dtype=torch.bfloat16, device=DEV)
    fb.fastvar_gemm_bf16(to_dev_bf16(A), to_dev_bf16(W), to_dev_bf16(bias), to_dev_bf16(res), M, N, K, epi, out)
    torch.cuda.synchronize()
    lin = O.linear(A, W, bias)
    ref = lin + res if epi == fb.EPI_BIAS_RES else O.gelu(lin)
    got = from_dev_bf16(out)
    assert np.isnan(got[M * N:]).all()
    assert max_rel(got[:M * N].reshape(M, N), ref) <= 2.0 ** -7, (M, N, K, epi)


@pytest.mark.parametrize("M", [1, 8, 13, 16])
@pytest.mark.parametrize("N,K", [(72, 512), (72, 1088), (72, 2112), (72, 4800), (72, 8064), (4112, 64), (4112, 1600),
                                 (4112, 2112), (4096, 4096), (2304, 2304), (12304, 128), (16400, 576)])
def test_gemm_few_rows_turns_in_flight(M, N, K):
    """One to four turns in flight for eight and sixteen waves, one and two rounds of them, and shapes on both sides of the
    rule that sends wide outputs to the tiled product."""
    test_gemm_few_rows(M, N, K, fb.EPI_BIAS_RES)


@pytest.mark.parametrize("B,N,L0", [(1, 5, 12), (3, 4, 7), (1, 16, 9)])
@pytest.mark.parametrize("dims", [synth.D16, synth.BlockDims(D=640, H=10, dh=64, F=2560), synth.BlockDims(D=1536, H=12, dh=128, F=6144),
                                  synth.BlockDims(D=2176, H=17, dh=128, F=8704)], ids=lambda d: f"D{d.D}")
def test_block_that_mixes_few_row_and_tiled_products(dims, B, N, L0):
    """LayerNorm in front of one product and split K in another (1536 columns, more than eight rows), every product tiled but
    two (2176 columns), one to three turns in flight."""
    test_block_all_tokens_kept_without_an_index_list(dims, B, N, L0)


@pytest.mark.parametrize("dims", [synth.BlockDims(D=64, H=1, dh=64, F=64), synth.BlockDims(D=192, H=3, dh=64, F=320),
                                  synth.BlockDims(D=1088, H=17, dh=64, F=1088), synth.D30, synth.INF2B,
                                  synth.BlockDims(D=2176, H=17, dh=128, F=2240)], ids=lambda d: f"D{d.D}")
@pytest.mark.parametrize("B,N,L0", [(1, 1, 0), (2, 8, 3), (1, 17, 300), (4, 8, 21), (3, 11, 40)])
def test_block_all_tokens_kept_without_an_index_list(dims, B, N, L0):
    print(f"[few rows] D={dims.D} B={B} N={N} L0={L0}", flush=True)
    L_cap = (L0 + N + 7) // 8 * 8 + 8
    x_np = synth.token_map(5, B, 1, N, dims.D)
    W = synth.block_weights(5, dims)
    kp, vp = synth.kv_prior(5, B, L0, dims.H, dims.dh)
    d = fb.make_dims(dims.D, dims.H, dims.dh, dims.F)
    wt, ws_struct = upload_weights(W)
    x = to_dev_bf16(x_np)
    kc, vc = make_caches(kp, vp, L_cap)
    y, h1 = (torch.full((B, N, dims.D), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    ws = empty_ws(fb.fastvar_block_workspace_bytes(d, B, N))
    ws.fill_(0xFF)
    fb.fastvar_attn_forward_pruned(x, N, None, B, N, d, ws_struct, kc, vc, L0, L_cap, h1, ws)
    kc, vc = make_caches(kp, vp, L_cap)
    ws.fill_(0xFF)
    fb.fastvar_block_forward_pruned(x, N, None, B, N, d, ws_struct, kc, vc, L0, L_cap, y, ws)
    torch.cuda.synchronize()
    yo, kn, vn, parts = O.block_forward_pruned(x_np, W, dims.H, kp, vp, return_parts=True)
    got, mid = from_dev_bf16(y), from_dev_bf16(h1)
    mid64 = mid.astype(np.float64)
    ffn = O.ffn_sublayer_pruned(mid64, W)
    kg, vg = cache_rows(kc, vc, L0, L0 + N)
    assert max(max_rel(got, yo), max_rel(mid, parts["h1"]), max_rel(kg, kn), max_rel(vg, vn),
               branch_error(mid, x_np, parts["h1"] - x_np, parts["h1"]),
               branch_error(got, mid64, ffn - mid64, ffn)) <= 2e-2


@pytest.mark.parametrize("rope", [False, True], ids=["plain", "rope"])
@pytest.mark.parametrize("dims", [synth.BlockDims(D=64, H=1, dh=64, F=64), synth.BlockDims(D=576, H=9, dh=64, F=2304), synth.D16,
                                  synth.BlockDims(D=1088, H=17, dh=64, F=1088), synth.D30, synth.INF2B,
                                  synth.BlockDims(D=2304, H=18, dh=128, F=4608)], ids=lambda d: f"D{d.D}")
def test_identity_list_is_bit_equal_to_no_list(dims, rope):
    """Every token kept, by an index list (LayerNorm in the gather's launch) and without one (up to 16 rows and 2048 columns
    in front of the product): the same sums in the same order, up to 16 rows and just beyond."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(dims.D)

    def rand(*shape, scale=1.0):
        return (torch.randn(shape, generator=gen, device=DEV) * scale).to(torch.bfloat16)

    D, H, dh, F = dims.D, dims.H, dims.dh, dims.F
    wt = dict(ln1_g=1 + rand(D, scale=0.1), ln1_b=rand(D, scale=0.1), w_qkv=rand(3 * D, D, scale=0.05), b_qkv=rand(3 * D),
              w_proj=rand(D, D, scale=0.05), b_proj=rand(D), ln2_g=1 + rand(D, scale=0.1), ln2_b=rand(D, scale=0.1),
              w_fc1=rand(F, D, scale=0.05), b_fc1=rand(F), w_fc2=rand(D, F, scale=0.05), b_fc2=rand(D))
    d, w = fb.make_dims(D, H, dh, F), fb.make_weights(wt)
    for B, h, wd, L0 in ((1, 1, 1, 0), (2, 2, 2, 3), (3, 1, 5, 9), (1, 3, 3, 5), (1, 4, 4, 30), (1, 1, 17, 4)):
        N = h * wd
        L_cap = (L0 + N + 7) // 8 * 8
        x, kc0, vc0 = rand(B, N, D, scale=3.0), rand(B, H, L_cap, dh), rand(B, H, dh, L_cap)
        cos, sin = (torch.empty(N, dh // 2, device=DEV) for _ in range(2))
        fb.fastvar_rope2d_table(h, wd, dh, 10000.0, h, wd, cos, sin)
        ws = empty_ws(fb.fastvar_block_workspace_bytes(d, B, N))
        got = []
        for idx in (None, torch.arange(N, dtype=torch.int32, device=DEV).repeat(B, 1).contiguous()):
            y, kc, vc = torch.empty_like(x), kc0.clone(), vc0.clone()
            ws.fill_(0xFF)
            if rope:
                fb.fastvar_block_forward_pruned_rope(x, N, idx, B, N, d, w, cos, sin, kc, vc, L0, L_cap, y, ws)
            else:
                fb.fastvar_block_forward_pruned(x, N, idx, B, N, d, w, kc, vc, L0, L_cap, y, ws)
            got.append((y, kc, vc))
        torch.cuda.synchronize()
        for a, b, what in zip(*got, ("y", "k", "v")):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16)), (what, B, N, L0)


@pytest.mark.parametrize("dims,B,N", [(synth.BlockDims(D=256, H=2, dh=128, F=512), 1, 12), (synth.BlockDims(D=256, H=2, dh=128, F=512), 3, 5),
                                      (synth.INF2B, 1, 16)], ids=["D256_b1", "D256_b3", "D2048"])
def test_few_rows_over_a_long_cache(dims, B, N):
    """Attention splits the keys between workgroups (heads of 128, 2048 keys or more): its arrival counters are cleared by the
    product with the LayerNorm in front, out of scratch that holds 0xFF."""
    test_block_all_tokens_kept_without_an_index_list(dims, B, N, 2200)


@pytest.mark.parametrize("name,dims,B,h,w,L0", [
    ("D192", synth.BlockDims(D=192, H=3, dh=64, F=320), 3, 1, 5, 29), ("D1024", synth.D16, 2, 2, 4, 11),
    ("D2048", synth.INF2B, 1, 4, 4, 14), ("D2176", synth.BlockDims(D=2176, H=17, dh=128, F=2240), 2, 2, 2, 5)],
    ids=["D192", "D1024", "D2048", "D2176"])
def test_rope_without_an_index_list(name, dims, B, h, w, L0):
    """A token's slot is its row within its sample; with the LayerNorm in front of the product and, at 2176 columns, not."""
    check_block_rope(name, dims, B, h, w, h * w, L0, (L0 + h * w + 7) // 8 * 8, seed=27)


@pytest.mark.parametrize("M,N,K", [(1, 72, 64), (3, 72, 192), (5, 72, 576), (16, 72, 4096), (16, 72, 4160), (8, 72, 8192), (9, 72, 8192),
                                   (1, 72, 65536), (1, 72, 65600), (1, 4096, 2048)])
def test_rows_through_lds(M, N, K):
    """Rows that are not whole loads of 64 chunks, the most that LDS takes (128 KB) and one turn or row more, one of them in many
    rounds of weights; one row over a round of K, in LDS in front of a residual and not in front of GELU."""
    test_gemm_few_rows(M, N, K, fb.EPI_BIAS_RES)
    test_gemm_few_rows(M, N, K, fb.EPI_BIAS_GELU)


@pytest.mark.parametrize("B,N", [(1, 1), (1, 16), (3, 5)])
def test_workgroups_of_twelve_columns(B, N):
    """4160 columns behind the LayerNorm: 347 workgroups of twelve, the last of eight."""
    test_block_all_tokens_kept_without_an_index_list(synth.BlockDims(D=128, H=2, dh=64, F=4160), B, N, 6)
