"""GPU parity of the tile shapes of the products, of out-proj and FC2 where their K is cut into slices, and of the launch that adds the slices up: rows one
short of, at and past the tiles that the plan picks, two to eight slices, one to nine 512-column groups (whole and
part-filled), with the LayerNorm behind the sum (out-proj in a block), without (its own entry point, a block's FC2) and with the
kept rows scattered into a map (a step).  Same bars as test_gpu_4_block.py, whose checks these are."""
import pytest
import torch

from paper_2503_23367_amd import binding as fb
from paper_2503_23367_amd import synth
from gpu_util import DEV, empty_ws
from tile_cases import QKV_SEAMS, QKV_TILES, ROPE_TILES, SEAMS, SLICED_ALONE, SLICED_DIMS, SLICED_ROWS, TILES
from test_gpu_3_components import test_qkv_gemm_appends_to_caches as check_qkv
from test_gpu_4_block import check_block

pytestmark = pytest.mark.gpu

@pytest.mark.parametrize("M,N,K,epi", [c for cases in [*TILES.values(), *SEAMS.values()] for c in cases])
def test_tiles(M, N, K, epi):
    """Every tile shape (tile_cases.py), against fp32."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(M + K)
    A, W, bias, res = (torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16) for s in ((M, K), (N, K), (N,), (M, N)))
    W = (W * 0.2).contiguous()
    out = torch.full((M * N + 4096,), float("nan"), dtype=torch.bfloat16, device=DEV)
    fb.fastvar_gemm_bf16(A, W, bias, res, M, N, K, epi, out)
    lin = torch.addmm(bias.float(), A.float(), W.float().T)
    ref = lin + res.float() if epi == fb.EPI_BIAS_RES else torch.nn.functional.gelu(lin)
    assert out[M * N:].isnan().all()
    err = (out[:M * N].view(M, N).float() - ref).abs().max() / ref.abs().max()
    assert err <= 2.0 ** -7, float(err)


@pytest.mark.parametrize("D,dh,B,k", list(QKV_TILES.values()))
def test_qkv_tiles(D, dh, B, k):
    check_qkv(_dims(D, D // dh, dh, D), B, k, 5, (5 + k + 7) // 8 * 8)


@pytest.mark.parametrize("rope", [False, True], ids=["plain", "rope"])
@pytest.mark.parametrize("D,dh,B,k", [*QKV_SEAMS.values(), *ROPE_TILES.values()])
def test_qkv_tiles_and_seams(D, dh, B, k, rope):
    """Queries, keys and values of every tile and over the seams between a workgroup's tiles, against fp32; the kept slots of a larger map."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(D + k)
    H, N, L0 = D // dh, k + 13, 5
    L_cap = (L0 + k + 7) // 8 * 8 + 8
    A, W, bias = (torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16) for s in ((B * k, D), (3 * D, D), (3 * D,)))
    W = (W * 0.2).contiguous()
    idx = torch.stack([torch.randperm(N, generator=gen, device=DEV)[:k].sort().values for _ in range(B)]).to(torch.int32)
    angle = torch.rand((N, dh // 2), generator=gen, device=DEV) * 6.3
    cos, sin = angle.cos().contiguous(), angle.sin().contiguous()
    q = torch.full((B, k, D), float("nan"), dtype=torch.bfloat16, device=DEV)
    kc, vc = (torch.full((B, H, *s), float("nan"), dtype=torch.bfloat16, device=DEV) for s in ((L_cap, dh), (dh, L_cap)))
    d = fb.make_dims(D, H, dh, D)
    if rope:
        fb.fastvar_qkv_gemm_rope(A, W, bias, idx, B, N, k, d, cos, sin, q, kc, vc, L0, L_cap)
    else:
        fb.fastvar_qkv_gemm(A, W, bias, B, k, d, q, kc, vc, L0, L_cap)
    ref = torch.addmm(bias.float(), A.float(), W.float().T).view(B, k, 3, H, dh)
    if rope:
        c, s = (t[idx.long()].view(B, k, 1, dh // 2) for t in (cos, sin))
        for part in (0, 1):
            a, b = ref[:, :, part, :, 0::2].clone(), ref[:, :, part, :, 1::2].clone()
            ref[:, :, part, :, 0::2], ref[:, :, part, :, 1::2] = a * c - b * s, a * s + b * c
    got = (q.view(B, k, H, dh), kc[:, :, L0:L0 + k].permute(0, 2, 1, 3), vc[..., L0:L0 + k].permute(0, 3, 1, 2))
    for part, g in enumerate(got):
        err = (g.float() - ref[:, :, part]).abs().max() / ref[:, :, part].abs().max()
        assert err <= 2.0 ** -7, (part, float(err))
    for t, axis in ((kc, 2), (vc, 3)):
        assert t.narrow(axis, 0, L0).isnan().all() and t.narrow(axis, L0 + k, L_cap - L0 - k).isnan().all()


def _dims(D, H, dh, F):
    return synth.BlockDims(D=D, H=H, dh=dh, F=F)


DIMS = [_dims(*d) for d in SLICED_DIMS]


@pytest.mark.parametrize("dims,B,h,w,k", [(d, *r) for d in DIMS for r in SLICED_ROWS] + [(_dims(*SLICED_ALONE[0]), *SLICED_ALONE[1])],
                         ids=lambda v: f"D{v.D}" if isinstance(v, synth.BlockDims) else str(v))
def test_block(dims, B, h, w, k):
    check_block(f"slices_{dims.D}", dims, B, h, w, k, 21, (21 + k + 7) // 8 * 8 + 8, seed=31)


@pytest.mark.parametrize("dims", DIMS[:3] + [synth.INF2B], ids=lambda d: f"D{d.D}")
@pytest.mark.parametrize("B,h,w,k", [(1, 8, 8, 31), (2, 12, 13, 70), (1, 24, 24, 400), (1, 30, 31, 929)])
def test_step_scatters_the_rows_of_the_block(dims, B, h, w, k):
    """The kept rows of a step's map are the block's own output for the step's index list, bit for bit."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(k)

    def rand(*shape, scale=1.0):
        return (torch.randn(shape, generator=gen, device=DEV) * scale).to(torch.bfloat16)

    D, H, dh, F, N, L0 = dims.D, dims.H, dims.dh, dims.F, h * w, 19
    wt = dict(ln1_g=1 + rand(D, scale=0.1), ln1_b=rand(D, scale=0.1), w_qkv=rand(3 * D, D, scale=0.05), b_qkv=rand(3 * D),
              w_proj=rand(D, D, scale=0.05), b_proj=rand(D), ln2_g=1 + rand(D, scale=0.1), ln2_b=rand(D, scale=0.1),
              w_fc1=rand(F, D, scale=0.05), b_fc1=rand(F), w_fc2=rand(D, F, scale=0.05), b_fc2=rand(D))
    d, wts = fb.make_dims(D, H, dh, F), fb.make_weights(wt)
    L_cap = (L0 + k + 7) // 8 * 8
    x, cache, kc0, vc0 = rand(B, N, D), rand(B, 6, D), rand(B, H, L_cap, dh), rand(B, H, dh, L_cap)
    y, y_kept = torch.full_like(x, float("nan")), torch.full((B, k, D), float("nan"), dtype=torch.bfloat16, device=DEV)
    idx = torch.empty((B, k), dtype=torch.int32, device=DEV)
    ws = empty_ws(fb.fastvar_step_workspace_bytes(d, B, N, k))
    ws.fill_(0xFF)
    kc, vc = kc0.clone(), vc0.clone()
    fb.fastvar_step(x, [2, h], [3, w], 1, 0, B, k, d, wts, kc, vc, L0, L_cap, cache, y, idx, ws)
    ws.fill_(0xFF)
    fb.fastvar_block_forward_pruned(x, N, idx, B, k, d, wts, kc0, vc0, L0, L_cap, y_kept, ws)
    torch.cuda.synchronize()
    assert not y.isnan().any()
    assert torch.equal(torch.gather(y, 1, idx.long()[..., None].expand(B, k, D)).view(torch.int16), y_kept.view(torch.int16))


@pytest.mark.parametrize("k", [1, 24, 130])
def test_attention_half_does_not_depend_on_mlp_weights(k):
    """The attention half with MLP weights and with NaN in their place: the same bits.  (What the launch fetches ahead never
    shows in its results; that nothing of the MLP half is on its list is checked in test_launch_math.py.)"""
    dims = synth.INF2B
    gen = torch.Generator(device=DEV)
    gen.manual_seed(k)

    def rand(*shape, scale=1.0):
        return (torch.randn(shape, generator=gen, device=DEV) * scale).to(torch.bfloat16)

    D, H, dh, F, N, L0 = dims.D, dims.H, dims.dh, dims.F, 196, 19
    wt = dict(ln1_g=1 + rand(D, scale=0.1), ln1_b=rand(D, scale=0.1), w_qkv=rand(3 * D, D, scale=0.05), b_qkv=rand(3 * D),
              w_proj=rand(D, D, scale=0.05), b_proj=rand(D), ln2_g=1 + rand(D, scale=0.1), ln2_b=rand(D, scale=0.1),
              w_fc1=rand(F, D, scale=0.05), b_fc1=rand(F), w_fc2=rand(D, F, scale=0.05), b_fc2=rand(D))
    d = fb.make_dims(D, H, dh, F)
    L_cap = (L0 + k + 7) // 8 * 8
    x, kc0, vc0 = rand(1, N, D), rand(1, H, L_cap, dh), rand(1, H, dh, L_cap)
    idx = torch.arange(k, dtype=torch.int32, device=DEV).view(1, k)
    ws = empty_ws(fb.fastvar_block_workspace_bytes(d, 1, k))
    out = []
    for weights in (wt, dict(wt, w_fc1=torch.full_like(wt["w_fc1"], float("nan")), w_fc2=torch.full_like(wt["w_fc2"], float("nan")))):
        kc, vc, y = kc0.clone(), vc0.clone(), torch.full((1, k, D), float("nan"), dtype=torch.bfloat16, device=DEV)
        fb.fastvar_attn_forward_pruned(x, N, idx, 1, k, d, fb.make_weights(weights), kc, vc, L0, L_cap, y, ws)
        out.append((y, kc, vc))
    for a, b in zip(*out):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
