"""The layer around the chunk loop on the GPU, through the C ABI: the
projection GEMM, the rotation table, the QKV projection with its fused split
and rotation, and the whole layer, each against the float64 oracle of
``oracle/layer.py``.

Tolerances (bf16 operands, fp32 accumulation, outputs rounded to bf16):
  * projection GEMM: every element within 2^-8 |ref| + 2^-8 max|ref| (the
    output rounding is 2^-9 relative; fp32 storage is rounded to bf16 on
    load, which adds about 2^-9 sqrt(2) relative);
  * rotation table: within 2e-7 of float64 cos / sin (the fp32 rounding);
  * QKV projection: as the GEMM (the rotation is done in fp32 on the fp32
    accumulator before the one rounding);
  * layer: max-abs error within 2e-2 max|ref|, the attention tolerance
    normalised by the output's scale.
Across chunkings and scheduling modes the layer output is bit-identical.
"""
import numpy as np
import pytest
import torch

from paper_2607_01817_amd import inputs
from oracle import layer as olayer
from tests import gemm_shapes as gs
from tests.gpu_util import bits, log

pytestmark = pytest.mark.gpu


def _f64(t: torch.Tensor) -> np.ndarray:
    return t.detach().to(torch.float64).cpu().numpy()


def _check_close(got: np.ndarray, want: np.ndarray, what: str, rel_max: float = 2.0 ** -8):
    scale = float(np.abs(want).max()) if want.size else 0.0
    err = np.abs(got - want)
    bound = rel_max * np.abs(want) + rel_max * scale
    bad = int((err > bound).sum())
    worst = float(err.max()) if err.size else 0.0
    log(f"    {what}: max-abs {worst:.3e} (max|ref| {scale:.3e})")
    assert np.all(np.isfinite(got)), f"{what}: non-finite output"
    assert bad == 0, f"{what}: {bad} elements outside {rel_max:g}(|ref| + max|ref|), worst {worst:.3e}"


@pytest.mark.parametrize("M,N,K,dtype", [
    (1, 8, 64, torch.bfloat16), (300, 264, 128, torch.bfloat16), (257, 520, 640, torch.bfloat16),
    (512, 256, 256, torch.bfloat16), (77, 40, 192, torch.float32), (256, 512, 64, torch.float32),
    (2049, 8200, 320, torch.bfloat16), (2049, 8200, 192, torch.float32)])
def test_linear_matches_oracle(hcms, M, N, K, dtype):
    """Row, column and tile tails, both storage types; the last two have more
    tiles (9 x 33) than CUs and a short K, so persistent workgroups take
    several tiles each, with an odd number of k-blocks (fp32, K = 192)."""
    log(f"[linear] M={M} N={N} K={K} {dtype}")
    g = torch.Generator().manual_seed(M * 1000 + N + K)
    x = torch.randn(M, K, generator=g).to(dtype)
    w = (torch.randn(N, K, generator=g) / K ** 0.5).to(dtype)
    got = hcms.linear(x.cuda(), w.cuda())
    want = olayer.linear(_f64(x), _f64(w).T)
    _check_close(_f64(got), want, "linear", 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -7)


def test_linear_empty_and_deterministic(hcms):
    x = torch.randn(0, 64).to(torch.bfloat16).cuda()
    w = torch.randn(8, 64).to(torch.bfloat16).cuda()
    assert hcms.linear(x, w).shape == (0, 8)
    x = torch.randn(1000, 256).to(torch.bfloat16).cuda()
    w = torch.randn(520, 256).to(torch.bfloat16).cuda()
    a = hcms.linear(x, w)
    b = hcms.linear(x, w)
    torch.cuda.synchronize()
    assert torch.equal(bits(a.cpu()), bits(b.cpu()))


@pytest.mark.parametrize("shape", [(56160, 1920, 5120), (56160, 5120, 640)])
def test_linear_sampled_rows_at_the_layer_shapes(hcms, shape):
    """The Wan2.2-shaped QKV projection (5 heads) and output projection of
    the bench's layer, checked on 32 sampled rows."""
    M, N, K = shape
    log(f"[linear] layer shape M={M} N={N} K={K}")
    g = torch.Generator().manual_seed(N + K)
    x = torch.randn(M, K, generator=g).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g) / K ** 0.5).to(torch.bfloat16)
    got = hcms.linear(x.cuda(), w.cuda()).cpu()
    rows = np.sort(np.random.default_rng(N).choice(M, 32, replace=False))
    want = olayer.linear(_f64(x[rows]), _f64(w).T)
    _check_close(_f64(got[rows]), want, "linear rows")


def _table_lookup(table: np.ndarray, w, tokens: np.ndarray) -> np.ndarray:
    """(cos, sin) [len(tokens)][d/2][2] read from the table by its documented
    layout: axis a's entries start after those of the earlier axes, then
    coordinate-major, pair-minor."""
    coords = olayer.grid_coords(w.grid)[tokens]
    out = np.empty((len(tokens), w.d // 2, 2))
    off, p0 = 0, 0
    for a, (G, n) in enumerate(zip(w.grid, w.axis_pairs)):
        for i in range(n):
            out[:, p0 + i, :] = table[off + coords[:, a] * n + i]
        off += G * n
        p0 += n
    return out


@pytest.mark.parametrize("name", ["layer_small", "layer_ragged", "layer_wan_p8"])
def test_rope_table_matches_the_oracle_angles(hcms, name):
    w = inputs.LAYERS[name]
    table = hcms.rope_table(w.grid, w.axis_pairs, w.base).cpu().numpy().astype(np.float64)
    assert table.shape[0] == sum(G * n for G, n in zip(w.grid, w.axis_pairs))
    tokens = inputs.sample_tokens(w, 0 if w.S < 5000 else 512)
    ang = olayer.rope_angles(w.grid, w.axis_pairs, w.base)[tokens]
    got = _table_lookup(table, w, tokens)
    err = max(float(np.abs(got[..., 0] - np.cos(ang)).max()),
              float(np.abs(got[..., 1] - np.sin(ang)).max()))
    log(f"[rope table] {name}: max error {err:.2e}")
    assert err <= 2e-7


def _oracle_qkv(w, x, w_qkv, rows, rotate=True):
    """Oracle q, k, v [len(rows)][H][d] of the token rows."""
    qkv = olayer.linear(_f64(x[rows]), _f64(w_qkv).T)
    q, k, v = olayer.split_qkv(qkv, w.H, w.d)
    if rotate:
        ang = olayer.rope_angles(w.grid, w.axis_pairs, w.base)[rows]
        q, k = olayer.rope(q, ang), olayer.rope(k, ang)
    return q, k, v


@pytest.mark.parametrize("name", ["layer_small", "layer_ragged", "layer_fp32", "layer_wan_p8"])
@pytest.mark.parametrize("rotate", [True, False])
def test_qkv_projection_matches_oracle(hcms, name, rotate):
    w = inputs.LAYERS[name]
    if name == "layer_wan_p8" and not rotate:
        pytest.skip("the unrotated split is covered by the small shapes")
    log(f"[qkv] {name} rotate={rotate}")
    x, w_qkv, _ = inputs.make_layer(w)
    table = hcms.rope_table(w.grid, w.axis_pairs, w.base) if rotate else None
    q, k, v = hcms.qkv_projection(x.cuda(), w_qkv.cuda(), w.H, w.d, table, w.grid, w.axis_pairs)
    rows = inputs.sample_tokens(w)
    want = _oracle_qkv(w, x, w_qkv, rows, rotate)
    rel = 2.0 ** -8 if w.dtype == "bf16" else 2.0 ** -7
    for name_t, got, ref in zip("qkv", (q, k, v), want):
        _check_close(_f64(got.cpu()[rows]), ref, f"{name} {name_t}", rel)


def _oracle_layer(oracle_mod, w, x, w_qkv, w_o, rows):
    ang = olayer.rope_angles(w.grid, w.axis_pairs, w.base)
    return olayer.layer_forward(_f64(x), _f64(w_qkv).T, _f64(w_o).T, ang, w.H, w.d, w.scale,
                                oracle_mod.attention_head, rows)


@pytest.mark.parametrize("name", ["layer_small", "layer_ragged", "layer_fp32", "layer_wan_p8"])
def test_layer_forward_matches_oracle(hcms, oracle_mod, name):
    """Whole layer against the oracle (every token of the small layers; 32
    sampled tokens of the Wan2.2-shaped share, S = 56160, D = 5120)."""
    w = inputs.LAYERS[name]
    log(f"[layer] {name} S={w.S} H={w.H} d={w.d} D={w.D}")
    x, w_qkv, w_o = inputs.make_layer(w)
    table = hcms.rope_table(w.grid, w.axis_pairs, w.base)
    ctx = hcms.Context(max_chunks=8)
    y = ctx.layer_forward(x.cuda(), w_qkv.cuda(), w_o.cuda(), w.P, w.H, w.d, w.scale,
                          w.chunkings[-1], table, w.grid, w.axis_pairs)
    torch.cuda.synchronize()
    ctx.close()
    rows = inputs.sample_tokens(w)
    want = _oracle_layer(oracle_mod, w, x, w_qkv, w_o, rows)
    got = _f64(y.cpu()[rows])
    err = float(np.abs(got - want).max())
    ref = float(np.abs(want).max())
    log(f"    max-abs {err:.3e}, normalised {err / ref:.3e}")
    assert np.all(np.isfinite(got))
    assert err <= 2e-2 * ref


@pytest.mark.parametrize("name", ["layer_small", "layer_ragged"])
def test_layer_forward_bitwise_across_chunkings_and_modes(hcms, name):
    w = inputs.LAYERS[name]
    x, w_qkv, w_o = (t.cuda() for t in inputs.make_layer(w))
    table = hcms.rope_table(w.grid, w.axis_pairs, w.base)
    ctx = hcms.Context(max_chunks=8)
    ref = None
    for sizes in w.chunkings + (tuple([1] * w.H),):
        for mode in (hcms.MODE_SERIAL, hcms.MODE_PIPELINED, hcms.MODE_INLINE, hcms.MODE_LANES,
                     hcms.MODE_AUTO):
            y = ctx.layer_forward(x, w_qkv, w_o, w.P, w.H, w.d, w.scale, sizes, table, w.grid,
                                  w.axis_pairs, mode=mode).clone()
            torch.cuda.synchronize()
            if ref is None:
                ref = bits(y.cpu())
            assert torch.equal(bits(y.cpu()), ref), f"{name}: chunks {sizes} mode {mode} differ"
    ctx.close()


def test_layer_forward_is_the_three_calls(hcms):
    """The layer entry point issues exactly the projection, the chunked
    forward and the output projection: same bits as calling them in turn."""
    w = inputs.LAYERS["layer_ragged"]
    x, w_qkv, w_o = (t.cuda() for t in inputs.make_layer(w))
    table = hcms.rope_table(w.grid, w.axis_pairs, w.base)
    ctx = hcms.Context(max_chunks=8)
    y = ctx.layer_forward(x, w_qkv, w_o, w.P, w.H, w.d, w.scale, (2, 1), table, w.grid,
                          w.axis_pairs).clone()
    q, k, v = hcms.qkv_projection(x, w_qkv, w.H, w.d, table, w.grid, w.axis_pairs)
    o = ctx.forward(q, k, v, w.P, w.scale, (2, 1))
    y2 = hcms.linear(o.view(w.S, w.H * w.d), w_o)
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(bits(y.cpu()), bits(y2.cpu()))


def _dtype(elem_bytes):
    return torch.bfloat16 if elem_bytes == gs.BF16 else torch.float32


def _check_linear(hcms, M, N, K, dtype):
    """Sampled rows against the oracle: one rounding of the exact product,
    bounds as in test_linear_matches_oracle."""
    g = torch.Generator().manual_seed(M + N + K)
    x = torch.randn(M, K, generator=g).to(dtype)
    w = (torch.randn(N, K, generator=g) / K ** 0.5).to(dtype)
    got = hcms.linear(x.cuda(), w.cuda())
    rows = np.unique(np.concatenate([np.arange(0, M, max(1, M // 97)), [M - 1]]))
    want = olayer.linear(_f64(x[rows]), _f64(w).T)
    _check_close(_f64(got[torch.from_numpy(rows).cuda()]), want, "linear",
                 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -7)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M,N,K", [
    (65, 72, 64), (130, 1032, 1024), (1025, 1928, 256), (1025, 15368, 64), (70, 15368, 512),
    (3001, 3008, 64), (3065, 4104, 320), (2000, 4880, 192), (4001, 4008, 64), (4100, 8200, 192)])
def test_linear_tiles_match_oracle(hcms, M, N, K, dtype):
    """Ragged rows and columns, small and large outputs, reductions of one
    stage, odd and even counts."""
    log(f"[linear tiles] M={M} N={N} K={K} {dtype}")
    _check_linear(hcms, M, N, K, dtype)


@pytest.mark.parametrize("tile,more,elem_bytes,M,N,K", gs.LINEAR)
def test_linear_on_every_tile(hcms, tile, more, elem_bytes, M, N, K):
    """Each tile of the GEMM, in one round of workgroups and in more (the host
    test of the tile rule checks that these shapes take it)."""
    log(f"[linear] tile {tile} rounds>1={more} M={M} N={N} K={K} {elem_bytes} bytes")
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    _check_linear(hcms, M, N, K, _dtype(elem_bytes))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("S,D,H,d", [(97, 64, 3, 8), (1301, 192, 5, 128), (3001, 128, 8, 128),
                                     (2600, 64, 13, 128), (4100, 128, 10, 128)])
def test_qkv_tiles_match_linear(hcms, S, D, H, d, dtype):
    """The split of the QKV epilogue at head boundaries inside and across
    segments: without a rotation q, k, v hold the bits of the plain product's
    columns."""
    log(f"[qkv tiles] S={S} D={D} H={H} d={d} {dtype}")
    g = torch.Generator().manual_seed(S + D)
    x = torch.randn(S, D, generator=g).to(dtype).cuda()
    w = (torch.randn(3 * H * d, D, generator=g) / D ** 0.5).to(dtype).cuda()
    qkv = torch.stack(hcms.qkv_projection(x, w, H, d), dim=1)
    plain = hcms.linear(x, w).view(S, 3, H, d)
    assert torch.equal(bits(qkv.cpu()), bits(plain.cpu()))


@pytest.mark.parametrize("tile,more,elem_bytes,grid,D,H,d", gs.QKV)
def test_qkv_on_every_tile(hcms, tile, more, elem_bytes, grid, D, H, d):
    """The split and the rotation of the QKV epilogue on each tile, in one round
    of workgroups and in more: the unrotated features hold the bits of the plain
    product, the rotated ones of sampled tokens are the oracle's."""
    S, dtype = grid[0] * grid[1], _dtype(elem_bytes)
    log(f"[qkv] tile {tile} rounds>1={more} S={S} D={D} H={H} d={d} {elem_bytes} bytes")
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    g = torch.Generator().manual_seed(S + D + H)
    x = torch.randn(S, D, generator=g).to(dtype)
    w = (torch.randn(3 * H * d, D, generator=g) / D ** 0.5).to(dtype)
    pairs = (d // 2 - 22, 22)
    q, k, v = hcms.qkv_projection(x.cuda(), w.cuda(), H, d, hcms.rope_table(grid, pairs, 10000.0), grid, pairs)
    plain = hcms.linear(x.cuda(), w.cuda()).view(S, 3, H, d)
    unrotated = torch.stack(hcms.qkv_projection(x.cuda(), w.cuda(), H, d), dim=1)
    assert torch.equal(bits(unrotated), bits(plain)) and torch.equal(bits(v.contiguous()), bits(plain[:, 2].contiguous()))
    rows = np.unique(np.concatenate([np.arange(0, S, max(1, S // 61)), [S - 1]]))
    wq, wk, _ = olayer.split_qkv(olayer.linear(_f64(x[rows]), _f64(w).T), H, d)
    ang = olayer.rope_angles(grid, pairs, 10000.0)[rows]
    rel = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -7
    for nm, got, want in (("q", q, wq), ("k", k, wk)):
        _check_close(_f64(got.cpu()[rows]), olayer.rope(want, ang), nm, rel)
