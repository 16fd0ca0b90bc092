"""GPU parity: the HIP library (through its C ABI) against the fp64 CPU oracle on the same seeded inputs.

Error metric (the one the target is stated in): max|Y_gpu - Y_ref| / max|Y_ref| over the whole output.
Bars: bf16 path <= 2e-2, fp32 debug path <= 1e-5.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2510_25977_amd import binding as B
from paper_2510_25977_amd import synth

pytestmark = pytest.mark.gpu

BF16_TOL = 2e-2
F32_TOL = 1e-5


def dev():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return torch.device("cuda:0")


def relmax(y, ref):
    return float(np.max(np.abs(y - ref)) / np.max(np.abs(ref)))


def relfro(y, ref):
    return float(np.linalg.norm(y - ref) / np.linalg.norm(ref))


def run_gated(gi, flags=0, max_M=None, rows=None):
    """Forward on the GPU; oracle on `rows` (default all).  Returns (Y_gpu rows, Y_ref rows, path)."""
    d = dev()
    f = {k: v.to(d) for k, v in gi.factors().items()}
    mlp = B.SvdMlp(max_M=max_M or gi.X.shape[0], flags=flags, **f)
    Y = mlp(gi.X.to(d))
    torch.cuda.synchronize()
    path = mlp.last_path
    Yh = Y.cpu().to(torch.float64).numpy()
    mlp.close()
    a = {k: synth.to_f64(v) for k, v in gi.factors().items()}
    X = synth.to_f64(gi.X)
    if rows is not None:
        X, Yh = X[rows], Yh[rows]
    ref = oracle.gated(X, **a)
    return Yh, ref, path


# ---------------------------------------------------------------------------------- fp32 debug path
@pytest.mark.parametrize("r", [16, 256])
def test_f32_linear_powerlaw(r):
    """Single factored linear layer, fp32, M=32, d=256, n=1024, W = Q1 diag(i^-0.7) Q2^T."""
    li = synth.make_linear_powerlaw(r=r)
    d = dev()
    mlp = B.SvdMlp(max_M=32, Ug=li.U.to(d), Vg=li.V.to(d), kind=B.SVDMLP_LINEAR)
    Y = mlp(li.X.to(d)).cpu().to(torch.float64).numpy()
    assert mlp.last_path == 1
    ref = oracle.linear(synth.to_f64(li.X), synth.to_f64(li.U), synth.to_f64(li.V))
    assert relmax(Y, ref) <= F32_TOL
    if r == 256:
        # full rank: the factored product is X W itself (up to the fp32 rounding of the stored factors)
        assert relmax(Y, synth.to_f64(li.X) @ li.W) <= 1e-5


@pytest.mark.parametrize("M,d,ffn,r,rd", [(37, 96, 200, 24, 40), (130, 256, 640, 64, 128), (1, 64, 64, 8, 8)])
def test_f32_gated_ragged(M, d, ffn, r, rd):
    gi = synth.make_gated(M, d, ffn, r, rd, stream=11, dtype=torch.float32)
    Y, ref, path = run_gated(gi)
    assert path == 1
    assert relmax(Y, ref) <= F32_TOL

@pytest.mark.parametrize("M,d,ffn,r,rd", [
    (31, 64, 64, 4, 4), (32, 65, 63, 5, 6), (33, 260, 61, 7, 61),      # edges of the 32- and 64-row tiles, one step +- 1
    (64, 1028, 1536, 66, 130), (65, 1027, 1537, 67, 129),              # rows of 16 bytes and not; several ranges of K, odd ones
    (200, 4096, 2048, 128, 64), (3, 4100, 8191, 255, 257),             # the most ranges; a short last range
    (1100, 1030, 1100, 100, 200),                                      # a product of more than 256 tiles
])
def test_f32_gated_tile_and_range_edges(M, d, ffn, r, rd):
    gi = synth.make_gated(M, d, ffn, r, rd, stream=12, dtype=torch.float32)
    Y, ref, path = run_gated(gi)
    assert path == 1
    assert relmax(Y, ref) <= F32_TOL


@pytest.mark.parametrize("M,d,ffn,r,rd", [
    (1, 1, 1, 1, 1), (3, 3, 5, 3, 2), (5, 4, 6, 4, 3), (33, 5, 7, 3, 4),       # rows shorter than, as long as and longer than four floats
    (40, 65, 66, 5, 7), (65, 63, 67, 62, 61), (70, 130, 257, 66, 65),          # every remainder, on either side of a step and a tile
    (100, 515, 1026, 131, 129),                                                # ranges over the contraction, the last one ragged
])
def test_f32_rows_of_any_length(M, d, ffn, r, rd):
    """Rows whose length is no multiple of four are loaded sixteen bytes at a time too, the last four floats of a row shifted
    into place: what is checked here is the values.  Inputs and factors lie in buffers full of NaN, which would show if
    a value from beyond them were used.  (A load past the end of a row whose values are dropped would not show: what lies
    beyond a contraction is zeroed and columns beyond the output are not stored.  A host test checks the addresses.)"""
    gi = synth.make_gated(M, d, ffn, r, rd, stream=85, dtype=torch.float32)

    def buried(t):
        buf = torch.full((t.numel() + 16,), float("nan"), device=dev())
        buf[4:4 + t.numel()] = t.to(dev()).reshape(-1)
        return buf[4:4 + t.numel()].view(t.shape)

    mlp = B.SvdMlp(max_M=M, **{k: buried(v) for k, v in gi.factors().items()})
    Y = mlp(buried(gi.X)).cpu().to(torch.float64).numpy()
    mlp.close()
    ref = oracle.gated(synth.to_f64(gi.X), **{k: synth.to_f64(v) for k, v in gi.factors().items()})
    assert np.isfinite(Y).all()
    assert relmax(Y, ref) <= F32_TOL


def test_f32_output_of_four_million_tiles():
    """O[2^20, 16384] (64 GiB) is 2^14 x 2^8 tiles of 64 x 64, more than a launch of 512-thread workgroups can number in one
    grid dimension of 2^31 threads.  Rows at the edges of tiles and at random, every column."""
    M, d, n, r = 1 << 20, 32, 16384, 8
    dv = dev()
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GiB of device memory")
    g = torch.Generator(device=dv)
    g.manual_seed(13)
    U, V = torch.randn(d, r, generator=g, device=dv), torch.randn(r, n, generator=g, device=dv)
    X = torch.randn(M, d, generator=g, device=dv)
    mlp = B.SvdMlp(max_M=M, Ug=U, Vg=V, kind=B.SVDMLP_LINEAR)
    O = torch.empty((M, n), device=dv)
    rows = torch.tensor([0, 63, 64, 4095, (1 << 18) - 1, 1 << 18, M // 2 + 31, M - 64, M - 1], device=dv)
    rows = torch.cat([rows, torch.randint(M, (40,), generator=g, device=dv)])
    O[rows] = -3.0
    mlp(X, O)
    got = O[rows].double()
    assert mlp.last_path == 1
    mlp.close()
    del O
    torch.cuda.empty_cache()
    ref = X[rows].double() @ U.double() @ V.double()
    assert float((got - ref).abs().max() / ref.abs().max()) <= F32_TOL


# ---------------------------------------------------------------------------------- bf16 tiled path
@pytest.mark.parametrize("M,d,ffn,r,rd", [
    (128, 128, 128, 128, 128),     # one tile of everything
    (200, 256, 384, 128, 128),     # ragged M (two row tiles), several chunks
    (333, 384, 1152, 192, 256),    # three row tiles, r not a power of two, NQ = 8
    (40, 512, 512, 128, 512),      # small M forced onto the tiled path, NQ = 16
    (129, 1024, 1024, 128, 1024),  # down rank split over two workgroups
])
def test_bf16_tiled_small(M, d, ffn, r, rd):
    gi = synth.make_gated(M, d, ffn, r, rd, stream=21)
    Y, ref, path = run_gated(gi, flags=B.FLAG_FORCE_TILED | B.FLAG_TILED_FUSED)
    assert path == 2
    assert relmax(Y, ref) <= BF16_TOL, (relmax(Y, ref), relfro(Y, ref))
    assert relfro(Y, ref) <= 1.5e-2


@pytest.mark.parametrize("M,d,ffn,r,rd", [
    (40, 512, 512, 128, 512),      # one row tile, mostly padding; two column tiles everywhere
    (300, 512, 1024, 192, 256),    # ragged M over two 256-row tiles, r not a power of two
    (520, 768, 512, 256, 512),     # odd number of row tiles, three output column tiles
    (300, 384, 512, 128, 256),     # d not a multiple of 256: the 128-column output kernel finishes the job
    (129, 1024, 1024, 128, 1024),  # four rank tiles
    (2304, 256, 7680, 128, 256),   # more tiles (9 x 30) than compute units: workgroups of k_gate_up take several
])
def test_bf16_staged_small(M, d, ffn, r, rd):
    """Tiled path with the gated activation staged through the workspace (path 5); the fused variant must agree."""
    gi = synth.make_gated(M, d, ffn, r, rd, stream=22)
    big = M > 1000
    rows = list(range(0, M, 97)) + [M - 1] if big else None
    Y, ref, path = run_gated(gi, flags=B.FLAG_FORCE_TILED, rows=rows)
    assert path == 5
    assert relmax(Y, ref) <= BF16_TOL, (relmax(Y, ref), relfro(Y, ref))
    assert relfro(Y, ref) <= 1.5e-2
    Yf, _, pathf = run_gated(gi, flags=B.FLAG_FORCE_TILED | B.FLAG_TILED_FUSED, rows=rows)
    assert pathf == 2
    assert relmax(Y, Yf) <= BF16_TOL


# ---------------------------------------------------------------------------------- bf16 single factored layer
@pytest.mark.parametrize("M,d,n,r", [
    (70, 256, 512, 128),       # one row tile, mostly padding
    (300, 384, 640, 256),      # n not a multiple of 256: 128-column output kernel
    (513, 1024, 768, 384),     # three 256-row tiles, r not a power of two
])
def test_bf16_linear_small(M, d, n, r):
    """O = (X U) V in bf16 (path 6) against the oracle's plain chain."""
    li = synth.make_linear_gaussian(M, d, n, r, stream=41)
    dv = dev()
    mlp = B.SvdMlp(max_M=M, Ug=li.U.to(dv), Vg=li.V.to(dv), kind=B.SVDMLP_LINEAR)
    O = mlp(li.X.to(dv))
    torch.cuda.synchronize()
    assert mlp.last_path == (7 if M <= 128 else 6) and tuple(O.shape) == (M, n)
    Oh = O.cpu().to(torch.float64).numpy()
    mlp.close()
    ref = oracle.linear(synth.to_f64(li.X), synth.to_f64(li.U), synth.to_f64(li.V))
    assert relmax(Oh, ref) <= BF16_TOL, (relmax(Oh, ref), relfro(Oh, ref))
    assert relfro(Oh, ref) <= 1.5e-2


def test_bf16_linear_many_tiles_uses_256_tile_first_stage():
    """Enough 256 x 256 tiles of T for the eight-wave first-stage kernel (k_in instead of k_s1); ragged M."""
    M, d, n, r = 3000, 4096, 4096, 4096
    li = synth.make_linear_gaussian(M, d, n, r, stream=43)
    dv = dev()
    mlp = B.SvdMlp(max_M=M, Ug=li.U.to(dv), Vg=li.V.to(dv), kind=B.SVDMLP_LINEAR)
    B.svdmlp_profile_begin(mlp.ctx, 1)
    O = mlp(li.X.to(dv))
    torch.cuda.synchronize()
    kernels, _ = B.svdmlp_profile_end(mlp.ctx)
    assert "k_in" in kernels, kernels
    rows = list(range(0, M, 61)) + [M - 1]
    Oh = O[rows].cpu().to(torch.float64).numpy()
    mlp.close()
    ref = oracle.linear(synth.to_f64(li.X)[rows], synth.to_f64(li.U), synth.to_f64(li.V))
    assert relmax(Oh, ref) <= BF16_TOL, relmax(Oh, ref)


def test_bf16_gated_many_tiles_uses_256_tile_first_stage():
    M, d, ffn, r, rd = 6000, 1024, 1024, 1024, 256
    gi = synth.make_gated(M, d, ffn, r, rd, stream=44)
    rows = list(range(0, M, 113)) + [M - 1]
    Y, ref, path = run_gated(gi, rows=rows)
    assert path == 5
    assert relmax(Y, ref) <= BF16_TOL, relmax(Y, ref)
    Yf, _, _ = run_gated(gi, rows=rows, flags=B.FLAG_TILED_FUSED)
    assert relmax(Yf, ref) <= BF16_TOL


def kernel_names(mlp, X):
    """Names of the kernels one forward launches (from the library's per-kernel event profile)."""
    B.svdmlp_profile_begin(mlp.ctx, 1)
    mlp(X)
    k, _ = B.svdmlp_profile_end(mlp.ctx)
    return list(k)


def test_bf16_linear_on_128_tiles_on_request():
    """SVDMLP_FLAG_TILE_128: the same layer as above on k_s1 + k_s5 (the small-block point of the block-size
    comparison); same parity bar, and bitwise reproducible."""
    M, d, n, r = 3000, 4096, 4096, 4096
    li = synth.make_linear_gaussian(M, d, n, r, stream=43)
    dv = dev()
    mlp = B.SvdMlp(max_M=M, Ug=li.U.to(dv), Vg=li.V.to(dv), kind=B.SVDMLP_LINEAR, flags=B.FLAG_TILE_128)
    X = li.X.to(dv)
    assert kernel_names(mlp, X) == ["k_s1", "k_s5"]
    O = mlp(X)
    O2 = mlp(X)
    torch.cuda.synchronize()
    assert torch.equal(O, O2)
    rows = list(range(0, M, 61)) + [M - 1]
    Oh = O[rows].cpu().to(torch.float64).numpy()
    mlp.close()
    ref = oracle.linear(synth.to_f64(li.X)[rows], synth.to_f64(li.U), synth.to_f64(li.V))
    assert relmax(Oh, ref) <= BF16_TOL, relmax(Oh, ref)


def test_bf16_first_stage_cuts_a_long_contraction_when_tiles_are_few():
    """32 tiles (256 x 256) of T and d = 16384: the eight-wave first-stage kernel runs over eight ranges of d and
    k_reduce adds them (linear layer and gated MLP); ragged M; the oracle evaluates a sample of rows."""
    dv = dev()
    rows = list(range(0, 1000, 37)) + [255, 256, 999]
    li = synth.make_linear_gaussian(1000, 16384, 2048, 2048, stream=46)
    mlp = B.SvdMlp(max_M=1000, Ug=li.U.to(dv), Vg=li.V.to(dv), kind=B.SVDMLP_LINEAR)
    Xd = li.X.to(dv)
    assert kernel_names(mlp, Xd)[0] == "k_in"
    O = mlp(Xd)
    torch.cuda.synchronize()
    Oh = O[rows].cpu().to(torch.float64).numpy()
    mlp.close()
    ref = oracle.linear(synth.to_f64(li.X)[rows], synth.to_f64(li.U), synth.to_f64(li.V))
    assert relmax(Oh, ref) <= BF16_TOL, relmax(Oh, ref)

    gi = synth.make_gated(1000, 16384, 1024, 1024, 256, stream=47)
    f = {k: v.to(dv) for k, v in gi.factors().items()}
    mlp = B.SvdMlp(max_M=1000, **f)
    Xd = gi.X.to(dv)
    assert kernel_names(mlp, Xd)[0] == "k_in"
    Y = mlp(Xd)
    Y2 = mlp(Xd)
    torch.cuda.synchronize()
    assert mlp.last_path == 5 and torch.equal(Y, Y2)
    Yh = Y[rows].cpu().to(torch.float64).numpy()
    mlp.close()
    ref = oracle.gated(synth.to_f64(gi.X)[rows], **{k: synth.to_f64(v) for k, v in gi.factors().items()})
    assert relmax(Yh, ref) <= BF16_TOL, relmax(Yh, ref)


def test_bf16_linear_paper_kernel_shape_sampled_rows():
    """The paper's kernel-evaluation shape X[M,8192] U[8192,4096] V[4096,16384] (Sec. 5.2) at M = 1024; the
    oracle evaluates a sample of rows."""
    li = synth.make_linear_gaussian(1024, 8192, 16384, 4096, stream=42)
    dv = dev()
    mlp = B.SvdMlp(max_M=1024, Ug=li.U.to(dv), Vg=li.V.to(dv), kind=B.SVDMLP_LINEAR, keep_factors=False)
    O = mlp(li.X.to(dv))
    torch.cuda.synchronize()
    rows = [0, 31, 32, 255, 256, 700, 1023]
    Oh = O[rows].cpu().to(torch.float64).numpy()
    mlp.close()
    ref = oracle.linear(synth.to_f64(li.X)[rows], synth.to_f64(li.U), synth.to_f64(li.V))
    assert relmax(Oh, ref) <= BF16_TOL, relmax(Oh, ref)


# ---------------------------------------------------------------------------------- bf16 streaming path
@pytest.mark.parametrize("M", [1, 4, 16, 32, 7])
@pytest.mark.parametrize("d,ffn,r,rd", [(256, 512, 128, 128), (512, 1408, 192, 256)])
@pytest.mark.parametrize("one_kernel", [False, True])
def test_bf16_stream_small(M, d, ffn, r, rd, one_kernel):
    """Weight-streaming path: as four launches (path 3, the default) and as one persistent kernel (path 4)."""
    gi = synth.make_gated(M, d, ffn, r, rd, stream=31)
    Y, ref, path = run_gated(gi, max_M=32, flags=B.FLAG_STREAM_ONE_KERNEL if one_kernel else 0)
    assert path == (4 if one_kernel else 3)
    assert relmax(Y, ref) <= BF16_TOL, (relmax(Y, ref), relfro(Y, ref))
    assert relfro(Y, ref) <= 1.5e-2


@pytest.mark.parametrize("M", [33, 48, 64, 65, 100, 128])
@pytest.mark.parametrize("d,ffn,r,rd", [(256, 512, 128, 128), (512, 1408, 192, 256)])
def test_bf16_stream_several_row_tiles(M, d, ffn, r, rd):
    """Weight-streaming path with the batch padded to two or four 32-row tiles (every weight frag still read once)."""
    gi = synth.make_gated(M, d, ffn, r, rd, stream=33)
    Y, ref, path = run_gated(gi, max_M=128, flags=B.FLAG_FORCE_STREAM)
    assert path == 3
    assert relmax(Y, ref) <= BF16_TOL, (relmax(Y, ref), relfro(Y, ref))
    assert relfro(Y, ref) <= 1.5e-2


@pytest.mark.parametrize("M", [1, 17, 33, 128])
@pytest.mark.parametrize("d,ffn,r,rd", [
    (128, 256, 64, 128),        # fewer contraction blocks than waves
    (1152, 2816, 320, 512),     # groups of the two-buffer loop left half full, in every phase
    (2432, 7424, 576, 768),     # an odd number of groups
])
def test_bf16_stream_contraction_remainders(M, d, ffn, r, rd):
    gi = synth.make_gated(M, d, ffn, r, rd, stream=23)
    Y, ref, path = run_gated(gi)
    assert path == 3
    assert relmax(Y, ref) <= BF16_TOL
    assert relfro(Y, ref) <= 8e-3      # four roundings to bf16; one block left out of the longest contraction: 4e-2


@pytest.mark.parametrize("d,ffn,r,rd", [
    (8192, 512, 100, 130),      # last product on 32-column tiles, a wave has one block
    (8192, 256, 64, 256),       # ranges of D2 and D4 shorter than the waves
    (384, 1536, 330, 300),      # 16-column tiles; the up strip starts inside no tile of 128
])
def test_bf16_stream_batches_of_16_row_operands(d, ffn, r, rd):
    """Up to 32 rows the activations hold the rows of the batch and no others: a row's result must not depend, bit for
    bit, on how many rows there are, on either side of 16."""
    gi = synth.make_gated(32, d, ffn, r, rd, stream=83)
    f = {k: v.to(dev()) for k, v in gi.factors().items()}
    X = gi.X.to(dev())
    mlp = B.SvdMlp(max_M=32, **f)
    full = mlp(X).clone()
    ref = oracle.gated(synth.to_f64(gi.X), **{k: synth.to_f64(v) for k, v in gi.factors().items()})
    assert relmax(full.cpu().to(torch.float64).numpy(), ref) <= BF16_TOL
    assert relfro(full.cpu().to(torch.float64).numpy(), ref) <= 8e-3
    for M in (31, 17, 16, 15, 2, 1):
        Y = torch.full((M + 1, d), 7.0, dtype=torch.bfloat16, device=dev())
        mlp(X[:M].contiguous(), Y[:M])
        torch.cuda.synchronize()
        assert mlp.last_path == 3
        assert torch.equal(Y[:M], full[:M]), M
        assert bool((Y[M] == 7.0).all()), M      # nothing is written past the last row
    mlp.close()


@pytest.mark.parametrize("d,ffn,r,rd", [
    (16512, 16640, 16448, 256),      # the first product has more 16-column tiles than tickets; blocks of D2 in fours
    (33024, 33024, 100, 33024),      # the down projection has; blocks of D2 in twos
    (33024, 33024, 192, 33000),      # ... in threes
])
@pytest.mark.parametrize("M", [3, 32])
def test_bf16_stream_few_rows_beyond_the_tickets_of_16_column_tiles(M, d, ffn, r, rd):
    """Ranks for which up to 32 rows run on the 32-row kernels, against the plain chain in 64 bits on the same device."""
    g = torch.Generator(device=dev())
    g.manual_seed(91)
    u = lambda a, b: (torch.randn(a, b, generator=g, device=dev()) * a ** -0.5).to(torch.bfloat16)
    f = dict(Ug=u(d, r), Vg=u(r, ffn), Uu=u(d, r), Vu=u(r, ffn), Ud=u(ffn, rd), Vd=u(rd, d))
    X = u(M, d) * M ** 0.5
    mlp = B.SvdMlp(max_M=32, **f)
    s = B.svdmlp_describe(mlp.desc, M)
    assert s.startswith("path=3 bf16-streaming: row_tiles=1 k_stream_d1[tiles=") and s.endswith(f"k_stream_d5[tiles={d // 32} row_groups=1]")
    Y = mlp(X)
    assert mlp.last_path == 3 and torch.equal(Y, mlp(X))
    mlp.close()
    x = X.double()
    gate = x @ f["Ug"].double() @ f["Vg"].double()
    up = x @ f["Uu"].double() @ f["Vu"].double()
    ref = (torch.nn.functional.silu(gate) * up @ f["Ud"].double() @ f["Vd"].double()).cpu().numpy()
    y = Y.double().cpu().numpy()
    assert relmax(y, ref) <= BF16_TOL
    assert relfro(y, ref) <= 8e-3      # four roundings to bf16; one of 2064 blocks left out: 2.2e-2


def test_bf16_stream_one_context_many_M():
    """One context, batches on both sides of every row-tile count; within a kernel family (up to 32 rows: 16-row operands;
    33..64 and 65..128 rows: two and four 32-row tiles) a row's result must not depend on M or on what an earlier, larger
    batch left in the workspace, bit for bit; across the families the summation order may differ; the tiled path must
    agree."""
    gi = synth.make_gated(128, 512, 1408, 192, 256, stream=34)
    d = dev()
    f = {k: v.to(d) for k, v in gi.factors().items()}
    X = gi.X.to(d)
    mlp = B.SvdMlp(max_M=128, flags=B.FLAG_FORCE_STREAM, **f)
    full = mlp(X).clone()
    upto64, upto32 = mlp(X[:64]).clone(), mlp(X[:32]).clone()
    for part in (upto64, upto32):
        assert relmax(part.cpu().to(torch.float64).numpy(), full[:len(part)].cpu().to(torch.float64).numpy()) <= 1e-2
    for M in (128, 97, 96, 65, 64, 33, 32, 31, 17, 16, 15, 1, 128, 64):
        y = mlp(X[:M]).clone()
        torch.cuda.synchronize()
        assert mlp.last_path == 3
        assert torch.equal(y, (full if M > 64 else upto64 if M > 32 else upto32)[:M]), M
    mlp.close()
    tiled = B.SvdMlp(max_M=128, flags=B.FLAG_FORCE_TILED, **f)
    yt = tiled(X)
    torch.cuda.synchronize()
    tiled.close()
    a = {k: synth.to_f64(v) for k, v in gi.factors().items()}
    ref = oracle.gated(synth.to_f64(gi.X), **a)
    assert relmax(full.cpu().to(torch.float64).numpy(), ref) <= BF16_TOL
    assert relmax(full.cpu().to(torch.float64).numpy(), yt.cpu().to(torch.float64).numpy()) <= BF16_TOL


def test_bf16_stream_and_tiled_agree_and_are_deterministic():
    gi = synth.make_gated(16, 512, 1408, 128, 256, stream=32)
    d = dev()
    f = {k: v.to(d) for k, v in gi.factors().items()}
    X = gi.X.to(d)
    outs = {}
    for name, flags in (("stream", B.FLAG_FORCE_STREAM), ("stream1", B.FLAG_FORCE_STREAM | B.FLAG_STREAM_ONE_KERNEL),
                        ("tiled", B.FLAG_FORCE_TILED)):
        mlp = B.SvdMlp(max_M=16, flags=flags, **f)
        y1 = mlp(X).clone()
        y2 = mlp(X).clone()
        y3 = mlp(X[:5]).clone()
        torch.cuda.synchronize()
        assert torch.equal(y1, y2), name            # bitwise reproducible
        assert torch.equal(y1[:5], y3), name        # rows do not depend on M
        outs[name] = y1.cpu().to(torch.float64).numpy()
        mlp.close()
    assert relmax(outs["stream"], outs["tiled"]) <= BF16_TOL
    assert relmax(outs["stream1"], outs["tiled"]) <= BF16_TOL


# ---------------------------------------------------------------------------------- full-size workloads
# Besides the stated max-norm bar: relative Frobenius error of the checked rows.  Five roundings to bf16 (T, SiLU(G) in the
# staged variant, H, Td, Y), each a relative error of rms 2^-9 / sqrt(3) = 1.1e-3 that the following products carry on,
# give 3.7e-3 .. 4.2e-3 on every workload here; a contraction block lost anywhere would show as >= 1 / sqrt(blocks)
# (3 % for the 896 blocks of the down projection at ffn = 14336), so the bar sits between the two.
WORKLOAD_FRO_TOL = 8e-3
@pytest.mark.parametrize("flags,want", [(0, 3), (B.FLAG_FORCE_TILED, 5)])
def test_workload_mlp_small(flags, want):
    """d=2048 ffn=8192 r=256 M=128: the weight-streaming path by default (four row tiles), the tiled one on request."""
    gi = synth.make_workload("mlp_small")
    Y, ref, path = run_gated(gi, flags=flags)
    assert path == want
    assert relmax(Y, ref) <= BF16_TOL, relmax(Y, ref)
    assert relfro(Y, ref) <= WORKLOAD_FRO_TOL, relfro(Y, ref)


@pytest.mark.parametrize("M", [64, 128])
def test_workload_decode_shape_larger_batches(M):
    """d=4096 ffn=14336 r=512 at batch sizes that take two and four row tiles of the streaming path."""
    gi = synth.make_workload("decode", M=M)
    Y, ref, path = run_gated(gi)
    assert path == 3
    assert relmax(Y, ref) <= BF16_TOL, relmax(Y, ref)
    assert relfro(Y, ref) <= WORKLOAD_FRO_TOL, relfro(Y, ref)


@pytest.mark.parametrize("one_kernel", [False, True])
@pytest.mark.parametrize("M", [1, 4, 16])
def test_workload_decode(M, one_kernel):
    """d=4096 ffn=14336 r=512, M in {1,4,16}."""
    gi = synth.make_workload("decode", M=M)
    Y, ref, path = run_gated(gi, flags=B.FLAG_STREAM_ONE_KERNEL if one_kernel else 0)
    assert path == (4 if one_kernel else 3)
    assert relmax(Y, ref) <= BF16_TOL, relmax(Y, ref)
    assert relfro(Y, ref) <= WORKLOAD_FRO_TOL, relfro(Y, ref)


SAMPLE_ROWS = [0, 1, 31, 32, 127, 128, 1000, 2047]


def assert_every_row_tile(Y, ref, rows_per_tile=256):
    """The stated bars over the whole output, and the Frobenius bar again for every row tile on its own (a tile that
    the launch mapping skipped or computed from another tile's operands cannot hide in the average)."""
    assert relmax(Y, ref) <= BF16_TOL, relmax(Y, ref)
    assert relfro(Y, ref) <= WORKLOAD_FRO_TOL, relfro(Y, ref)
    for m0 in range(0, Y.shape[0], rows_per_tile):
        e = relfro(Y[m0:m0 + rows_per_tile], ref[m0:m0 + rows_per_tile])
        assert e <= WORKLOAD_FRO_TOL, (m0, e)


@pytest.mark.parametrize("r", [256, 512, 1024])
def test_workload_prefill_all_rows(r):
    """d=4096 ffn=14336 M=4096 in the launch configuration of the benchmark: all 4096 rows (sixteen 256-row tiles, the
    XCD grid of the gate/up kernel and its mixed round of full and half tiles) against the oracle."""
    gi = synth.make_workload("prefill", r=r)
    Y, ref, path = run_gated(gi)
    assert path == 5
    assert Y.shape == (4096, 4096)
    assert_every_row_tile(Y, ref)


@pytest.mark.parametrize("M", [200, 1100, 3000, 5000])
def test_workload_prefill_extents_other_row_counts_all_rows(M):
    """d=4096 ffn=14336 r=512 at row counts off the benchmark's: few rows (leftover rounds as half tiles, many
    contraction ranges), ragged last tiles, row counts that are no multiple of the chip's tile rounds.  All rows."""
    gi = synth.make_workload("prefill", M=M, r=512)
    Y, ref, path = run_gated(gi)
    assert path == 5
    assert_every_row_tile(Y, ref)


def test_workload_prefill_extents_16384_rows_one_row_of_every_tile():
    """d=4096 ffn=14336 r=512, M = 16384 (first stage on 256 x 256 tiles): the oracle evaluates the tile borders and a
    row of every 128-row tile, at a position that moves through the tile."""
    M = 16384
    gi = synth.make_workload("prefill", M=M, r=512)
    rows = sorted({r for r in (0, 1, 31, 32, 127, 128, 255, 256, 1023, 1024, 4095, 4096, 8191, 8192, 12345,
                               M - 257, M - 129, M - 33, M - 2, M - 1)} | {128 * t + (37 * t) % 128 for t in range(M // 128)})
    Y, ref, path = run_gated(gi, rows=rows)
    assert path == 5
    assert relmax(Y, ref) <= BF16_TOL, relmax(Y, ref)
    assert relfro(Y, ref) <= WORKLOAD_FRO_TOL, relfro(Y, ref)


def test_gate_up_xcd_grid_and_mixed_round_all_rows():
    """Eight row tiles x 40 column tiles of the gate/up kernel = 320 tiles on 256 CUs: one round of full tiles and 64
    leftover tiles run as 128 halves, on an XCD grid (the planner's description says so); all rows against the oracle."""
    import re
    M, d, ffn, r = 2048, 256, 10240, 256
    gi = synth.make_gated(M, d, ffn, r, r, stream=77)
    dv = dev()
    f = {k: v.to(dv) for k, v in gi.factors().items()}
    mlp = B.SvdMlp(max_M=M, flags=B.FLAG_FORCE_TILED, **f)
    text = B.svdmlp_describe(mlp.desc, M)
    m = re.search(r"k_gate_up\[tile=256x256 tiles=(\d+) workgroups=(\d+) full=(\d+) halves=(\d+) xcd_grid=(\d+)x(\d+)\]", text)
    assert m, text
    tiles, wgs, full, halves, g0, g1 = map(int, m.groups())
    assert (tiles, wgs, full, halves) == (320, 256, 256, 128) and g0 * g1 == 8, text
    Y = mlp(gi.X.to(dv))
    torch.cuda.synchronize()
    assert mlp.last_path == 5
    Yh = Y.cpu().to(torch.float64).numpy()
    mlp.close()
    ref = oracle.gated(synth.to_f64(gi.X), **{k: synth.to_f64(v) for k, v in gi.factors().items()})
    assert_every_row_tile(Yh, ref)


@pytest.mark.parametrize("M,d,ffn,r,rd", [
    (2300, 512, 1792, 256, 256),    # nine row tiles: bands of five and four; seven column tiles: k_gate_up in bands too
    (4300, 384, 1280, 192, 384),    # seventeen (thirty-four of 128 rows): six, six, five; 128-wide last product
    (700, 1024, 2816, 320, 256),    # one band; the first product cut into ranges
])
def test_banded_tile_order_covers_every_tile(M, d, ffn, r, rd):
    gi = synth.make_gated(M, d, ffn, r, rd, stream=29)
    Y, ref, path = run_gated(gi)
    assert path == 5
    assert relmax(Y, ref) <= BF16_TOL
    assert_every_row_tile(Y, ref)


def test_banded_tile_order_with_leftover_halves():
    """Nine row tiles x 31 column tiles, which divide into no XCD grid: one round of 256 whole tiles in bands, then 23 more
    as 46 halves in the same launch; the last row tile has 52 rows."""
    M, d, ffn, r, rd = 2100, 256, 31 * 256, 192, 256
    gi = synth.make_gated(M, d, ffn, r, rd, stream=33)
    dv = dev()
    mlp = B.SvdMlp(max_M=M, **{k: v.to(dv) for k, v in gi.factors().items()})
    assert "k_gate_up[tile=256x256 tiles=279 workgroups=256 full=256 halves=46 xcd_grid=0x0]" in B.svdmlp_describe(mlp.desc, M)
    mlp.close()
    Y, ref, path = run_gated(gi)
    assert path == 5
    assert relmax(Y, ref) <= BF16_TOL
    assert_every_row_tile(Y, ref)


@pytest.mark.parametrize("M", [129, 256, 257, 384, 385, 512])   # one to four 128-row halves, the last full or nearly empty
@pytest.mark.parametrize("d,ffn,r,rd", [(512, 1792, 192, 512), (640, 2304, 64, 200)])
def test_staged_path_on_128_row_halves(M, d, ffn, r, rd):
    gi = synth.make_gated(M, d, ffn, r, rd, stream=31)
    Y, ref, path = run_gated(gi, flags=B.FLAG_FORCE_TILED)
    assert path == 5
    assert_every_row_tile(Y, ref, rows_per_tile=128)


def test_prefill_extents_row_count_whose_activation_passes_4_gib():
    """Maximum-size edge: 150093 rows at d=4096 ffn=14336 r=512.  The gated activation in the workspace is 4.3 GB and X
    and Y are 1.2 GB each, so every byte offset that is formed from a row index must be a 64-bit one (and the first stage
    must leave the kernel whose row offsets are 32-bit).  Rows of X are drawn from 8192 seeded rows through a fixed
    scrambling of the row index, so a row fetched from a wrong place does not match; the oracle evaluates rows on both
    sides of the 2^31 and 2^32 byte marks of the activation, and the ragged last rows."""
    M = 150093
    gi = synth.make_workload("prefill", M=8192, r=512)
    d = dev()
    src = torch.arange(M, dtype=torch.int64)
    src = (src * 7919 + src // 8192 * 131) % 8192
    Xs = gi.X.to(d)
    X = Xs[src.to(d)].contiguous()
    f = {k: v.to(d) for k, v in gi.factors().items()}
    mlp = B.SvdMlp(max_M=M, **f)
    Y = mlp(X)
    torch.cuda.synchronize()
    assert mlp.last_path == 5
    per_row = 14336 * 2
    rows = sorted({0, 1, 255, 256, 8191, 8192, 65535, 65536, (1 << 31) // per_row - 1, (1 << 31) // per_row, (1 << 31) // per_row + 300,
                   (1 << 32) // per_row - 1, (1 << 32) // per_row, (1 << 32) // per_row + 1, 150015, 150016, M - 2, M - 1})
    Yh = Y[torch.tensor(rows, device=d)].cpu().to(torch.float64).numpy()
    mlp.close()
    del Y, X
    a = {k: synth.to_f64(v) for k, v in gi.factors().items()}
    ref = oracle.gated(synth.to_f64(gi.X)[src[rows].numpy()], **a)
    assert relmax(Yh, ref) <= BF16_TOL, relmax(Yh, ref)
    assert relfro(Yh, ref) <= WORKLOAD_FRO_TOL, relfro(Yh, ref)


def test_linear_layer_with_an_x_beyond_4_gib_takes_the_first_stage_with_64_bit_row_offsets():
    """Maximum-size edge of the single factored layer: 270001 rows of d = 8192 (X is 4.4 GB).  The eight-wave first stage
    forms its row offsets in 32 bits, so the planner must hand this to the other first-stage kernel; the oracle evaluates
    rows on both sides of the 2^32 byte mark of X and the ragged last rows."""
    M, d_, n, r = 270001, 8192, 1024, 512
    li = synth.make_linear_gaussian(4096, d_, n, r, stream=47)
    dv = dev()
    src = torch.arange(M, dtype=torch.int64)
    src = (src * 7919 + src // 4096 * 131) % 4096
    X = li.X.to(dv)[src.to(dv)].contiguous()
    mlp = B.SvdMlp(max_M=M, Ug=li.U.to(dv), Vg=li.V.to(dv), kind=B.SVDMLP_LINEAR)
    names = kernel_names(mlp, X)
    assert names[0] == "k_s1", names
    O = mlp(X)
    torch.cuda.synchronize()
    assert mlp.last_path == 6
    per_row = d_ * 2
    rows = sorted({0, 1, 255, 256, 4095, 4096, (1 << 31) // per_row - 1, (1 << 31) // per_row, (1 << 32) // per_row - 1,
                   (1 << 32) // per_row, (1 << 32) // per_row + 129, 269999, M - 1})
    Oh = O[torch.tensor(rows, device=dv)].cpu().to(torch.float64).numpy()
    mlp.close()
    del O, X
    ref = oracle.linear(synth.to_f64(li.X)[src[rows].numpy()], synth.to_f64(li.U), synth.to_f64(li.V))
    assert relmax(Oh, ref) <= BF16_TOL, relmax(Oh, ref)


def test_workload_prefill_fused_variant_all_rows():
    """The same workload with the gated activation kept in registers (one fused kernel, path 2), all rows."""
    gi = synth.make_workload("prefill", r=512)
    Y, ref, path = run_gated(gi, flags=B.FLAG_TILED_FUSED)
    assert path == 2
    assert_every_row_tile(Y, ref, rows_per_tile=128)


def test_workload_wide_all_rows():
    """d=5120 ffn=27648 r=1024 M=2048, power-law U columns, 1 % of X entries x20: all 2048 rows against the oracle."""
    gi = synth.make_workload("wide")
    Y, ref, path = run_gated(gi)
    assert path == 5
    assert Y.shape == (2048, 5120)
    assert_every_row_tile(Y, ref)


# ---------------------------------------------------------------------------------- edge cases
def test_empty_and_invalid_calls():
    gi = synth.make_gated(8, 128, 128, 128, 128, stream=41)
    d = dev()
    f = {k: v.to(d) for k, v in gi.factors().items()}
    mlp = B.SvdMlp(max_M=8, **f)
    X = gi.X.to(d)
    Y = torch.full((8, 128), 7.0, dtype=torch.bfloat16, device=d)
    B.svdmlp_forward(mlp.ctx, X.data_ptr(), 0, Y.data_ptr())          # M = 0: nothing happens
    torch.cuda.synchronize()
    assert torch.all(Y == 7.0)
    with pytest.raises(B.SvdMlpError) as ei:
        B.svdmlp_forward(mlp.ctx, X.data_ptr(), 9, Y.data_ptr())      # M > max_M
    assert ei.value.status == B.SVDMLP_INVALID_ARGUMENT
    with pytest.raises(B.SvdMlpError):
        B.svdmlp_forward(mlp.ctx, X.data_ptr(), 8, X.data_ptr())      # aliasing
    with pytest.raises(B.SvdMlpError):
        B.svdmlp_forward(mlp.ctx, X.data_ptr() + 2, 4, Y.data_ptr())  # misaligned
    # only the first M rows of Y are written
    B.svdmlp_forward(mlp.ctx, X.data_ptr(), 3, Y.data_ptr())
    torch.cuda.synchronize()
    assert torch.all(Y[3:] == 7.0) and not torch.all(Y[:3] == 7.0)
    mlp.close()


def test_one_context_many_M_staged_path_row_boundaries():
    """One context, forwards at every size around the path switch (128 / 129), around the row-tile counts of the
    streaming path and around the 256-row tile edges, largest first so that the smaller calls run over stale rows of the workspace; rows beyond M of the
    output must stay untouched and each call must be bitwise repeatable."""
    d_, ffn, r, rd, maxM = 512, 768, 128, 256, 520
    gi = synth.make_gated(maxM, d_, ffn, r, rd, stream=45)
    dv = dev()
    f = {k: v.to(dv) for k, v in gi.factors().items()}
    mlp = B.SvdMlp(max_M=maxM, **f)
    Xd = gi.X.to(dv)
    a = {k: synth.to_f64(v) for k, v in gi.factors().items()}
    ref = oracle.gated(synth.to_f64(gi.X), **a)
    scale = np.max(np.abs(ref))
    for M in (520, 513, 512, 511, 257, 256, 255, 130, 129, 128, 127, 65, 64, 33, 32, 31, 1):
        Y = torch.full((maxM, d_), 7.0, dtype=torch.bfloat16, device=dv)
        B.svdmlp_forward(mlp.ctx, Xd.data_ptr(), M, Y.data_ptr())
        torch.cuda.synchronize()
        assert mlp.last_path == (5 if M > 128 else 3), (M, mlp.last_path)
        assert torch.all(Y[M:] == 7.0), M
        Yh = Y[:M].cpu().to(torch.float64).numpy()
        assert np.max(np.abs(Yh - ref[:M])) / scale <= BF16_TOL, M
        Y2 = torch.empty_like(Y)
        B.svdmlp_forward(mlp.ctx, Xd.data_ptr(), M, Y2.data_ptr())
        torch.cuda.synchronize()
        assert torch.equal(Y[:M], Y2[:M]), M
    mlp.close()


def test_zero_input_gives_zero_output():
    gi = synth.make_gated(64, 128, 256, 128, 128, stream=42)
    d = dev()
    f = {k: v.to(d) for k, v in gi.factors().items()}
    for flags, M in ((B.FLAG_FORCE_TILED, 64), (0, 16)):
        mlp = B.SvdMlp(max_M=64, flags=flags, **f)
        Y = mlp(torch.zeros((M, 128), dtype=torch.bfloat16, device=d))
        torch.cuda.synchronize()
        assert torch.all(Y == 0)
        mlp.close()


@pytest.mark.parametrize("M,d,ffn,r,rd,flags", [
    (300, 512, 1024, 192, 256, 0), (300, 384, 512, 128, 256, 0), (200, 256, 384, 128, 128, 0),
    (300, 512, 1024, 192, 256, B.FLAG_TILED_FUSED), (100, 512, 1408, 192, 256, 0), (1000, 16384, 1024, 1024, 256, 0),
])
def test_describe_matches_the_kernels_that_run(M, d, ffn, r, rd, flags):
    """The host-only plan description names exactly the kernels a forward launches, in order."""
    import re
    gi = synth.make_gated(M, d, ffn, r, rd, stream=48)
    dv = dev()
    f = {k: v.to(dv) for k, v in gi.factors().items()}
    mlp = B.SvdMlp(max_M=M, flags=flags, **f)
    text = B.svdmlp_describe(mlp.desc, M)
    ran = kernel_names(mlp, gi.X.to(dv))
    assert int(re.match(r"path=(\d)", text).group(1)) == mlp.last_path
    mlp.close()
    said = re.findall(r" (k_[a-z0-9_]+)", text)
    # the reduction that follows a first stage cut into ranges is timed together with it
    if len(said) > 1 and said[1] == "k_reduce" and said[0] in ("k_in", "k_s1"):
        said.pop(1)
    assert said == ran, (text, ran)


def _random_shapes(n, seed):
    """Seeded draw from the lattice of supported bf16 extents (d, ffn multiples of 128; r a multiple of 64, >= 128;
    r_down in {128, 256, 512}), M anywhere from one row to a few row tiles."""
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        d = 128 * int(rng.integers(1, 9))
        ffn = 128 * int(rng.integers(1, 13))
        lim = min(d, ffn)
        if lim < 128:
            continue
        r = 64 * int(rng.integers(2, lim // 64 + 1))
        rd_choices = [x for x in (128, 256, 512) if x <= lim]
        rd = int(rng.choice(rd_choices))
        M = int(rng.choice([int(rng.integers(1, 33)), int(rng.integers(33, 129)), int(rng.integers(129, 700))]))
        out.append((M, d, ffn, r, rd))
    return out


@pytest.mark.parametrize("M,d,ffn,r,rd", _random_shapes(24, 20251025))
def test_bf16_random_supported_extents(M, d, ffn, r, rd):
    """Whatever path the planner picks for a supported extent, the result matches the oracle; the plan description
    agrees with the path taken."""
    gi = synth.make_gated(M, d, ffn, r, rd, stream=60)
    dv = dev()
    f = {k: v.to(dv) for k, v in gi.factors().items()}
    mlp = B.SvdMlp(max_M=M, **f)
    Y = mlp(gi.X.to(dv))
    torch.cuda.synchronize()
    path = mlp.last_path
    assert B.svdmlp_describe(mlp.desc, M).startswith(f"path={path} ")
    mlp.close()
    ref = oracle.gated(synth.to_f64(gi.X), **{k: synth.to_f64(v) for k, v in gi.factors().items()})
    Yh = Y.cpu().to(torch.float64).numpy()
    assert relmax(Yh, ref) <= BF16_TOL, (path, relmax(Yh, ref))


@pytest.mark.parametrize("M,d,ffn,r,rd", _random_shapes(12, 977))
@pytest.mark.parametrize("flags", [B.FLAG_FORCE_TILED, B.FLAG_FORCE_TILED | B.FLAG_TILED_FUSED])
def test_bf16_random_extents_forced_tiled_variants(M, d, ffn, r, rd, flags):
    """The same lattice with the tiled path forced (also for tiny M) in both of its variants."""
    gi = synth.make_gated(M, d, ffn, r, rd, stream=61)
    Y, ref, path = run_gated(gi, flags=flags)
    assert path in (2, 5) and (path == 2 or not flags & B.FLAG_TILED_FUSED)
    assert relmax(Y, ref) <= BF16_TOL, (path, relmax(Y, ref))


def _random_linear_shapes(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        d, nn = 128 * int(rng.integers(1, 17)), 128 * int(rng.integers(1, 13))
        r = 128 * int(rng.integers(1, min(d, nn) // 128 + 1))
        out.append((int(rng.integers(1, 600)), d, nn, r))
    return out


@pytest.mark.parametrize("M,d,n,r", _random_linear_shapes(10, 31337))
def test_bf16_linear_random_supported_extents(M, d, n, r):
    li = synth.make_linear_gaussian(M, d, n, r, stream=62)
    dv = dev()
    mlp = B.SvdMlp(max_M=M, Ug=li.U.to(dv), Vg=li.V.to(dv), kind=B.SVDMLP_LINEAR)
    O = mlp(li.X.to(dv))
    torch.cuda.synchronize()
    assert mlp.last_path == (7 if M <= 128 else 6)
    Oh = O.cpu().to(torch.float64).numpy()
    mlp.close()
    ref = oracle.linear(synth.to_f64(li.X), synth.to_f64(li.U), synth.to_f64(li.V))
    assert relmax(Oh, ref) <= BF16_TOL, relmax(Oh, ref)


@pytest.mark.parametrize("M,flags", [(8, 0), (100, 0), (300, 0), (8, B.FLAG_STREAM_ONE_KERNEL), (20, B.FLAG_STREAM_ONE_KERNEL)])
def test_forward_can_be_captured_in_a_graph_and_replayed(M, flags):
    """svdmlp_forward only enqueues kernels (no memset, no allocation, no synchronisation), so a caller may capture
    it; every replay, interleaved with eager work and synchronisations, must reproduce the eager result bit for bit."""
    gi = synth.make_gated(M, 512, 1024, 192, 256, stream=63)
    dv = dev()
    f = {k: v.to(dv) for k, v in gi.factors().items()}
    mlp = B.SvdMlp(max_M=M, flags=flags, **f)
    X = gi.X.to(dv)
    Y = torch.empty_like(X)
    eager = mlp(X).clone()
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        mlp(X, Y)
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mlp(X, Y)
    for rep in range(4):
        Y.fill_(3.0)
        X2 = (X * 0.5).contiguous()          # eager work between replays
        other = mlp(X2)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, eager), rep
        assert not torch.equal(other, eager)
    del g
    mlp.close()


@pytest.mark.parametrize("M,d,ffn,r,rd", [(300, 1024, 1024, 256, 768), (530, 1536, 1536, 384, 1280), (20, 1024, 1024, 256, 768),
                                          (100, 1024, 1024, 256, 768)])
def test_bf16_down_rank_of_three_or_five_256_tiles(M, d, ffn, r, rd):
    """Down ranks that only the staged variant takes (a multiple of 256 that is neither 256, 512 nor a multiple of 512),
    on the tiled and on the streaming path."""
    gi = synth.make_gated(M, d, ffn, r, rd, stream=64)
    Y, ref, path = run_gated(gi)
    assert path == (5 if M > 128 else 3)
    assert relmax(Y, ref) <= BF16_TOL, (path, relmax(Y, ref))


@pytest.mark.parametrize("M,d,ffn,r,rd", [
    (300, 512, 1024, 200, 300), (40, 512, 640, 17, 33), (700, 1024, 1024, 129, 513), (129, 384, 1152, 100, 384),
    (16, 512, 1408, 250, 100), (100, 256, 512, 1, 1), (520, 640, 768, 320, 640),
    (300, 512, 1000, 200, 300), (50, 256, 200, 100, 64), (200, 384, 1153, 130, 257),   # ffn is free as well
])
@pytest.mark.parametrize("flags", [0, B.FLAG_FORCE_TILED | B.FLAG_TILED_FUSED])
def test_bf16_arbitrary_ranks(M, d, ffn, r, rd, flags):
    """Ranks (and ffn) that are not multiples of anything: the library rounds them up to its tiles with zero columns /
    rows in its re-tiled copies of the factors, which must not change the result."""
    gi = synth.make_gated(M, d, ffn, r, rd, stream=65)
    Y, ref, path = run_gated(gi, flags=flags)
    assert relmax(Y, ref) <= BF16_TOL, (path, relmax(Y, ref))


@pytest.mark.parametrize("M,d,n,r", [(300, 512, 640, 100), (70, 256, 512, 7), (513, 1024, 768, 300)])
def test_bf16_linear_arbitrary_rank(M, d, n, r):
    li = synth.make_linear_gaussian(M, d, n, r, stream=66)
    dv = dev()
    mlp = B.SvdMlp(max_M=M, Ug=li.U.to(dv), Vg=li.V.to(dv), kind=B.SVDMLP_LINEAR)
    O = mlp(li.X.to(dv))
    torch.cuda.synchronize()
    Oh = O.cpu().to(torch.float64).numpy()
    mlp.close()
    ref = oracle.linear(synth.to_f64(li.X), synth.to_f64(li.U), synth.to_f64(li.V))
    assert relmax(Oh, ref) <= BF16_TOL, relmax(Oh, ref)


@pytest.mark.parametrize("M,ranges", [(200, 1), (200, 4), (200, 7), (200, 9), (200, 16), (200, 17), (200, 32),   # 4, 8, 16 loads at once
                                      (2400, 3), (2400, 13), (4000, 2), (4000, 9)])                       # many waves: 4, then one
def test_bf16_sums_of_any_number_of_ranges(M, ranges):
    """The sum over contraction ranges loads several of them at a time: every count on either side of a batch."""
    gi = synth.make_gated(M, 256, 4096, 100, 256, stream=84)
    mlp = B.SvdMlp(max_M=M, flags=B.FLAG_PLAN_ROOM | B.FLAG_FORCE_TILED, **{k: v.to(dev()) for k, v in gi.factors().items()})
    B.svdmlp_force_plan(mlp.ctx, 0, 0, ranges, 0)
    Y = mlp(gi.X.to(dev()))
    rows = np.arange(0, M, 7)
    ref = oracle.gated(synth.to_f64(gi.X)[rows], **{k: synth.to_f64(v) for k, v in gi.factors().items()})
    y = Y.cpu().to(torch.float64).numpy()[rows]
    mlp.close()
    assert relmax(y, ref) <= BF16_TOL
    assert relfro(y, ref) <= 8e-3      # five roundings to bf16; one of 32 ranges left out or taken twice: 0.18


@pytest.mark.parametrize("M,ffn,rd,ranges", [(129, 8448, 256, 33), (384, 8448, 256, 33), (256, 12288, 512, 48), (150, 12032, 512, 47)])
def test_bf16_more_than_32_ranges_of_few_rows(M, ffn, rd, ranges):
    """Few rows cut the down projection into up to 48 ranges of at least eight 32-wide steps."""
    gi = synth.make_gated(M, 512, ffn, 100, rd, stream=87)
    f = gi.factors()
    mlp = B.SvdMlp(max_M=M, flags=B.FLAG_FORCE_TILED, **{k: v.to(dev()) for k, v in f.items()})
    assert f"ranges={ranges} " in B.svdmlp_describe(mlp.desc, M).split("k_down1")[1].split("k_reduce")[0]
    Y = mlp(gi.X.to(dev()))
    rows = np.unique(np.r_[np.arange(0, M, 7), M - 1])
    ref = oracle.gated(synth.to_f64(gi.X)[rows], **{k: synth.to_f64(v) for k, v in f.items()})
    y = Y.cpu().to(torch.float64).numpy()[rows]
    mlp.close()
    assert relmax(y, ref) <= BF16_TOL
    assert relfro(y, ref) <= 8e-3      # five roundings to bf16; one of 48 ranges left out or taken twice: 0.14


def test_one_kernel_decode_successive_forwards_with_different_inputs():
    """The one-launch streaming variant hands activations from workgroup to workgroup inside the kernel; a second
    forward with other inputs on the same context must not see anything of the first (activation buffers, counters,
    tickets), for one and for two 16-row tiles, and must agree bit for bit with a fresh context."""
    d_, ffn, r, rd = 512, 1408, 192, 256
    gi = synth.make_gated(32, d_, ffn, r, rd, stream=67)
    gj = synth.make_gated(32, d_, ffn, r, rd, stream=68)
    dv = dev()
    f = {k: v.to(dv) for k, v in gi.factors().items()}
    a = {k: synth.to_f64(v) for k, v in gi.factors().items()}
    mlp = B.SvdMlp(max_M=32, flags=B.FLAG_STREAM_ONE_KERNEL, **f)
    outs = []
    for X in (gi.X, gj.X, gi.X[:9], gj.X[:16], gi.X[:17], gj.X):
        Y = mlp(X.to(dv).contiguous())
        torch.cuda.synchronize()
        assert mlp.last_path == 4
        ref = oracle.gated(synth.to_f64(X), **a)
        assert relmax(Y.cpu().to(torch.float64).numpy(), ref) <= BF16_TOL, X.shape
        outs.append(Y.clone())
    mlp.close()
    fresh = B.SvdMlp(max_M=32, flags=B.FLAG_STREAM_ONE_KERNEL, **f)
    Y = fresh(gj.X.to(dv))
    torch.cuda.synchronize()
    fresh.close()
    assert torch.equal(Y, outs[1]) and torch.equal(Y, outs[5])


def test_one_kernel_decode_reports_a_wait_that_ran_out():
    """Error path of the one-kernel variant, forced from the host: with a poll limit of zero every wait that is not
    already satisfied gives up at once.  The kernel still ends normally; the forward's output is NaN (never silently
    partial), svdmlp_check reports the time-out once and clears it, and the next forward with the normal bound is right."""
    gi = synth.make_gated(8, 512, 1408, 192, 256, stream=58)
    d = dev()
    f = {k: v.to(d) for k, v in gi.factors().items()}
    mlp = B.SvdMlp(max_M=8, flags=B.FLAG_STREAM_ONE_KERNEL, **f)
    X = gi.X.to(d)
    good = mlp(X).clone()
    torch.cuda.synchronize()
    assert mlp.last_path == 4
    B.svdmlp_check(mlp.ctx)                                   # nothing to report
    L = B.lib()
    assert L.svdmlp_debug_set_poll_limit(mlp.ctx, 0) == 0
    bad = mlp(X).clone()
    torch.cuda.synchronize()
    assert L.svdmlp_check(mlp.ctx) == B.SVDMLP_TIMED_OUT
    assert L.svdmlp_check(mlp.ctx) == B.SVDMLP_OK             # reported once, then cleared
    assert bool(torch.isnan(bad.float()).all()), "a forward whose wait ran out must not look like a result"
    assert L.svdmlp_debug_set_poll_limit(mlp.ctx, -1) == 0
    again = mlp(X)
    torch.cuda.synchronize()
    B.svdmlp_check(mlp.ctx)
    assert torch.equal(again, good)
    mlp.close()


def test_contexts_on_two_streams_run_concurrently_without_interference():
    """Two contexts (a streaming-path one and a tiled-path one), each with its own workspace, enqueue forwards on two
    streams at the same time; every output equals, bit for bit, what the same context gives when it runs alone."""
    dv = dev()
    ga = synth.make_gated(24, 512, 1408, 192, 256, stream=71)
    gb = synth.make_gated(700, 512, 1024, 192, 256, stream=72)
    A = B.SvdMlp(max_M=24, **{k: v.to(dv) for k, v in ga.factors().items()})
    Bc = B.SvdMlp(max_M=700, **{k: v.to(dv) for k, v in gb.factors().items()})
    Xa, Xb = ga.X.to(dv), gb.X.to(dv)
    Ya0, Yb0 = A(Xa).clone(), Bc(Xb).clone()
    torch.cuda.synchronize()
    assert A.last_path == 3 and Bc.last_path == 5
    sa, sb = torch.cuda.Stream(device=dv), torch.cuda.Stream(device=dv)
    Ya = [torch.empty_like(Ya0) for _ in range(8)]
    Yb = [torch.empty_like(Yb0) for _ in range(8)]
    torch.cuda.synchronize()
    for i in range(8):
        A.forward(Xa, Ya[i], stream=sa)
        Bc.forward(Xb, Yb[i], stream=sb)
    sa.synchronize()
    sb.synchronize()
    for i in range(8):
        assert torch.equal(Ya[i], Ya0) and torch.equal(Yb[i], Yb0), i
    A.close()
    Bc.close()


def test_small_ranks_take_the_fused_variant_by_themselves():
    """r and r_down within one 128-wide tile: the planner picks the variant that keeps the gated activation in registers
    (path 2) without the flag, and the streaming path runs the down rank unpadded; same parity bar."""
    gi = synth.make_gated(700, 512, 1024, 100, 128, stream=73)
    Y, ref, path = run_gated(gi)
    assert path == 2
    assert relmax(Y, ref) <= BF16_TOL, relmax(Y, ref)
    assert relfro(Y, ref) <= 1.5e-2
    Ys, refs, paths = run_gated(synth.make_gated(20, 512, 1024, 100, 128, stream=73))
    assert paths == 3
    assert relmax(Ys, refs) <= BF16_TOL, relmax(Ys, refs)


@pytest.mark.parametrize("scale", [2.0 ** -10, 64.0])
@pytest.mark.parametrize("M", [20, 300])
def test_gate_in_its_linear_and_in_its_saturated_regime(M, scale):
    """Inputs scaled by a power of two (exact in bf16): tiny gate pre-activations, where SiLU(g) ~ g / 2 and the output
    is quadratic in the scale, and large ones, where SiLU(g) is g or 0 to rounding and exp2 of the negated gate
    overflows or underflows inside the kernels.  Streaming and tiled path, same parity bar."""
    gi = synth.make_gated(M, 512, 1408, 192, 256, stream=74)
    gi.X = (gi.X.to(torch.float32) * scale).to(torch.bfloat16)
    Y, ref, path = run_gated(gi)
    assert path == (3 if M <= 128 else 5)
    assert np.isfinite(Y).all()
    assert relmax(Y, ref) <= BF16_TOL, relmax(Y, ref)
    assert relfro(Y, ref) <= 1.5e-2


@pytest.mark.parametrize("M", [1, 16, 32, 33, 64, 100, 128])
@pytest.mark.parametrize("d,n,r", [(256, 512, 128), (512, 1408 - 128, 200), (1024, 4096, 512)])
def test_bf16_linear_streaming_small_batches(M, d, n, r):
    """O = (X U) V for up to 128 rows on the weight-streaming kernels (path 7) against the oracle's plain chain, and
    against the MFMA-tiled path of the same context family (forced), which rounds at the same two places."""
    li = synth.make_linear_gaussian(M, d, n, r, stream=81)
    dv = dev()
    U, V, X = li.U.to(dv), li.V.to(dv), li.X.to(dv)
    mlp = B.SvdMlp(max_M=128, Ug=U, Vg=V, kind=B.SVDMLP_LINEAR)
    O = mlp(X)
    O2 = mlp(X)
    torch.cuda.synchronize()
    assert mlp.last_path == 7 and tuple(O.shape) == (M, n)
    assert torch.equal(O, O2)                                  # fixed-order sums: bit-reproducible
    mlp.close()
    ref = oracle.linear(synth.to_f64(li.X), synth.to_f64(li.U), synth.to_f64(li.V))
    Oh = O.cpu().to(torch.float64).numpy()
    assert relmax(Oh, ref) <= BF16_TOL, (relmax(Oh, ref), relfro(Oh, ref))
    assert relfro(Oh, ref) <= 1.5e-2
    tiled = B.SvdMlp(max_M=128, Ug=U, Vg=V, kind=B.SVDMLP_LINEAR, flags=B.FLAG_FORCE_TILED)
    Ot = tiled(X)
    torch.cuda.synchronize()
    assert tiled.last_path == 6
    tiled.close()
    assert relmax(Ot.cpu().to(torch.float64).numpy(), ref) <= BF16_TOL


@pytest.mark.parametrize("M", [5, 20, 40, 100])
@pytest.mark.parametrize("d,n,r", [
    # blocks per wave of the last product, up to 32 rows (32 wide) / from 33 rows on (16 wide)
    (256, 8192, 128), (512, 8320, 256), (1024, 8192, 384), (2048, 8192, 640),   # 32-column tiles: 1, 1, 2, 3 / 1, 2, 3, 5
    (256, 16512, 128), (1024, 17408, 896),                                      # more than 512 of them: 1, 4 / 1, 7
    (1536, 4736, 256), (2688, 6400, 768), (4096, 1024, 1024),                   # 16-column / 32-column tiles: 1, 3, 4 / 2, 6, 8
])
def test_bf16_linear_streaming_short_contraction_ranges(M, d, n, r):
    li = synth.make_linear_gaussian(M, d, n, r, stream=72)
    dv = dev()
    mlp = B.SvdMlp(max_M=M, Ug=li.U.to(dv), Vg=li.V.to(dv), kind=B.SVDMLP_LINEAR)
    O = mlp(li.X.to(dv)).cpu().to(torch.float64).numpy()
    assert mlp.last_path == 7
    mlp.close()
    ref = oracle.linear(synth.to_f64(li.X), synth.to_f64(li.U), synth.to_f64(li.V))
    assert relmax(O, ref) <= BF16_TOL
    assert relfro(O, ref) <= 4e-3      # two roundings to bf16 (2.4e-3); one block left out of the longest contraction: 6e-2


@pytest.mark.parametrize("M", [3, 16, 32])
@pytest.mark.parametrize("d,n,r,blocks", [
    (1024, 8320, 768, [3] * 8), (1024, 8320, 640, [3] * 6 + [2, 0]), (1280, 10112, 1152, [5] * 7 + [1]),   # 257 .. 512 tiles
    (1024, 17408, 640, [3] * 6 + [2, 0]), (1024, 16512, 896, [4] * 7 + [0]), (1536, 16512, 1408, [6] * 7 + [2]),   # more (32 rows)
    (1024, 24704, 640, [3] * 6 + [2, 0]), (1024, 24704, 384, [2] * 6 + [0, 0]),   # more than 768 (any rows)
])
def test_bf16_linear_streaming_last_product_with_one_register_buffer(M, d, n, r, blocks):
    """The loop of one register buffer takes blocks in pairs and an odd one by itself: waves with every remainder."""
    kw = -(-r // 256)
    assert blocks == [max(0, min(kw, r // 32 - w * kw)) for w in range(8)]
    li = synth.make_linear_gaussian(M, d, n, r, stream=88)
    dv = dev()
    mlp = B.SvdMlp(max_M=M, Ug=li.U.to(dv), Vg=li.V.to(dv), kind=B.SVDMLP_LINEAR)
    assert B.svdmlp_describe(mlp.desc, M).endswith("buffers=2]" if 16384 < n <= 24576 and M <= 16 else "buffers=1]")
    O = mlp(li.X.to(dv)).cpu().to(torch.float64).numpy()
    assert mlp.last_path == 7
    mlp.close()
    ref = oracle.linear(synth.to_f64(li.X), synth.to_f64(li.U), synth.to_f64(li.V))
    assert relmax(O, ref) <= BF16_TOL
    assert relfro(O, ref) <= 4e-3      # two roundings to bf16 (2.4e-3); one of 44 blocks left out: 0.15


def test_bf16_linear_streaming_can_be_captured_and_matches_describe():
    """Path 7 under stream capture (replayed three times with eager work in between), and the kernels svdmlp_describe
    names are the ones that run."""
    li = synth.make_linear_gaussian(20, 512, 1024, 256, stream=82)
    dv = dev()
    mlp = B.SvdMlp(max_M=64, Ug=li.U.to(dv), Vg=li.V.to(dv), kind=B.SVDMLP_LINEAR)
    X = li.X.to(dv)
    assert kernel_names(mlp, X) == ["k_stream_d1", "k_stream_d5"]
    assert B.svdmlp_describe(mlp.desc, 20).startswith("path=7 bf16-linear-streaming: row_tiles=1 k_stream_d1[tile=16")
    eager = mlp(X).clone()
    torch.cuda.synchronize()
    O = torch.empty_like(eager)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        mlp(X, O)
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mlp(X, O)
    for i in range(3):
        O.fill_(3.0)
        other = mlp((X * 0.5).contiguous())      # eager work between the replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(O, eager), i
        assert not torch.equal(other, eager)
    del g
    mlp.close()
