"""GPU parity of the building blocks through the C ABI: MFMA linear layers with
their fused epilogues, and attention, against the oracle's plain definitions
on the same (bf16-rounded where bf16) inputs."""
import numpy as np
import pytest

import synth
from oracle import model as om

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TDT = {"f32": torch.float32, "bf16": torch.bfloat16}


def rel_l2(g, r):
    return float(np.linalg.norm(g - r) / max(np.linalg.norm(r), 1e-30))


def _inputs(name, shape, dt, scale=1.0):
    a = synth.normal(name, shape, scale)
    return synth.bf16_round(a) if dt == "bf16" else a


def _dev(a, dt):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV).to(TDT[dt])


@pytest.mark.parametrize("dt", ["bf16", "f32"])
# Beyond the small and model shapes, four bf16 shapes reach each multi-round tile
# of the wide kernel with a ragged row tail: 256 x 288 with a ragged column tile
# (4100 x 4616), 256 x 256 (4100 x 4352), 128 x 432 (4000 x 3456) and 128 x 128
# (4000 x 2304).
@pytest.mark.parametrize("M,N,K", [(300, 200, 136), (128, 128, 64), (1, 16, 8), (517, 384, 1152),
                                   (4096, 1152, 1152), (4100, 4612, 1152), (130, 260, 192), (1000, 1160, 256),
                                   (4100, 4616, 64), (4100, 4352, 128), (4000, 3456, 64), (4000, 2304, 64)])
@pytest.mark.parametrize("epi", ["bias", "gelu", "gate"])
def test_linear(bclib, dt, M, N, K, epi):
    if dt == "f32" and M * N * K > 1e8:
        pytest.skip("fp32 path is for the small model")
    A = _inputs(f"A{M}{N}{K}", (M, K), dt)
    W = _inputs(f"W{M}{N}{K}", (N, K), dt, 0.05)
    b = _inputs(f"b{M}{N}{K}", (N,), dt, 0.1)
    y = om.linear(A.astype(np.float64), W.astype(np.float64), b.astype(np.float64))
    tA, tW, tb = _dev(A, dt), _dev(W, dt), _dev(b, dt)
    if epi == "gate":
        rpg = max(1, M // 3)
        G = synth.normal(f"g{M}", ((M + rpg - 1) // rpg, N), 0.5)
        R = synth.normal(f"r{M}", (M, N), 1.0)
        exp = R.astype(np.float64) + np.repeat(G, rpg, axis=0)[:M] * y
        out = torch.from_numpy(R).to(DEV)
        bclib.linear(tA, tW, tb, out, bclib.EPI_GATE_RES, res=out, gate=torch.from_numpy(G).to(DEV),
                     rows_per_gate=rpg)
        tol = 1e-5
    else:
        exp = om.gelu_tanh(y) if epi == "gelu" else y
        out = torch.empty((M, N), dtype=TDT[dt], device=DEV)
        bclib.linear(tA, tW, tb, out, bclib.EPI_BIAS_GELU if epi == "gelu" else bclib.EPI_BIAS)
        tol = 5e-3 if dt == "bf16" else 1e-5
    torch.cuda.synchronize()
    err = rel_l2(out.float().cpu().numpy().astype(np.float64), exp)
    assert err <= tol, err


def test_linear_rejects_bad_k(bclib):
    A = torch.zeros((4, 12), dtype=torch.bfloat16, device=DEV)
    W = torch.zeros((16, 12), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(bclib.BCError) as e:
        bclib.linear(A, W, None, torch.empty((4, 16), dtype=torch.bfloat16, device=DEV))
    assert e.value.code == bclib.ERR_UNSUPPORTED


@pytest.mark.parametrize("dt,B,H,Tq,Tk,d", [
    ("bf16", 2, 3, 200, 200, 72), ("bf16", 1, 2, 100, 37, 128), ("bf16", 2, 2, 64, 64, 32),
    ("bf16", 1, 1, 130, 257, 64), ("bf16", 1, 1, 1, 1, 72), ("bf16", 16, 16, 256, 256, 72),
    ("bf16", 1, 2, 1100, 700, 72), ("bf16", 2, 1, 600, 1030, 32), ("bf16", 1, 2, 520, 333, 128),
    # enough (sample, head) pairs for several rounds of 128-query workgroups
    ("bf16", 8, 32, 300, 300, 72), ("bf16", 8, 32, 300, 270, 64), ("bf16", 4, 32, 300, 333, 128),
    # resident key tiles with 32 queries per wave (short key sequences, large grids)
    ("bf16", 8, 32, 300, 120, 72), ("bf16", 8, 32, 300, 200, 128), ("bf16", 8, 32, 260, 256, 32),
    ("f32", 2, 4, 64, 64, 32), ("f32", 1, 2, 77, 131, 64)])
def test_attention(bclib, dt, B, H, Tq, Tk, d):
    q = _inputs(f"q{Tq}{d}", (B, Tq, H, d), dt)
    k = _inputs(f"k{Tk}{d}", (B, Tk, H, d), dt)
    v = _inputs(f"v{Tk}{d}", (B, Tk, H, d), dt)
    exp = om.attention(*(a.astype(np.float64).transpose(0, 2, 1, 3) for a in (q, k, v))).transpose(0, 2, 1, 3)
    out = torch.empty((B, Tq, H, d), dtype=TDT[dt], device=DEV)
    bclib.attention(_dev(q, dt), _dev(k, dt), _dev(v, dt), out)
    torch.cuda.synchronize()
    err = rel_l2(out.float().cpu().numpy().astype(np.float64), exp)
    assert err <= (1e-2 if dt == "bf16" else 1e-5), err


# Pre-scaled queries (the form the blocks' projections write): the resident
# loop, and the streaming loop with 16 and 32 queries per wave (64: see
# ATT_VARIANTS); at d = 128 the last key tile holds 13 keys (333) or 54 (310).
@pytest.mark.parametrize("B,H,Tq,Tk,d", [
    (16, 16, 256, 256, 72), (1, 2, 100, 37, 128), (1, 2, 1100, 700, 72), (1, 2, 520, 333, 128),
    (2, 1, 600, 1030, 32), (4, 16, 300, 300, 72), (4, 32, 300, 333, 128), (4, 32, 300, 310, 128),
    (8, 32, 300, 300, 72), (8, 32, 300, 270, 64), (8, 32, 300, 120, 72), (8, 32, 300, 200, 128),
    (1, 1, 1, 1, 72)])
def test_attention_prescaled(bclib, B, H, Tq, Tk, d):
    q = _inputs(f"q{Tq}{d}", (B, Tq, H, d), "bf16")
    k = _inputs(f"k{Tk}{d}", (B, Tk, H, d), "bf16")
    v = _inputs(f"v{Tk}{d}", (B, Tk, H, d), "bf16")
    # the producer's rounding: q * log2(e) / sqrt(d) in fp32, rounded to bf16
    c = np.float32(1.4426950408889634) / np.sqrt(np.float32(d))
    qs = synth.bf16_round((q.astype(np.float32) * c).astype(np.float32))
    # softmax(q k^T / sqrt(d)) with the queries the stored values stand for
    qeff = qs.astype(np.float64) / float(c)
    exp = om.attention(*(a.astype(np.float64).transpose(0, 2, 1, 3) for a in (qeff, k, v))).transpose(0, 2, 1, 3)
    out = torch.empty((B, Tq, H, d), dtype=torch.bfloat16, device=DEV)
    bclib.attention(_dev(qs, "bf16"), _dev(k, "bf16"), _dev(v, "bf16"), out, prescaled=True)
    torch.cuda.synchronize()
    err = rel_l2(out.float().cpu().numpy().astype(np.float64), exp)
    assert err <= 1e-2, err


# Output rows that are not 8-byte aligned take the per-element stores.
@pytest.mark.parametrize("B,H,Tq,Tk,d", [(2, 3, 200, 200, 72), (1, 2, 520, 333, 128)])
def test_attention_unaligned_output(bclib, B, H, Tq, Tk, d):
    q = _inputs(f"q{Tq}{d}", (B, Tq, H, d), "bf16")
    k = _inputs(f"k{Tk}{d}", (B, Tk, H, d), "bf16")
    v = _inputs(f"v{Tk}{d}", (B, Tk, H, d), "bf16")
    exp = om.attention(*(a.astype(np.float64).transpose(0, 2, 1, 3) for a in (q, k, v))).transpose(0, 2, 1, 3)
    n = B * Tq * H * d
    buf = torch.zeros(n + 2, dtype=torch.bfloat16, device=DEV)
    out = buf[2:].view(B, Tq, H, d)     # 4 bytes past an aligned start
    assert out.data_ptr() % 8 == 4
    bclib.attention(_dev(q, "bf16"), _dev(k, "bf16"), _dev(v, "bf16"), out)
    torch.cuda.synchronize()
    err = rel_l2(out.float().cpu().numpy().astype(np.float64), exp)
    assert err <= 1e-2, err
    assert float(buf[:2].abs().sum()) == 0.0     # nothing written before the output


# Output rows at every 2-byte alignment, from the resident and the streaming loops.
@pytest.mark.parametrize("off", [1, 2, 3, 4])
@pytest.mark.parametrize("B,H,Tq,Tk,d", [(1, 2, 70, 100, 72), (1, 2, 70, 300, 128)])
def test_attention_output_alignment(bclib, B, H, Tq, Tk, d, off):
    g = torch.Generator(device=DEV)
    g.manual_seed(off)
    q, k, v = (torch.empty((B, T, H, d), device=DEV).normal_(generator=g).bfloat16() for T in (Tq, Tk, Tk))
    want = torch.empty_like(q)
    bclib.attention(q, k, v, want)
    buf = torch.full((q.numel() + 8,), 7.0, dtype=torch.bfloat16, device=DEV)
    out = buf[off:off + q.numel()].view(q.shape)
    bclib.attention(q, k, v, out)
    torch.cuda.synchronize()
    assert bool((out == want).all())
    assert bool((buf[:off] == 7.0).all()) and bool((buf[off + q.numel():] == 7.0).all())    # nothing written outside


def test_attention_prescaled_rejects_fp32(bclib):
    z = torch.zeros((1, 4, 1, 32), dtype=torch.float32, device=DEV)
    with pytest.raises(bclib.BCError) as e:
        bclib.attention(z, z, z, torch.empty_like(z), prescaled=True)
    assert e.value.code == bclib.ERR_UNSUPPORTED


def test_attention_rejects_unsupported_head_dim(bclib):
    z = torch.zeros((1, 4, 1, 40), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(bclib.BCError) as e:
        bclib.attention(z, z, z, torch.empty_like(z))
    assert e.value.code == bclib.ERR_UNSUPPORTED


# The k-split linear of small grids, against 64 bits: every tile shape it takes
# (bf16: 32 x 48, 64 x 48, 64 x 64, 64 x 80; fp32: 16 x 16, 32 x 48), fewer
# k-steps than waves (64 bf16 / 32 fp32 values a step) and numbers of them that
# leave the waves unequal shares, ragged rows and columns, columns that are not
# a multiple of 4 and an output that is not 16-byte aligned (element-wise
# epilogue), a gate that changes within a tile.
@pytest.mark.parametrize("epi", ["bias", "gelu", "gate"])
@pytest.mark.parametrize("dt,M,N,K,off", [
    ("bf16", 1, 8, 64, 0), ("bf16", 250, 1152, 4608, 0), ("bf16", 256, 3072, 576, 0), ("bf16", 250, 3456, 640, 0),
    ("bf16", 1020, 1152, 1088, 0), ("bf16", 250, 1151, 576, 0), ("bf16", 70, 300, 192, 2),
    ("f32", 1, 8, 32, 0), ("f32", 130, 200, 288, 0), ("f32", 600, 900, 160, 0), ("f32", 70, 301, 96, 0),
    ("f32", 70, 300, 96, 2)])
def test_linear_small_grids(bclib, dt, M, N, K, off, epi):
    g = torch.Generator(device=DEV)
    g.manual_seed(M * 7 + N)

    def rnd(*s, scale=1.0):
        return torch.empty(s, device=DEV).normal_(0.0, scale, generator=g)

    A, W, b = rnd(M, K).to(TDT[dt]), rnd(N, K, scale=0.05).to(TDT[dt]), rnd(N, scale=0.1).to(TDT[dt])
    y = A.double() @ W.double().T.contiguous() + b.double()
    odt = torch.float32 if epi == "gate" else TDT[dt]
    buf = torch.full((M * N + off + 8,), 7.0, dtype=odt, device=DEV)
    out = buf[off:off + M * N].view(M, N)
    if epi == "gate":
        rpg = max(1, M // 3)
        G, R = rnd((M + rpg - 1) // rpg, N, scale=0.5), rnd(M, N)
        y = R.double() + G.double().repeat_interleave(rpg, 0)[:M] * y
        bclib.linear(A, W, b, out, bclib.EPI_GATE_RES, res=R, gate=G, rows_per_gate=rpg)
    elif epi == "gelu":
        y = torch.nn.functional.gelu(y, approximate="tanh")
        bclib.linear(A, W, b, out, bclib.EPI_BIAS_GELU)
    else:
        bclib.linear(A, W, b, out)
    torch.cuda.synchronize()
    err = float((out.double() - y).norm() / y.norm())
    # bf16 outputs are rounded once (2^-9 relative at most, 1.7e-3 in the mean); else fp32 sums of K terms
    assert err <= (2.5e-3 if odt == torch.bfloat16 else 2e-6), err
    assert bool((buf[:off] == 7.0).all()) and bool((buf[off + M * N:] == 7.0).all())    # nothing written outside


# The phased kernel of large grids against 64 bits: 256 x 256 tiles (4100 x 4352)
# and 256 x 288 (4090 x 4600), ragged rows and columns, 2 to 7 k-steps (its
# prologue, its last two steps, and both parities of the main loop), a gate that
# changes within a tile.
@pytest.mark.parametrize("epi", ["bias", "gelu", "gate"])
@pytest.mark.parametrize("M,N,K", [(4100, 4352, 128), (4100, 4352, 192), (4100, 4352, 256), (4100, 4352, 448),
                                   (4090, 4600, 128), (4090, 4600, 192), (4090, 4600, 256), (4090, 4600, 448)])
def test_linear_large_grids(bclib, M, N, K, epi):
    test_linear_small_grids(bclib, "bf16", M, N, K, 0, epi)


# Small grids of the streaming attention: 16 queries per wave in workgroups of 4
# or 8 waves, queries one past a tile, key tiles of one key; and the resident
# workgroups of 4 waves (at most 256 workgroups of 64 queries).
@pytest.mark.parametrize("prescaled", [False, True])
@pytest.mark.parametrize("B,H,Tq,Tk,d", [
    (1, 2, 65, 257, 64), (1, 4, 1020, 300, 72), (2, 16, 1025, 321, 64), (1, 24, 1025, 385, 128), (1, 2, 129, 513, 128),
    (1, 3, 65, 256, 128), (1, 3, 70, 65, 32), (2, 30, 129, 640, 32)])
def test_attention_four_waves(bclib, prescaled, B, H, Tq, Tk, d):
    g = torch.Generator(device=DEV)
    g.manual_seed(Tq + d)
    q, k, v = (torch.empty((B, T, H, d), device=DEV).normal_(0.0, 2.0, generator=g).bfloat16() for T in (Tq, Tk, Tk))
    scale = np.log(2.0) if prescaled else d ** -0.5
    if prescaled:
        q = (q.float() * (1.4426950408889634 / d ** 0.5)).bfloat16()
    t = [a.double().permute(0, 2, 1, 3).contiguous() for a in (q, k, v)]
    want = (torch.softmax(t[0] @ t[1].transpose(2, 3).contiguous() * scale, -1) @ t[2]).permute(0, 2, 1, 3)
    out = torch.empty_like(q)
    bclib.attention(q, k, v, out, prescaled=prescaled)
    torch.cuda.synchronize()
    err = float((out.double() - want).norm() / want.norm())
    assert err <= 1e-2, err      # probabilities and outputs rounded to bf16 (about 3e-3 together)


# The 128 x 144 and 128 x 192 tiles: ragged rows and columns, every remainder of
# the k-steps by the four stages.
@pytest.mark.parametrize("epi", ["bias", "gelu", "gate"])
@pytest.mark.parametrize("M,N,K", [(3900, 1144, 1024), (3900, 1144, 1088), (3900, 1144, 1152), (3900, 1144, 1216),
                                   (1840, 3000, 1152), (1840, 3000, 1216), (1840, 3000, 1280), (1840, 3000, 1344)])
def test_linear_one_round(bclib, M, N, K, epi):
    test_linear_small_grids(bclib, "bf16", M, N, K, 0, epi)


# 128 x 128 tiles of more than one round: a last round of few workgroups, whose
# gated epilogue reads the residual ahead (544 tiles, K = 512; not at 448), and a
# fuller one (720 tiles); ragged rows and columns.
@pytest.mark.parametrize("epi", ["bias", "gelu", "gate"])
@pytest.mark.parametrize("M,N,K", [(3990, 2120, 512), (3990, 2120, 448), (5690, 2040, 512)])
def test_linear_last_round(bclib, M, N, K, epi):
    test_linear_small_grids(bclib, "bf16", M, N, K, 0, epi)


# Every workgroup shape of the bf16 attention at every head dim it is built for:
# (16-query groups per wave, waves, streaming key tiles) and a call that the
# choice sends there.  Ragged queries and keys; tests/test_attention_variants.py
# checks on the CPU that these calls still take these shapes.
ATT_VARIANTS = [((2, 8, 0), (8, 32, 300, 120)), ((1, 4, 0), (1, 3, 65, 70)), ((1, 8, 0), (4, 32, 130, 200)),
                ((4, 8, 1), (8, 32, 500, 300)), ((2, 4, 1), (2, 24, 1025, 300)), ((1, 8, 1), (1, 24, 1025, 385)),
                ((1, 4, 1), (1, 2, 65, 257))]
ATT_VARIANT_CASES = [(v, s + (d,)) for v, s in ATT_VARIANTS for d in (32, 64, 72, 128) if not (v[0] == 4 and d == 128)]


@pytest.mark.parametrize("prescaled", [False, True])
@pytest.mark.parametrize("variant,shape", ATT_VARIANT_CASES)
def test_attention_variants(bclib, variant, shape, prescaled):
    test_attention_four_waves(bclib, prescaled, *shape)
