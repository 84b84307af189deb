"""GPU parity of lvlm_prefill_attn (the layer's attention with the scores as its by-product) against the CPU
oracle, through the C ABI.

Tolerances (max |gpu - oracle| / max |oracle|): outputs 2e-2 (bf16) / 1e-5 (fp32); the row normalisers and
the scores are fp32 whatever the input dtype: 1e-5.
"""
import numpy as np
import pytest
import torch

import paper_2509_00419_amd as lv
from oracle import lvlm_oracle as O
from workloads import configs

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = {torch.float32: 1e-5, torch.bfloat16: 2e-2}


def f64(t):
    return t.detach().double().cpu().numpy()


def rel_err(got, ref):
    got, ref = np.asarray(got, dtype=np.float64), np.asarray(ref, dtype=np.float64)
    return float(np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-30))


@pytest.fixture(scope="module")
def ctx():
    return lv.Context(0)


def _qkv(B, N, Hq, Hkv, d, dtype, seed, q_gain=1.0):
    """q, k, v as views of one fused projection output [B, N, Hq + 2 Hkv, d], as a model lays them out."""
    g = torch.Generator().manual_seed(seed)
    fused = torch.randn(B, N, Hq + 2 * Hkv, d, generator=g)
    fused[:, :, :Hq] *= q_gain
    fused = fused.to(dtype)
    return fused, (lambda t: (t[:, :, :Hq], t[:, :, Hq:Hq + Hkv], t[:, :, Hq + Hkv:]))


CASES = [
    # dtype, B, N, Hq, Hkv, d, causal, T, img_begin, n_img, q_gain        what it covers
    (torch.float32, 1, 640, 4, 4, 64, True, 32, 32, 576, 1.0),            # config 1
    (torch.float32, 2, 77, 4, 2, 128, True, 5, 3, 60, 2.0),               # fp32, d = 128, ragged
    (torch.float32, 1, 130, 2, 1, 64, False, 0, 0, 0, 1.0),               # fp32, no mask, attention only
    (torch.bfloat16, 2, 333, 6, 2, 128, True, 9, 5, 300, 1.0),            # ragged rows and keys, G = 3
    (torch.bfloat16, 1, 233, 8, 8, 64, False, 0, 0, 0, 1.0),              # d = 64, no mask, attention only
    (torch.bfloat16, 1, 257, 4, 2, 64, True, 40, 10, 200, 3.0),           # d = 64 causal, peaky rows, one row past a block
    (torch.bfloat16, 3, 500, 8, 4, 128, True, 64, 20, 400, 1.0),          # 12 (batch, KV head) pairs: 8 + 4 over the XCDs
    (torch.bfloat16, 1, 31, 2, 2, 128, True, 31, 0, 20, 1.0),             # shorter than one tile, every row an instruction row
    (torch.bfloat16, 1, 1, 2, 1, 128, True, 1, 0, 1, 1.0),                # one token
    (torch.float32, 1, 1, 2, 2, 64, True, 1, 0, 1, 1.0),                  # one token, fp32
    (torch.bfloat16, 2, 150, 4, 2, 128, False, 10, 5, 100, 1.0),          # scores without a causal mask
    (torch.bfloat16, 1, 128, 2, 1, 128, True, 3, 0, 125, 1.0),            # exactly one full query block
    (torch.bfloat16, 1, 2176, 28, 4, 128, True, 64, 64, 2048, 1.0),       # config 2 layer
]


@pytest.mark.parametrize("dtype,B,N,Hq,Hkv,d,causal,T,img0,n_img,gain", CASES)
def test_prefill_attn_matches_oracle(ctx, dtype, B, N, Hq, Hkv, d, causal, T, img0, n_img, gain):
    fused, split = _qkv(B, N, Hq, Hkv, d, dtype, 100 + N, gain)
    q, k, v = split(fused)
    qd, kd, vd = split(fused.to(DEV))
    out, lse, sh, sm = ctx.prefill_attn(qd, kd, vd, causal=causal, n_text=T, img_begin=img0, n_img=n_img)
    torch.cuda.synchronize()
    o_out, o_lse = O.prefill_attn(f64(q), f64(k), f64(v), causal=causal, dtype="bf16" if dtype == torch.bfloat16 else "f32")
    assert rel_err(out.float().cpu(), o_out) < TOL[dtype]
    assert np.abs(lse.cpu().numpy() - o_lse).max() < 1e-5 * max(1.0, np.abs(o_lse).max())
    if T > 0:
        osh, osm = O.score_tokens(f64(q[:, N - T:]), f64(k), q_pos0=N - T, img_begin=img0, n_img=n_img, causal=causal)
        assert rel_err(sh.cpu(), osh) < 1e-5 and rel_err(sm.cpu(), osm) < 1e-5
        # and exactly what lvlm_score_tokens gives from the same normalisers
        sh2, sm2 = ctx.score_tokens(qd[:, N - T:], kd, q_pos0=N - T, img_begin=img0, n_img=n_img, causal=causal,
                                    row_lse=lse[:, :, N - T:].contiguous())
        assert torch.equal(sh, sh2) and torch.equal(sm, sm2)
    else:
        assert sh is None and sm is None


def test_prefill_attn_config3_shape_two_sequences(ctx):
    # InternVL2.5-8B-shaped layer (32 / 8 heads, 1792 image + 96 text tokens), two of the eight sequences for the oracle
    w = configs.CFG3
    B, N = 2, w.seq_len
    fused, split = _qkv(B, N, w.n_q_heads, w.n_kv_heads, w.head_dim, torch.bfloat16, 7)
    q, k, v = split(fused)
    qd, kd, vd = split(fused.to(DEV))
    out, lse, sh, sm = ctx.prefill_attn(qd, kd, vd, n_text=w.n_text, img_begin=w.n_sys, n_img=w.n_img)
    o_out, o_lse = O.prefill_attn(f64(q), f64(k), f64(v), dtype="bf16")
    assert rel_err(out.float().cpu(), o_out) < 2e-2
    assert np.abs(lse.cpu().numpy() - o_lse).max() < 1e-5 * np.abs(o_lse).max()
    osh, osm = O.score_tokens(f64(q[:, N - w.n_text:]), f64(k), q_pos0=N - w.n_text, img_begin=w.n_sys, n_img=w.n_img)
    assert rel_err(sh.cpu(), osh) < 1e-5 and rel_err(sm.cpu(), osm) < 1e-5


def test_prefill_attn_config5_shape_sampled_group(ctx):
    # 16512 tokens, 48 / 8 heads on the GPU; the oracle checks one KV group (its 6 query heads), every row
    w = configs.CFG5
    N, Hq, Hkv, d = w.seq_len, w.n_q_heads, w.n_kv_heads, w.head_dim
    fused, split = _qkv(1, N, Hq, Hkv, d, torch.bfloat16, 11)
    q, k, v = split(fused)
    qd, kd, vd = split(fused.to(DEV))
    out, lse, sh, sm = ctx.prefill_attn(qd, kd, vd, n_text=w.n_text, img_begin=w.n_sys, n_img=w.n_img)
    torch.cuda.synchronize()
    g, G = Hkv - 1, Hq // Hkv
    heads = slice(g * G, (g + 1) * G)
    o_out, o_lse = O.prefill_attn(f64(q[:, :, heads]), f64(k[:, :, g:g + 1]), f64(v[:, :, g:g + 1]), dtype="bf16")
    assert rel_err(out[:, :, heads].float().cpu(), o_out) < 2e-2
    assert np.abs(lse[:, heads].cpu().numpy() - o_lse).max() < 1e-5 * np.abs(o_lse).max()
    osh, _ = O.score_tokens(f64(q[:, N - w.n_text:, heads]), f64(k[:, :, g:g + 1]), q_pos0=N - w.n_text,
                            img_begin=w.n_sys, n_img=w.n_img)
    assert rel_err(sh[:, g:g + 1].cpu(), osh) < 1e-5
    # properties that hold for every head: rows are convex combinations of the values they see
    vmax = vd.float().abs().amax()
    assert float(out.float().abs().amax()) <= float(vmax) * (1 + 2 ** -7)
    assert torch.isfinite(lse).all()


@pytest.mark.parametrize("d", [64, 128])
def test_prefill_attn_row_sums_of_long_rows(ctx, d):
    """Sixteen thousand keys of which few weigh much (unit noise plus three times a salience): small probabilities must
    not drop out of a row's sum.  A tile's probabilities are summed on their own before they meet the running sum, some
    N / 32 + 16 additions a lane; one by one into the running sum they leave the normalisers about 4e-6 too low
    (rms 4.2e-6), tile by tile without a bias (rms of the sum 2e-7).  The bounds: the sum's logarithm, the reference's
    product and their total are each rounded at a magnitude below 16, at most 9.5e-7 apiece and 0.6e-6 in rms, and do not
    lean to a side."""
    N, rows = 16512, 512
    g = torch.Generator().manual_seed(23)
    q, k, v = (torch.randn(1, N, 1, d, generator=g) for _ in range(3))
    u = torch.zeros(d)
    u[0] = 1.0
    k += 3.0 * d ** 0.25 * torch.randn(1, N, 1, 1, generator=g) * u
    q[..., 0] = d ** 0.25
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    _, lse, _, _ = ctx.prefill_attn(q.to(DEV), k.to(DEV), v.to(DEV))
    s = (q[0, N - rows:, 0].double() @ k[0, :, 0].double().T) * d ** -0.5
    s = s.masked_fill(torch.arange(N)[None, :] > torch.arange(N - rows, N)[:, None], float("-inf"))
    ref = torch.logsumexp(s, dim=1)
    assert float(ref.abs().max()) < 24.0
    err = lse[0, 0, N - rows:].cpu().double() - ref
    assert abs(float(err.mean())) < 1e-6 and float(err.pow(2).mean().sqrt()) < 2e-6


def test_prefill_attn_logits_far_above_the_first_tile(ctx):
    """Rows whose later logits exceed everything in the first 32 keys by far more than fp32 can hold as a
    probability ratio (natural-log distance 120): the kernel that fixes its reference at the first tile must
    give these workgroups to the one that follows the running maximum.  Also the reverse (a dominant first key)
    and ordinary rows in the same launch."""
    B, N, Hq, Hkv, d = 1, 420, 4, 2, 64
    g = torch.Generator().manual_seed(3)
    q = 0.05 * torch.randn(B, N, Hq, d, generator=g)
    k = 0.05 * torch.randn(B, N, Hkv, d, generator=g)
    v = torch.randn(B, N, Hkv, d, generator=g)
    q[:, :, 0:2, 0] = 22.0                       # heads 0, 1 (KV head 0): logit = 22 * k0 / 8
    k[:, :32, 0, 0] = -22.0                      # first tile: -60.5
    k[:, 32:, 0, 0] = 22.0                       # later keys: +60.5
    k[:, 200, 0, 0] = 30.0                       # and one at +82.5
    q[:, :, 2, 0] = 22.0                         # head 2 (KV head 1): a dominant first key, the rest far below
    k[:, 0, 1, 0] = 22.0
    k[:, 1:, 1, 0] = -22.0
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    out, lse, sh, sm = ctx.prefill_attn(q.to(DEV), k.to(DEV), v.to(DEV), n_text=20, img_begin=8, n_img=380)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all() and torch.isfinite(lse).all()
    o_out, o_lse = O.prefill_attn(f64(q), f64(k), f64(v), dtype="bf16")
    assert rel_err(out.float().cpu(), o_out) < 2e-2
    assert np.abs(lse.cpu().numpy() - o_lse).max() < 1e-5 * np.abs(o_lse).max()
    osh, osm = O.score_tokens(f64(q[:, N - 20:]), f64(k), q_pos0=N - 20, img_begin=8, n_img=380)
    assert rel_err(sh.cpu(), osh) < 1e-5 and rel_err(sm.cpu(), osm) < 1e-5


def test_prefill_attn_far_logits_in_the_middle_of_a_long_row(ctx):
    """One sequence of nine query blocks with few heads; logits that jump far above everything before them in the
    middle of the rows (natural-log distance 120 and more), so that only the workgroups whose rows reach those keys
    do them again with the running reference, the others do not, in the same launch."""
    B, N, Hq, Hkv, d = 1, 1100, 4, 2, 128
    g = torch.Generator().manual_seed(5)
    q = 0.05 * torch.randn(B, N, Hq, d, generator=g)
    k = 0.05 * torch.randn(B, N, Hkv, d, generator=g)
    v = torch.randn(B, N, Hkv, d, generator=g)
    q[:, :, 0:2, 0] = 26.0                       # heads 0, 1: logit = 26 * k0 / sqrt(128)
    k[:, :, 0, 0] = -26.0                        # -59.8 everywhere ...
    k[:, 300:330, 0, 0] = 26.0                   # ... but +59.8 on 30 keys inside a later part
    k[:, 700, 0, 0] = 30.0
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    out, lse, sh, sm = ctx.prefill_attn(q.to(DEV), k.to(DEV), v.to(DEV), n_text=40, img_begin=16, n_img=1000)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all() and torch.isfinite(lse).all()
    o_out, o_lse = O.prefill_attn(f64(q), f64(k), f64(v), dtype="bf16")
    assert rel_err(out.float().cpu(), o_out) < 2e-2
    assert np.abs(lse.cpu().numpy() - o_lse).max() < 1e-5 * np.abs(o_lse).max()
    osh, osm = O.score_tokens(f64(q[:, N - 40:]), f64(k), q_pos0=N - 40, img_begin=16, n_img=1000)
    assert rel_err(sh.cpu(), osh) < 1e-5 and rel_err(sm.cpu(), osm) < 1e-5


@pytest.mark.parametrize("B,N,Hq,Hkv,d", [
    (1, 200, 3, 1, 64), (1, 200, 11, 1, 128),     # heads that do not fill the eight XCDs: workgroups without a block
    (16, 250, 32, 2, 64), (16, 250, 32, 2, 128),  # 1024 workgroups, several to a compute unit, some with a second sweep, some without
    (35, 500, 16, 2, 64), (35, 500, 16, 2, 128),  # 2240: blocks of several tiles in front of the second sweep's
    (1376, 300, 8, 1, 64)])                       # 33024: many turns of the chip
def test_prefill_attn_many_far_logits(ctx, B, N, Hq, Hkv, d):
    """Every query block of two sequences out of three sees later logits far beyond the reference of its first tile (natural-log
    distance 120): its workgroup does it again with the running reference, in the LDS that the first sweep and its output used."""
    g = torch.Generator(device=DEV).manual_seed(N + d)
    q, k, v = (torch.randn(B, N, h, d, generator=g, device=DEV) for h in (Hq, Hkv, Hkv))
    a = (60.0 * d ** 0.5) ** 0.5
    far = (torch.arange(B, device=DEV) % 3 != 1).float()[:, None, None]
    q, k = 0.05 * q, 0.05 * k
    q[..., 0] = a * far
    k[..., 0] = a * far
    k[:, :32, :, 0] = -a * far
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    out = torch.full((B, N, Hq, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    out, lse, _, _ = ctx.prefill_attn(q, k, v, out=out)
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
    pick = sorted({0, B // 2, B - 1, max(B - 2, 0)})
    o_out, o_lse = O.prefill_attn(f64(q[pick].cpu()), f64(k[pick].cpu()), f64(v[pick].cpu()), dtype="bf16")
    assert rel_err(out[pick].float().cpu(), o_out) < 2e-2
    assert np.abs(lse[pick].cpu().numpy() - o_lse).max() < 1e-5 * np.abs(o_lse).max()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("wave", [0, 1])
def test_prefill_attn_far_logits_of_one_wave(ctx, d, wave):
    """Of a block's 128 rows only one wave's 64 see logits far beyond their first tile: the other wave has written its rows by then,
    and writes them again.  Whole, ragged and single-wave blocks, rows of a wider array beside which nothing is written."""
    B, N, Hq, Hkv = 3, 450, 5, 1
    g = torch.Generator().manual_seed(70 + d + wave)
    q, k, v = (torch.randn(B, N, h, d, generator=g) for h in (Hq, Hkv, Hkv))
    a = (60.0 * d ** 0.5) ** 0.5
    far = (torch.arange(N) // 64 % 2 == wave).float()[None, :, None]
    q, k = 0.05 * q, 0.05 * k
    q[..., 0] = a * far
    k[..., 0] = a
    k[:, :32, :, 0] = -a
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    wide = torch.full((B, N, Hq, d + 8), -7.0, dtype=torch.bfloat16, device=DEV)
    _, lse, _, _ = ctx.prefill_attn(q.to(DEV), k.to(DEV), v.to(DEV), out=wide[..., :d])
    o_out, o_lse = O.prefill_attn(f64(q), f64(k), f64(v), dtype="bf16")
    assert rel_err(wide[..., :d].float().cpu(), o_out) < 2e-2
    assert np.abs(lse.cpu().numpy() - o_lse).max() < 1e-5 * np.abs(o_lse).max()
    assert bool((wide[..., d:] == -7.0).all())


@pytest.mark.parametrize("d,which", [(64, "k"), (128, "v"), (128, "kv")])
def test_prefill_attn_rows_64_mib_apart(ctx, d, which):
    """Row strides of 64 MiB, beyond the 32-bit offsets inside a tile of the kernels that pipeline or share tiles: attention
    and scores of such rows go to the kernels with 64-bit addresses (a whole and a ragged tile, 2.6 GB apart)."""
    N, T, H, step = 40, 6, 2, 1 << 25
    g = torch.Generator().manual_seed(d)
    q, k, v = (torch.randn(1, N, H, d, generator=g).bfloat16() for _ in range(3))

    def apart(x):
        t = torch.empty((N - 1) * step + H * d, dtype=torch.bfloat16, device=DEV).as_strided((1, N, H, d), (N * step, step, d, 1))
        return t.copy_(x.to(DEV))
    kd, vd = (apart(x) if c in which else x.to(DEV) for c, x in (("k", k), ("v", v)))
    out, lse, sh, sm = ctx.prefill_attn(q.to(DEV), kd, vd, n_text=T, img_begin=3, n_img=30)
    o_out, o_lse = O.prefill_attn(f64(q), f64(k), f64(v), dtype="bf16")
    assert rel_err(out.float().cpu(), o_out) < 2e-2
    assert np.abs(lse.cpu().numpy() - o_lse).max() < 1e-5 * np.abs(o_lse).max()
    kw = dict(q_pos0=N - T, img_begin=3, n_img=30)
    osh, osm = O.score_tokens(f64(q[:, N - T:]), f64(k), **kw)
    assert rel_err(sh.cpu(), osh) < 1e-5 and rel_err(sm.cpu(), osm) < 1e-5
    sh, sm = ctx.score_tokens(q[:, N - T:].to(DEV), kd, **kw)
    assert rel_err(sh.cpu(), osh) < 1e-5 and rel_err(sm.cpu(), osm) < 1e-5


def test_prefill_attn_random_shapes(ctx):
    """Seeded sweep over small shapes: lengths around the tile and block edges, head counts and groups (G = 1 ... 7),
    both head dimensions and dtypes, with and without the mask, any number of instruction rows, any image span,
    flat and peaky rows."""
    rng = np.random.default_rng(20250901)
    for it in range(24):
        dtype = torch.bfloat16 if rng.random() < 0.8 else torch.float32
        d = int(rng.choice([64, 128]))
        Hkv, G = int(rng.choice([1, 2, 3, 4, 8])), int(rng.choice([1, 2, 4, 5, 7]))
        Hq = Hkv * G
        B = int(rng.choice([1, 1, 2, 3, 9]))
        N = int(rng.choice([1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 255, 256, 257, 300, 511, 513, 640]))
        if dtype == torch.float32:
            N = min(N, 300)
        if B * Hq * N * N > 4e7:
            B = 1
        causal = bool(rng.random() < 0.8)
        T = int(rng.integers(0, min(N, 70) + 1))
        n_img = int(rng.integers(1, N + 1)) if T > 0 else 0
        img0 = int(rng.integers(0, N - n_img + 1)) if T > 0 else 0
        fused, split = _qkv(B, N, Hq, Hkv, d, dtype, 3000 + it, float(rng.choice([1.0, 1.0, 3.0, 6.0])))
        q, k, v = split(fused)
        qd, kd, vd = split(fused.to(DEV))
        out, lse, sh, sm = ctx.prefill_attn(qd, kd, vd, causal=causal, n_text=T, img_begin=img0, n_img=n_img)
        torch.cuda.synchronize()
        case = (it, dtype, B, N, Hq, Hkv, d, causal, T, img0, n_img)
        o_out, o_lse = O.prefill_attn(f64(q), f64(k), f64(v), causal=causal, dtype="bf16" if dtype == torch.bfloat16 else "f32")
        assert rel_err(out.float().cpu(), o_out) < TOL[dtype], case
        assert np.abs(lse.cpu().numpy() - o_lse).max() < 1e-5 * max(1.0, np.abs(o_lse).max()), case
        if T > 0:
            osh, osm = O.score_tokens(f64(q[:, N - T:]), f64(k), q_pos0=N - T, img_begin=img0, n_img=n_img, causal=causal)
            assert rel_err(sh.cpu(), osh) < 1e-5 and rel_err(sm.cpu(), osm) < 1e-5, case


# fp32 calls with the launch their sizes take (tests/test_host_prefill_rules.py holds the library's rule to it): blocks of 16 rows, one or
# two to a workgroup, or tiles shared by 128 rows; "dealt": causal blocks dealt out to the compute units, "grouped": an XCD's heads in groups
F32_ROW_BLOCKS = [
    (1, 1, 1, 1, 64, True, "one"), (2, 15, 4, 4, 64, True, "one"), (1, 16, 2, 1, 128, False, "one"), (1, 17, 4, 2, 64, True, "one"),
    (1, 97, 3, 1, 128, True, "one"), (1, 128, 2, 2, 64, True, "one"), (1, 129, 2, 2, 64, False, "one"),
    (2, 161, 4, 1, 128, True, "one"), (683, 33, 8, 4, 64, True, "two"), (1, 385, 24, 4, 128, True, "one dealt")]
F32_WHOLE_TURNS = [
    (64, 50, 4, 4, 64, True, "shared"), (64, 64, 4, 2, 64, False, "shared"),             # one block, one turn of the chip
    (32, 125, 8, 4, 64, True, "shared"), (64, 128, 4, 1, 64, False, "shared"),
    (32, 250, 4, 4, 64, False, "shared"), (64, 640, 4, 4, 64, False, "shared"),          # two blocks, five
    (64, 250, 4, 2, 64, True, "shared dealt"), (64, 255, 4, 4, 64, True, "shared dealt"),        # causal, beyond one turn: two blocks
    (32, 500, 4, 4, 64, True, "shared dealt"), (63, 500, 2, 1, 64, True, "shared dealt"),        # four, of 128 heads and of quarters of 126
    (64, 640, 4, 4, 64, True, "shared dealt"),                                                   # five
    (32, 250, 4, 4, 64, True, "one dealt"), (16, 510, 4, 4, 64, True, "one dealt"),      # one turn of several causal blocks: not shared
    (8, 610, 26, 2, 64, True, "one dealt"), (64, 130, 4, 4, 64, True, "one dealt"),      # a last turn of 16, a last block of two rows
    (64, 1, 4, 4, 128, True, "shared"), (64, 31, 4, 4, 128, False, "shared"), (50, 33, 4, 2, 128, True, "shared"),
    (32, 129, 4, 1, 128, True, "shared"),                                                # 200 of 256 places; two blocks in one turn
    (16, 500, 4, 4, 128, False, "shared"), (8, 640, 7, 1, 128, True, "one dealt"),
    (100, 643, 4, 2, 128, True, "two grouped"),                                          # six blocks: sixteen-row blocks again
    (683, 33, 8, 4, 64, False, "two"), (205, 128, 10, 2, 128, False, "two"),             # ... a last turn of two
    (100, 700, 4, 2, 64, True, "two grouped"), (100, 700, 4, 1, 64, True, "two dealt"), (50, 643, 8, 1, 128, True, "two dealt"),
    (23, 194, 9, 3, 128, True, "shared dealt"), (47, 500, 5, 5, 64, True, "shared dealt"),       # heads no multiple of eight: 207, 235
    (31, 511, 8, 8, 64, True, "shared dealt"), (26, 700, 8, 8, 64, True, "one grouped"),         # 248; heads of an XCD in groups of 16
    (40, 643, 10, 10, 128, True, "two grouped"), (60, 700, 7, 7, 64, True, "two grouped"),       # ... of 50, eight at a time; of 53
    (13, 530, 12, 12, 128, True, "one grouped")]
F32_DEALT = [
    (1, 1024, 4, 4, 64, True, "one"),               # 256 blocks: the plain grid
    (1, 1025, 4, 2, 64, True, "one dealt"),         # 260: halves of heads, a turn of an XCD's 32 compute units and one block
    (1, 4097, 1, 1, 64, True, "one dealt"),         # eighths of one head, 33 levels of which the last is one part's
    (1, 1377, 3, 1, 128, True, "one dealt"),        # three eighths to an XCD, a turn and one block
    (3, 1300, 2, 1, 64, True, "one dealt"),         # quarters
    (5, 700, 5, 1, 64, True, "one dealt"),          # 25 heads of 44 blocks
    (2, 660, 8, 2, 128, False, "one"),              # whole heads, no mask
    (64, 129, 5, 1, 64, True, "one dealt"),         # nine blocks to each of 320 heads
    (16, 500, 8, 2, 64, True, "shared dealt"),      # shared tiles, four blocks of 128 heads
    (9, 500, 28, 4, 128, True, "shared dealt"),     # ... of 252 heads in halves
    (27, 700, 4, 2, 64, True, "one dealt"),         # six: blocks of 16 rows, whole turns
    (16, 512, 4, 4, 64, True, "one dealt"),         # one turn of four blocks: not shared
    (41, 64, 4, 4, 64, True, "one"), (25, 112, 4, 4, 64, True, "one"),                   # too short to level, 700 blocks
    (29, 112, 4, 4, 64, True, "one dealt"), (16, 113, 3, 1, 64, True, "one dealt"),      # 812; 384, one token more
    (37, 112, 5, 1, 128, True, "one"), (11, 113, 3, 1, 128, True, "one dealt"),          # of 128 channels
    (29, 135, 13, 13, 64, True, "one dealt")]       # 377 heads of nine blocks, the last XCD with 41 instead of 48


@pytest.mark.parametrize("B,N,Hq,Hkv,d,causal,form", F32_ROW_BLOCKS)
def test_prefill_attn_fp32_row_blocks_and_key_tiles(ctx, B, N, Hq, Hkv, d, causal, form):
    fused, split = _qkv(B, N, Hq, Hkv, d, torch.float32, 500 + N, 2.0)
    q, k, v = split(fused)
    out, lse, _, _ = ctx.prefill_attn(*split(fused.to(DEV)), causal=causal)
    o_out, o_lse = O.prefill_attn(f64(q), f64(k), f64(v), causal=causal, dtype="f32")
    assert rel_err(out.cpu(), o_out) < 1e-5
    assert np.abs(lse.cpu().numpy() - o_lse).max() < 1e-5 * max(1.0, np.abs(o_lse).max())


@pytest.mark.parametrize("B,N,Hq,Hkv,d,causal,form", F32_WHOLE_TURNS)
def test_prefill_attn_fp32_shared_tiles(ctx, B, N, Hq, Hkv, d, causal, form):
    """fp32 launches of whole turns of the chip: the kernel whose four waves share their tiles, at the edges of its rule, of
    its 128-row blocks and of its 32-key tiles.  Sampled sequences against the oracle, every row written."""
    fused, split = _qkv(B, N, Hq, Hkv, d, torch.float32, 700 + N, 2.0)
    out = torch.full((B, N, Hq, d), float("nan"), device=DEV)
    out, lse, _, _ = ctx.prefill_attn(*split(fused.to(DEV)), causal=causal, out=out)
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
    pick = [0, B // 2, B - 1]
    q, k, v = (x[pick] for x in split(fused))
    o_out, o_lse = O.prefill_attn(f64(q), f64(k), f64(v), causal=causal, dtype="f32")
    assert rel_err(out[pick].cpu(), o_out) < 1e-5
    assert np.abs(lse[pick].cpu().numpy() - o_lse).max() < 1e-5 * max(1.0, np.abs(o_lse).max())


@pytest.mark.parametrize("B,N,Hq,Hkv,d,causal,form", F32_DEALT)
def test_prefill_attn_fp32_blocks_dealt_to_compute_units(ctx, B, N, Hq, Hkv, d, causal, form):
    """Every block of every head is done once, however heads are cut for the XCDs and turns end."""
    fused, split = _qkv(B, N, Hq, Hkv, d, torch.float32, 900 + N, 2.0)
    out = torch.full((B, N, Hq, d), float("nan"), device=DEV)
    out, lse, _, _ = ctx.prefill_attn(*split(fused.to(DEV)), causal=causal, out=out)
    q, k, v = split(fused)
    o_out, o_lse = O.prefill_attn(f64(q), f64(k), f64(v), causal=causal, dtype="f32")
    assert rel_err(out.cpu(), o_out) < 1e-5
    assert np.abs(lse.cpu().numpy() - o_lse).max() < 1e-5 * max(1.0, np.abs(o_lse).max())


@pytest.mark.parametrize("N", [1, 3, 31, 33, 63, 65, 97, 127, 130, 161])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("far", [False, True])
def test_prefill_attn_writes_its_rows_and_nothing_else(ctx, N, d, far):
    """Rows leave the bf16 kernels several to a store: block and store edges, into rows of a wider and longer array whose other
    elements stay as they were; `far`: every block is done again with the running reference."""
    B, Hq, Hkv = 2, 5, 1
    g = torch.Generator().manual_seed(N + d)
    q, k, v = (torch.randn(B, N, h, d, generator=g) for h in (Hq, Hkv, Hkv))
    if far:
        q, k = 0.05 * q, 0.05 * k
        q[..., 0] = k[..., 0] = (60.0 * d ** 0.5) ** 0.5
        k[:, :32, :, 0] *= -1.0
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    wide = torch.full((B, N + 5, Hq + 2, d + 8), -7.0, dtype=torch.bfloat16, device=DEV)
    out = wide[:, 2:2 + N, 1:1 + Hq, :d]
    ctx.prefill_attn(q.to(DEV), k.to(DEV), v.to(DEV), out=out)
    o_out, _ = O.prefill_attn(f64(q), f64(k), f64(v), dtype="bf16")
    assert rel_err(out.float().cpu(), o_out) < 2e-2
    out.fill_(-7.0)
    assert bool((wide == -7.0).all())


def test_prefill_attn_rejects_bad_arguments(ctx):
    fused, split = _qkv(1, 64, 4, 2, 64, torch.bfloat16, 1)
    qd, kd, vd = split(fused.to(DEV))
    with pytest.raises(lv.LvlmError):
        ctx.prefill_attn(qd, kd, vd, scale=0.0)                     # scale must be positive
    with pytest.raises(lv.LvlmError):
        ctx.prefill_attn(qd, kd, vd, n_text=65, img_begin=0, n_img=10)      # more instruction rows than rows
    with pytest.raises(lv.LvlmError):
        ctx.prefill_attn(qd, kd, vd, n_text=8, img_begin=60, n_img=10)      # image span outside the sequence
