"""The tile plan of the encode and prefill GEMM at its edges, against the oracle: row counts around
every tile height (ragged last tiles, a single row), K of one, two and three 64-wide steps (shorter
than the ring of LDS stages), whole column rounds with a leftover launch, and the K-sliced GELU, SwiGLU,
residual and store epilogues of problems with few rows."""
import numpy as np
import pytest

from oracle import vlm
from paper_2509_21301_amd import synth
from tests import stage_cases as sc

pytestmark = pytest.mark.gpu

TOL = 1e-4     # fp32 accumulation of exact bf16 products, compared norm-wise with float64


@pytest.mark.parametrize("m,k,n", [(1, 64, 128), (31, 128, 256), (32, 192, 256), (33, 1280, 3840), (63, 1280, 1280),
                                   (65, 640, 5120), (127, 1280, 128), (129, 3584, 4608), (200, 512, 37888),
                                   (255, 1280, 1280), (257, 320, 5120), (511, 1280, 3840), (700, 256, 9472),
                                   (1025, 1280, 1280), (4161, 128, 1280)])
def test_linear_tile_edges(gpu_lib, m, k, n):
    import torch
    x = synth.normal((m, k), 3, f"gt_x{m}x{k}", std=1.0)
    w = synth.normal((n, k), 3, f"gt_w{n}x{k}", std=0.05)
    base = synth.normal((m, n), 4, f"gt_o{m}x{n}", std=1.0)
    guard = torch.full((m + 1, n), 7.0, dtype=torch.float32, device="cuda")
    guard[:m].copy_(torch.from_numpy(base))
    gpu_lib.linear(gpu_lib.LINEAR_TILED, torch.from_numpy(x).cuda().to(torch.bfloat16),
                   torch.from_numpy(w).cuda().to(torch.bfloat16), guard[:m])
    torch.cuda.synchronize()
    assert vlm.max_rel_err(guard[:m].cpu().numpy(), base + vlm.linear(x, w)) < TOL
    assert bool((guard[m] == 7.0).all())          # nothing written past the last row


# 2560-wide layers with 256-wide MLPs: few tiles and a long K, so the MLP up projections (GELU here,
# SwiGLU below) run as K slices too; images of 4 and 40 patches, two at a time
@pytest.mark.parametrize("h,w", [(28, 28), (56, 140)])
def test_vit_few_rows(gpu_lib, h, w):
    import torch
    cfg = synth.VitConfig(hidden=2560, heads=32, mlp=256, layers=2, patch=14, merge=2, out_hidden=256, image_h=h,
                          image_w=w, name=f"vit_few_{h}x{w}")
    wt = synth.vit_weights(cfg, seed=8)
    imgs = synth.image(2, h, w, seed=3)
    out = gpu_lib.Vit(cfg, wt).encode(torch.from_numpy(imgs).cuda().to(torch.bfloat16)).float().cpu().numpy()
    for i in range(2):
        assert vlm.max_rel_err(out[i], vlm.vit_encode(imgs[i], wt, cfg)) < sc.TOL_BF16, f"image {i}"


# patch embedding with its position table (3456 patches x 1280: more tiles than one round of any tile)
def test_vit_patch_embed_positions(gpu_lib):
    import torch
    cfg = synth.VitConfig(hidden=1280, heads=16, mlp=256, layers=0, patch=4, merge=2, out_hidden=256, image_h=192,
                          image_w=288, name="vit_pos")
    for batch in (1, 4):
        wt = synth.vit_weights(cfg, seed=8)
        imgs = synth.image(batch, cfg.image_h, cfg.image_w, seed=3)
        out = gpu_lib.Vit(cfg, wt).encode(torch.from_numpy(imgs).cuda().to(torch.bfloat16)).float().cpu().numpy()
        for i in range(batch):
            assert vlm.max_rel_err(out[i], vlm.vit_encode(imgs[i], wt, cfg)) < sc.TOL_BF16, f"image {i}"


# patch extraction: odd patch sizes and row lengths (scalar and 16-byte image loads), more than 16 patches
# per grid row with a ragged last group, one patch, and patches too large for the LDS tile
@pytest.mark.parametrize("patch,h,w", [(7, 21, 133), (14, 28, 14 * 37), (16, 32, 16 * 21), (40, 40, 120), (75, 75, 150),
                                       (14, 14, 14)])
def test_patch_extraction(gpu_lib, patch, h, w):
    import torch
    cfg = synth.VitConfig(hidden=128, heads=2, mlp=128, layers=0, patch=patch, merge=1, out_hidden=128, image_h=h,
                          image_w=w, name=f"vit_patch{patch}_{h}x{w}")
    wt = synth.vit_weights(cfg, seed=8)
    imgs = synth.image(3, h, w, seed=3)
    for act, tol in ((gpu_lib.ACT_BF16, sc.TOL_BF16), (gpu_lib.ACT_F32, sc.TOL_F32)):
        out = gpu_lib.Vit(cfg, wt, act=act).encode(torch.from_numpy(imgs).cuda().to(torch.bfloat16)).float().cpu().numpy()
        for i in range(3):
            assert vlm.max_rel_err(out[i], vlm.vit_encode(imgs[i], wt, cfg)) < tol, f"image {i}"


# fp32 mode on both sides of its tile rule: 15x60 patches (all projections as 32x64 tiles, ragged rows)
# and 60x60 (the MLP up projection as 29 x 40 tiles of 128x128)
@pytest.mark.parametrize("h,w", [(60, 240), (240, 240)])
def test_vit_f32_tiles(gpu_lib, h, w):
    import torch
    cfg = synth.VitConfig(hidden=1280, heads=16, mlp=5120, layers=1, patch=4, merge=1, out_hidden=256, image_h=h,
                          image_w=w, name=f"vit_f32_{h}x{w}")
    wt = synth.vit_weights(cfg, seed=8)
    img = synth.image(1, h, w, seed=3)
    out = gpu_lib.Vit(cfg, wt, act=gpu_lib.ACT_F32).encode(torch.from_numpy(img).cuda().to(torch.bfloat16))[0].cpu().numpy()
    tokens = [0, 59, 60, 450, cfg.n_patches - 1]
    assert vlm.max_rel_err(out[tokens], vlm.vit_encode_tokens(img[0], wt, cfg, tokens)) < sc.TOL_F32


@pytest.mark.parametrize("n_vis,n_text", [(0, 1), (3, 30), (0, 33), (70, 60)])
def test_prefill_few_rows(gpu_lib, n_vis, n_text):
    import torch
    cfg = synth.LlmConfig(hidden=2560, n_q=20, n_kv=4, head_dim=128, inter=200, vocab=16384, layers=2, name="llm_few")
    wt = synth.llm_weights(cfg, seed=6)
    vis = synth.vision_embeds(n_vis, cfg.hidden) if n_vis else np.zeros((0, cfg.hidden), np.float32)
    ids = synth.text_ids(n_text, cfg.vocab)
    table, pool = synth.block_tables([n_vis + n_text], cfg.block, seed=5)
    kref = vlm.PagedKV(cfg.layers, pool, cfg.n_kv, cfg.block, cfg.head_dim)
    ref, _ = vlm.llm_prefill(vis, ids, wt, cfg, kv=kref, table=table[0])
    llm = gpu_lib.Llm(cfg, wt)
    kv = gpu_lib.KvPool(llm, pool)
    logits = torch.empty(cfg.vocab, dtype=torch.float32, device="cuda")
    llm.prefill(torch.from_numpy(vis).cuda().to(torch.bfloat16) if n_vis else None, torch.from_numpy(ids).cuda(),
                torch.from_numpy(table[0]).cuda(), kv, logits=logits)
    torch.cuda.synchronize()
    assert vlm.max_rel_err(logits.cpu().numpy(), ref) < sc.TOL_BF16
    ek, ev = sc.kv_errors(kref.k, kref.v, kv.k5.float().cpu().numpy(), kv.v5.float().cpu().numpy())
    assert ek < sc.TOL_BF16 and ev < sc.TOL_BF16


@pytest.mark.parametrize("m,k,n", [(17, 256, 16384), (32, 768, 16384)])
def test_thin_linear_ring(gpu_lib, m, k, n):
    import torch
    x = synth.normal((m, k), 5, f"gt_x{m}x{k}", std=1.0)
    w = synth.normal((n, k), 5, f"gt_w{n}x{k}", std=0.05)
    out = torch.ones((m, n), dtype=torch.float32, device="cuda")
    gpu_lib.linear(gpu_lib.LINEAR_THIN, torch.from_numpy(x).cuda().to(torch.bfloat16),
                   torch.from_numpy(w).cuda().to(torch.bfloat16), out)
    torch.cuda.synchronize()
    assert vlm.max_rel_err(out.cpu().numpy(), 1.0 + vlm.linear(x, w)) < TOL


# a head of 132,096 rows: the LM head's 128-row workgroups, one and two column groups, partly filled
# and on partitions, where small batches run it as 64-row workgroups
@pytest.mark.parametrize("bsz,cus", [(1, 0), (16, 0), (17, 0), (32, 0), (3, 128), (5, 128), (8, 192)])
def test_decode_wide_head(gpu_lib, bsz, cus):
    import torch
    cfg = synth.LlmConfig(hidden=256, n_q=4, n_kv=2, head_dim=64, inter=688, vocab=132096, layers=1, name="llm_head")
    wt = synth.llm_weights(cfg, seed=2)
    ctx = [5 + 3 * b for b in range(bsz)]
    tables, pool = synth.block_tables([c + 1 for c in ctx], cfg.block, seed=9)
    rng = np.random.default_rng(3)
    kref = vlm.PagedKV(cfg.layers, pool, cfg.n_kv, cfg.block, cfg.head_dim)
    kref.k[:] = synth.bf16_round(rng.standard_normal(kref.k.shape, dtype=np.float32))
    kref.v[:] = synth.bf16_round(rng.standard_normal(kref.v.shape, dtype=np.float32))
    llm = gpu_lib.Llm(cfg, wt)
    kv = gpu_lib.KvPool(llm, pool)
    kv.k5.copy_(torch.from_numpy(kref.k.astype(np.float32)).to(torch.bfloat16))
    kv.v5.copy_(torch.from_numpy(np.swapaxes(kref.v, -1, -2).astype(np.float32)).to(torch.bfloat16))
    ids, pos = synth.text_ids(bsz, cfg.vocab, seed=12), np.array(ctx, np.int32)
    logits = torch.full((bsz, cfg.vocab), float("nan"), dtype=torch.float32, device="cuda")
    stream = gpu_lib.set_stage_partition(gpu_lib.STAGE_DECODE, gpu_lib.make_cu_mask(cus)) if cus else None
    args = [torch.from_numpy(a).cuda() for a in (ids, pos, tables)]
    torch.cuda.synchronize()
    nxt = llm.decode(*args, kv, max_ctx=max(ctx) + 1, logits=logits, stream=stream)
    torch.cuda.synchronize()
    ref, _ = vlm.llm_decode_step(ids, pos, tables, kref, wt, cfg)
    got = logits.cpu().numpy()
    for b in range(bsz):
        assert vlm.max_rel_err(got[b], ref[b]) < sc.TOL_BF16, f"seq {b}"
    assert np.array_equal(nxt.cpu().numpy(), np.argmax(got, axis=1))      # the fused argmax, lowest id on ties


# gate/up of 8 x units row tiles: 8 or 32 tiles past the GPU's 256 compute units (one and two column groups,
# 4 chunks of K over 2..4 slices), 40 (more than the arrival counters hold: no slices), 200 on a partition of
# 64 compute units, 520 there (64-row workgroups with slices at batch 12, 128-row ones at 13), and 264 tiles in
# fp32; a second step on the same workspace finds its counters zero again
@pytest.mark.parametrize("bsz,units,cus,act", [(1, 33, 0, "bf16"), (8, 36, 0, "bf16"), (17, 36, 0, "bf16"),
                                               (32, 33, 0, "bf16"), (5, 37, 0, "bf16"), (3, 25, 64, "bf16"),
                                               (12, 65, 64, "bf16"), (13, 65, 64, "bf16"), (16, 33, 0, "f32")])
def test_decode_gate_up_tail(gpu_lib, bsz, units, cus, act):
    import torch
    cfg = synth.LlmConfig(hidden=1024, n_q=16, n_kv=4, head_dim=64, inter=256 * units, vocab=4096, layers=2, name="llm_tail")
    wt = synth.llm_weights(cfg, seed=2)
    ctx = [5 + 3 * b for b in range(bsz)]
    tables, pool = synth.block_tables([c + 1 for c in ctx], cfg.block, seed=9)
    rng = np.random.default_rng(3)
    kref = vlm.PagedKV(cfg.layers, pool, cfg.n_kv, cfg.block, cfg.head_dim)
    kref.k[:] = synth.bf16_round(rng.standard_normal(kref.k.shape, dtype=np.float32))
    kref.v[:] = synth.bf16_round(rng.standard_normal(kref.v.shape, dtype=np.float32))
    llm = gpu_lib.Llm(cfg, wt, act=gpu_lib.ACT_F32 if act == "f32" else gpu_lib.ACT_BF16)
    kv = gpu_lib.KvPool(llm, pool)
    kv.k5.copy_(torch.from_numpy(kref.k.astype(np.float32)).to(kv.k5.dtype))
    kv.v5.copy_(torch.from_numpy(np.swapaxes(kref.v, -1, -2).astype(np.float32)).to(kv.v5.dtype))
    ids, pos = synth.text_ids(bsz, cfg.vocab, seed=12), np.array(ctx, np.int32)
    stream = gpu_lib.set_stage_partition(gpu_lib.STAGE_DECODE, gpu_lib.make_cu_mask(cus)) if cus else None
    args = [torch.from_numpy(a).cuda() for a in (ids, pos, tables)]
    steps = []
    for _ in range(2):
        logits = torch.full((bsz, cfg.vocab), float("nan"), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        llm.decode(*args, kv, max_ctx=max(ctx) + 1, logits=logits, stream=stream)
        torch.cuda.synchronize()
        steps.append(logits.cpu().numpy())
    ref, _ = vlm.llm_decode_step(ids, pos, tables, kref, wt, cfg)
    for b in range(bsz):
        assert vlm.max_rel_err(steps[0][b], ref[b]) < (sc.TOL_F32 if act == "f32" else sc.TOL_BF16), f"seq {b}"
    assert np.array_equal(steps[0], steps[1])


# the prompt's rows and their first RMSNorm at the widths where the kernel's register rows change (full and
# partly filled), row counts that leave a workgroup partly filled
@pytest.mark.parametrize("hidden,layers,n_vis,n_text,act", [(1024, 1, 3, 2, "bf16"), (1280, 1, 0, 1, "bf16"),
                                                            (4096, 1, 6, 1, "bf16"), (512, 2, 2, 5, "bf16"),
                                                            (1280, 1, 4, 3, "f32"), (768, 2, 5, 1, "f32")])
def test_prefill_embedding(gpu_lib, hidden, layers, n_vis, n_text, act):
    import torch
    cfg = synth.LlmConfig(hidden=hidden, n_q=4, n_kv=2, head_dim=64, inter=256, vocab=16384, layers=layers, name="llm_embed")
    wt = synth.llm_weights(cfg, seed=6)
    f32 = act == "f32"
    vis = synth.vision_embeds(n_vis, cfg.hidden) if n_vis else np.zeros((0, cfg.hidden), np.float32)
    ids = synth.text_ids(n_text, cfg.vocab)
    table, pool = synth.block_tables([n_vis + n_text], cfg.block, seed=5)
    kref = vlm.PagedKV(cfg.layers, pool, cfg.n_kv, cfg.block, cfg.head_dim)
    ref, _ = vlm.llm_prefill(vis, ids, wt, cfg, kv=kref, table=table[0])
    llm = gpu_lib.Llm(cfg, wt, act=gpu_lib.ACT_F32 if f32 else gpu_lib.ACT_BF16)
    kv = gpu_lib.KvPool(llm, pool)
    logits = torch.empty(cfg.vocab, dtype=torch.float32, device="cuda")
    llm.prefill(torch.from_numpy(vis).cuda().to(torch.float32 if f32 else torch.bfloat16) if n_vis else None,
                torch.from_numpy(ids).cuda(), torch.from_numpy(table[0]).cuda(), kv, logits=logits)
    torch.cuda.synchronize()
    assert vlm.max_rel_err(logits.cpu().numpy(), ref) < (sc.TOL_F32 if f32 else sc.TOL_BF16)
