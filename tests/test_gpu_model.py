"""GPU parity: prefill / verify_forward against the oracle's full-recompute transformer forward."""
import numpy as np
import pytest
import torch

from oracle.forward import forward
from paper_2505_15141_amd import synth

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}          # absolute tolerance on logits


def bs():
    from paper_2505_15141_amd import binding
    return binding


MID = synth.cfg(4, 512, 8, 64, 1408, 4096, dtype="bf16")
MID_GQA = synth.cfg(3, 512, 8, 64, 1024, 2048, n_kv_heads=2, dtype="bf16")
WIDE = synth.cfg(2, 1024, 8, 128, 2816, 8192, n_kv_heads=2, dtype="bf16")
ODD_F32 = synth.cfg(2, 72, 3, 24, 104, 130, dtype="f32")
ODD_BF16 = synth.cfg(2, 96, 2, 64, 160, 1000, n_kv_heads=1, dtype="bf16")   # row counts that are not multiples of 64
# narrow but with many projection columns: 432 units of 16 columns for QKV and for gate/up, i.e. two or one per compute
# unit, which is where verification passes of up to 16 rows take the whole-K projections with fused epilogues
ROWS = synth.cfg(2, 256, 36, 64, 6912, 512, dtype="bf16")
ROWS_GQA = synth.cfg(1, 320, 36, 128, 6912, 512, n_kv_heads=9, dtype="bf16")
ROWS_MANY = synth.cfg(1, 128, 72, 64, 10240, 512, dtype="bf16")             # 864 and 640 units: four / three per compute unit


def setup(c, B, max_len, seed, std=None, packed=False):
    W = synth.make_weights(c, seed, std if std is not None else 0.02 * (4096 / c["d_model"]) ** 0.5 if c["dtype"] == "bf16" else 0.02)
    if c["dtype"] == "bf16":
        W = {k: (v if k.endswith("norm") else synth.to_bf16_grid(v)) for k, v in W.items()}
    m = bs().Model.from_numpy(c, W)
    if packed:
        m.pack(release_originals=True)
    kv = bs().KV(m, B, max_len)
    return W, m, kv


def off(got, ref):
    """Relative error in the 2-norm.  Activations are two bf16 planes; a second plane left out, or taken from the row beside it, in front of a single
    projection costs 1.6e-3 and more in the models below (1.6e-3 in front of down or the LM head, 2.3e-3 of O and gate/up, 6e-3 of QKV: the oracle with
    that projection's input rounded), which stays within the absolute tolerance."""
    got = got.cpu().numpy().astype(np.float64)
    return np.linalg.norm(got - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("c,B,n_prefix,q_len,packed", [
    (synth.TINY_TARGET, 1, 32, 5, False), (synth.TINY_DRAFT, 2, 9, 3, False), (ODD_F32, 3, 17, 4, False),
    (MID, 1, 70, 9, False), (MID_GQA, 2, 130, 5, False), (WIDE, 1, 200, 9, False), (MID, 3, 1, 2, False),
    (MID, 1, 70, 9, True), (MID_GQA, 2, 130, 5, True), (WIDE, 1, 200, 9, True), (MID, 3, 1, 2, True),
    (ODD_BF16, 1, 40, 7, False), (ODD_BF16, 2, 150, 3, True),
    # at most four rows on packed weights: the fused few-row schedule of the draft steps
    (MID, 1, 70, 2, True), (MID_GQA, 2, 130, 1, True), (WIDE, 1, 200, 4, True), (ODD_BF16, 2, 150, 2, True),
    (MID, 4, 33, 1, True), (WIDE, 1, 1, 1, True),
    # prompt chunks of 120 and 250..290 rows: the many-row kernel with 8 and 16 row tiles, one and two blocks of 256 rows
    (MID, 1, 120, 3, True), (MID_GQA, 3, 40, 2, False), (MID, 1, 250, 3, True), (ODD_BF16, 1, 290, 2, False),
    # 129..224 rows: the many-row kernel with 10, 12 and 14 row tiles; several 16-row attention tiles per head
    (MID, 1, 150, 3, True), (ODD_BF16, 1, 185, 2, False), (MID_GQA, 1, 215, 2, True),
    # more than 256 rows: several blocks of 256 rows in one GEMM launch (ragged last block), attention over many row tiles
    (MID, 1, 700, 3, True), (MID_GQA, 4, 128, 2, False), (ODD_BF16, 1, 300, 2, True),
    # 36..45 rows in the verification pass itself (a batch): the many-row kernel for every projection and for the LM head,
    # with a vocabulary that is no multiple of 16
    (ODD_BF16, 5, 20, 9, True), (MID, 4, 30, 9, False),
    # a prompt longer than the largest chunk: 1024 rows (four blocks of 256), then the rest against 1024 cached tokens
    (MID_GQA, 1, 1100, 2, True),
    # grouped queries with 17..32 rows per kv head: two row tiles share every K and V block (head_dim 128 and 64)
    (WIDE, 2, 200, 6, True), (WIDE, 1, 333, 8, False), (MID_GQA, 3, 77, 7, True),
    # the same against a cache long enough for several key splits (partials + merge)
    (MID_GQA, 1, 1100, 6, True), (WIDE, 1, 1100, 5, True),
    # 3..16 rows on models with several 16-column units per compute unit: whole-K QKV and gate/up with fused epilogues
    (ROWS, 1, 70, 9, True), (ROWS, 1, 33, 3, True), (ROWS, 2, 40, 8, True), (ROWS, 1, 10, 16, True), (ROWS_GQA, 1, 70, 9, True),
    (ROWS_GQA, 3, 20, 5, True), (ROWS_MANY, 1, 40, 7, True), (ROWS_MANY, 2, 300, 2, True)])
def test_prefill_then_verify_matches_full_recompute(c, B, n_prefix, q_len, packed):
    W, m, kv = setup(c, B, max(320, n_prefix + q_len + 8), seed=3, packed=packed)
    toks = synth.make_prompts(B, n_prefix + q_len, c["vocab"], seed=4)
    dtoks = torch.from_numpy(toks.astype(np.int32)).cuda()
    last = bs().prefill(m, kv, dtoks, n_prefix, want_logits=True)
    q = dtoks[:, n_prefix:n_prefix + q_len].contiguous()
    kvl = torch.full((B,), n_prefix, dtype=torch.int32, device="cuda")
    logits = bs().verify_forward(m, kv, q, kvl)
    torch.cuda.synchronize()
    tol = TOL[c["dtype"]]
    for b in range(B):
        ref = forward(c, W, toks[b], storage=c["dtype"])
        assert np.max(np.abs(last[b].cpu().numpy() - ref[n_prefix - 1])) < tol
        got = logits[b].cpu().numpy()
        assert got.shape == (q_len, c["vocab"])
        assert np.max(np.abs(got - ref[n_prefix:n_prefix + q_len])) < tol, np.max(np.abs(got - ref[n_prefix:n_prefix + q_len]))


# d_model / 16 units for O and down at least four fifths of the compute units: all four projections of a layer with fused
# epilogues and tiled activation planes between them (6 kernels per layer); two layers so that the down projection's planes and
# sums of squares feed a QKV projection.  The second shape has two units per compute unit for O and down, dealt unevenly.
WIDE_ROWS = synth.cfg(2, 3328, 26, 128, 6912, 512, dtype="bf16")
WIDE_ROWS2 = synth.cfg(1, 6656, 52, 128, 6912, 512, n_kv_heads=4, dtype="bf16")


@pytest.mark.parametrize("c,B,n_prefix,q_len,max_len", [
    (WIDE_ROWS, 1, 40, 9, 2100), (WIDE_ROWS, 1, 33, 3, 2100), (WIDE_ROWS, 2, 20, 8, 2100), (WIDE_ROWS, 1, 40, 9, 320),
    (WIDE_ROWS2, 1, 24, 7, 2100),
    # up to 16 rows per head group against a cache long enough for several key splits: the splits are combined inside the
    # attention kernel (head_dim 64 and 128, one and several query heads per kv head, more splits than rows and fewer)
    (MID, 1, 200, 9, 2100), (MID, 2, 150, 5, 2100), (MID_GQA, 2, 130, 3, 4200), (WIDE, 1, 100, 4, 1100), (MID, 1, 900, 16, 1100),
    (MID, 3, 40, 4, 8300)])
def test_up_to_16_rows_on_a_wide_model(c, B, n_prefix, q_len, max_len):
    """Verification passes of 3..16 rows where every projection takes the whole-K kernel with its consumer's work in the
    epilogue; with the short cache the attention has one key split and the O projection keeps the 16-row kernel."""
    Wd = synth.make_weights_device(c, 41, "cuda", std=0.02 * (4096 / c["d_model"]) ** 0.5)     # a hundred million weights: drawn on the GPU
    W = {k: v.float().cpu().numpy() for k, v in Wd.items()}
    m = bs().Model(c, Wd).pack(release_originals=True)
    kv = bs().KV(m, B, max_len)
    toks = synth.make_prompts(B, n_prefix + q_len, c["vocab"], seed=42)
    dtoks = torch.from_numpy(toks.astype(np.int32)).cuda()
    bs().prefill(m, kv, dtoks, n_prefix, want_logits=False)
    kvl = torch.full((B,), n_prefix, dtype=torch.int32, device="cuda")
    logits = bs().verify_forward(m, kv, dtoks[:, n_prefix:n_prefix + q_len].contiguous(), kvl)
    torch.cuda.synchronize()
    for b in range(B):
        ref = forward(c, W, toks[b], storage="bf16")
        err = np.max(np.abs(logits[b].cpu().numpy() - ref[n_prefix:n_prefix + q_len]))
        assert err < TOL["bf16"], (b, err)


# Prompt chunks with at least a whole round of items for the O and down projections, which then finish x, the planes and the
# sums of squares themselves: 160 whole items; 256 whole ones and 24 split along K; 44 row blocks (a last group of less than
# four), row-major weights and a ragged last block.
WIDE_RESID = synth.cfg(2, 2048, 16, 128, 1024, 512, n_kv_heads=4, dtype="bf16")


@pytest.mark.parametrize("B,n,packed", [(40, 128, True), (70, 128, True), (88, 127, False)])
def test_residual_projections_of_many_rows(B, n, packed):
    W, m, kv = setup(WIDE_RESID, B, n + 8, seed=61, packed=packed)
    toks = synth.make_prompts(B, n, 512, seed=62)
    last = bs().prefill(m, kv, torch.from_numpy(toks.astype(np.int32)).cuda(), n, want_logits=True)
    for b in (0, B // 2, B - 1):
        ref = forward(WIDE_RESID, W, toks[b], storage="bf16")
        assert np.max(np.abs(last[b].cpu().numpy() - ref[n - 1])) < TOL["bf16"], b


@pytest.mark.parametrize("B,q_len", [(1, 47), (3, 16), (7, 7), (4, 13), (1, 130)])
def test_f32_groups_of_eight_rows_under_wide_matrices(B, q_len):
    """fp32, 47 rows (groups of four) and 48..130 (of eight, whole and with rests) under gate/up, down and an LM head just above 4M
    elements, beside O and QKV below; columns that four does not divide, the LM head at an address that 16 does not divide."""
    c = synth.cfg(1, 512, 2, 32, 8200, 8201, n_kv_heads=1, dtype="f32")
    W = synth.make_weights(c, 29)
    dev = {k: torch.from_numpy(v).cuda() for k, v in W.items()}
    head = torch.empty(8201 * 512 + 1, device="cuda")[1:].view(8201, 512)
    dev["lm_head"] = head.copy_(dev["lm_head"])
    m = bs().Model(c, dev)
    kv = bs().KV(m, B, q_len)
    toks = synth.make_prompts(B, q_len, c["vocab"], seed=30)
    logits = bs().verify_forward(m, kv, torch.from_numpy(toks.astype(np.int32)).cuda(), torch.zeros(B, dtype=torch.int32, device="cuda"))
    for b in range(B):
        ref = forward(c, W, toks[b], storage="f32")
        assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["f32"], b


@pytest.mark.parametrize("B,n", [(1, 300), (33, 261)])
def test_prompt_pass_in_the_workspace_it_asks_for_and_in_less(B, n):
    """One chunk, and two chunks of 128 with a rest of 5; with room for 40 tokens only, chunks of 40 or more."""
    import ctypes as C
    W, m, kv = setup(PLAN_EDGE, B, n, seed=65, packed=True)
    toks = synth.make_prompts(B, n, 512, seed=66)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    full = bs().lib.bs_prefill_workspace_bytes(C.byref(m.cfg), B, n, n)
    less = m.forward_workspace_bytes(B, 40, n)
    assert less < full
    ref = {b: forward(PLAN_EDGE, W, toks[b], storage="bf16")[n - 1] for b in (0, B - 1)}
    for size in (full, less):
        kv.buf.zero_()
        ws = torch.zeros(size + 256, dtype=torch.uint8, device="cuda")
        ws[size:] = 77
        last = bs().prefill(m, kv, dt, n, want_logits=True, workspace=ws[:size])
        for b in ref:
            assert np.max(np.abs(last[b].cpu().numpy() - ref[b])) < TOL["bf16"], (size, b)
        assert bool((ws[size:] == 77).all())


# Rows at the edges of the plans: 96 rows leave O and down to the GEMM, from 97 on their items are split and finished by the fix-up
# kernel; one and two blocks of 256 rows, a ragged last row tile; columns that no tile of 192 or 256 divides, 17 and 43 stages.
PLAN_EDGE = synth.cfg(2, 544, 6, 64, 1376, 512, n_kv_heads=3, dtype="bf16")


@pytest.mark.parametrize("B,n,packed", [(1, 96, True), (1, 97, True), (3, 43, False), (1, 256, True), (1, 257, False), (4, 160, True)])
def test_rows_at_the_edges_of_the_many_row_plans(B, n, packed):
    W, m, kv = setup(PLAN_EDGE, B, n + 8, seed=63, packed=packed)
    toks = synth.make_prompts(B, n, 512, seed=64)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    kvl = torch.zeros(B, dtype=torch.int32, device="cuda")
    logits = bs().verify_forward(m, kv, dt, kvl)
    for b in {0, B - 1}:
        ref = forward(PLAN_EDGE, W, toks[b], storage="bf16")
        assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["bf16"], b


# Each way the split QKV and gate/up items are finished: a workgroup per unit with four or eight ranges in flight, or all units
# of an item together, for three and four weight tiles per wavefront.
@pytest.mark.parametrize("c,n", [
    (synth.cfg(1, 2048, 16, 64, 128, 512, n_kv_heads=8), 33),           # QKV 4 tiles 16 ranges, gate/up 4 tiles 16 ranges
    (synth.cfg(1, 1024, 35, 128, 128, 512, n_kv_heads=7), 33),          # QKV 4 tiles 4 ranges, gate/up 3 tiles 8 ranges
    (synth.cfg(1, 512, 4, 64, 2816, 512), 33),                          # QKV 3 tiles 4 ranges, gate/up 4 tiles 4 ranges
    (synth.cfg(1, 256, 15, 128, 1472, 512, n_kv_heads=5), 300),         # QKV and gate/up 3 tiles together
    (synth.cfg(1, 512, 4, 64, 6560, 512), 130),                         # gate/up 4 tiles together
    (synth.cfg(1, 2048, 41, 128, 128, 512, n_kv_heads=1), 520)])        # QKV 4 tiles together, 3 ranges
def test_every_way_of_finishing_split_items(c, n):
    W, m, kv = setup(c, 1, n, seed=67, packed=True)
    toks = synth.make_prompts(1, n, 512, seed=68)
    logits = bs().verify_forward(m, kv, torch.from_numpy(toks.astype(np.int32)).cuda(), torch.zeros(1, dtype=torch.int32, device="cuda"))
    ref = forward(c, W, toks[0], storage="bf16")
    assert np.max(np.abs(logits[0].cpu().numpy() - ref)) < TOL["bf16"]


@pytest.mark.parametrize("heads,hd", [(16, 128), (32, 64)])
def test_new_keys_of_many_rows_have_the_bits_of_the_written_rotation(heads, hd):
    """Rows of +-1, one weight per key column and a norm_eps of 3 make every projected value exact (x w / 2), so the keys of a prompt
    chunk of 4096 rows (whole items and split ones) must have the very bits of the rotation
        r0 = fma(v0, cos, -(v1 sin)),  r1 = fma(v1, cos, v0 sin),
    also the few that would round to the neighbouring bf16 value with the other product rounded first."""
    c = dict(synth.cfg(1, 256, heads, hd, 256, 512), norm_eps=3.0)
    d, n = c["d_model"], 4096
    g = torch.Generator(device="cuda").manual_seed(5)
    W = synth.make_weights_device(c, 5)
    W["embed"] = (torch.randint(0, 2, (512, d), generator=g, device="cuda") * 2 - 1).bfloat16()
    w = torch.randn(heads * hd, generator=g, device="cuda").bfloat16()
    W["l0.wk"].zero_()
    W["l0.wk"][torch.arange(heads * hd), torch.arange(heads * hd) % d] = w
    m = bs().Model(c, W)
    kv = bs().KV(m, 1, n)
    toks = torch.randint(0, 512, (1, n), generator=g, device="cuda", dtype=torch.int32)
    x = W["embed"][toks[0].long()].double()
    bs().prefill(m, kv, toks, n, want_logits=False)
    got = kv.buf.view(torch.bfloat16).view(2, heads, n, hd)[0].float()
    v = (x[:, torch.arange(heads * hd, device="cuda") % d] * w.double() / 2).view(n, heads, hd).transpose(0, 1)
    ang = torch.arange(n, device="cuda").double()[:, None] * c["rope_base"] ** (-2.0 * torch.arange(hd // 2, device="cuda").double() / hd)
    cs, sn = torch.cos(ang).float().double(), torch.sin(ang).float().double()
    v0, v1 = v[..., 0::2], v[..., 1::2]
    f32 = lambda t: t.float().double()                       # a product of two float32 values and its sum with a third are near enough exact in 64 bits
    key = lambda r0, r1: torch.stack((r0, r1), -1).flatten(-2).float().bfloat16().float()
    want = key(v0 * cs - f32(v1 * sn), v1 * cs + f32(v0 * sn))
    other = key(f32(v0 * cs) - v1 * sn, f32(v1 * cs) + v0 * sn)
    assert int((want != other).sum()) >= 20
    assert int((got != want).sum()) == 0


# Row-major weights whose d_model or d_ff is no multiple of 32: QKV, gate/up, O and down then take different schedules, and the
# sums of squares that one of them leaves are read by another.  O leaves 3, 2, 4 and 16 sums per row to a SwiGLU kernel, the
# second model's down projection leaves 2 to a RoPE kernel.
@pytest.mark.parametrize("c,B,n", [
    (synth.cfg(2, 512, 2, 64, 1000, 512), 2, 32), (synth.cfg(2, 272, 2, 64, 160, 512), 2, 33), (synth.cfg(2, 272, 4, 64, 1000, 512), 3, 40),
    (synth.cfg(2, 768, 12, 64, 3064, 512), 16, 128), (synth.cfg(1, 4096, 32, 128, 11000, 512), 32, 128)])
def test_schedules_meet_at_widths_that_32_does_not_divide(c, B, n):
    Wd = synth.make_weights_device(c, 91, "cuda", std=0.02 * (4096 / c["d_model"]) ** 0.5)
    W = {k: v.float().cpu().numpy() for k, v in Wd.items()}
    m = bs().Model(c, Wd)
    q_len = 17
    kv = bs().KV(m, B, n + q_len)
    toks = synth.make_prompts(B, n + q_len, c["vocab"], seed=92)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    last = bs().prefill(m, kv, dt, n, want_logits=True)
    kvl = torch.full((B,), n, dtype=torch.int32, device="cuda")
    logits = bs().verify_forward(m, kv, dt[:, n:].contiguous(), kvl)
    for b in {0, B // 2, B - 1}:
        ref = forward(c, W, toks[b], storage="bf16")
        assert np.max(np.abs(last[b].cpu().numpy() - ref[n - 1])) < TOL["bf16"], b
        assert np.max(np.abs(logits[b].cpu().numpy() - ref[n:])) < TOL["bf16"], b


# Prompt chunks large enough for the attention kernel whose wavefronts own different rows: head_dim 64 and 128, 64 and 128
# rows per workgroup, grouped queries, chunks with cached keys in front, last workgroups with a few rows only
PROMPT_128 = synth.cfg(2, 512, 16, 128, 256, 512, n_kv_heads=8, dtype="bf16")
PROMPT_64 = synth.cfg(2, 256, 36, 64, 256, 512, dtype="bf16")


@pytest.mark.parametrize("c,B,n", [(MID, 8, 256), (PROMPT_64, 4, 385), (PROMPT_128, 8, 465), (PROMPT_128, 8, 900), (PROMPT_128, 3, 1100), (WIDE, 8, 511)])
def test_prompt_attention(c, B, n):
    W, m, kv = setup(c, B, n + 8, seed=71, packed=True)
    toks = synth.make_prompts(B, n, c["vocab"], seed=72)
    last = bs().prefill(m, kv, torch.from_numpy(toks.astype(np.int32)).cuda(), n, want_logits=True)
    for b in (0, B - 1):
        ref = forward(c, W, toks[b], storage="bf16")
        assert np.max(np.abs(last[b].cpu().numpy() - ref[n - 1])) < TOL["bf16"], b


def test_prompt_attention_rows_and_a_sequence_left_out():
    """A pass of 256 rows per sequence behind 70 cached keys, every row's logits; sequence 3 has no room and is left out."""
    b, c, B, n_prefix, q_len = bs(), MID, 9, 70, 256
    max_len = n_prefix + q_len
    W, m, kv = setup(c, B, max_len, seed=73, packed=True)
    toks = synth.make_prompts(B, max_len, c["vocab"], seed=74)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    b.prefill(m, kv, dt, n_prefix)
    kvl = torch.full((B,), n_prefix, dtype=torch.int32, device="cuda")
    kvl[3] = n_prefix + 1
    ws = torch.zeros(m.forward_workspace_bytes(B, q_len, max_len), dtype=torch.uint8, device="cuda")
    logits = b.verify_forward(m, kv, dt[:, n_prefix:].contiguous(), kvl, workspace=ws)
    assert int(ws[:4].view(torch.int32).cpu()[0]) == 1
    for i in (0, 2, 4, 8):
        ref = forward(c, W, toks[i], storage="bf16")
        assert np.max(np.abs(logits[i].cpu().numpy() - ref[n_prefix:])) < TOL["bf16"], i


@pytest.mark.parametrize("hd,B,n_prefix,q_len,max_len", [(32, 1, 63, 1, 80), (128, 2, 60, 3, 80), (64, 3, 64, 5, 80), (72, 1, 700, 2, 1100), (24, 2, 129, 6, 1100)])
def test_f32_rows_and_splits(hd, B, n_prefix, q_len, max_len):
    """fp32: 1..18 rows in groups of four, attention rows in groups of two against one key split (the output itself) and several."""
    c = synth.cfg(2, 72, 2, hd, 264, 131, n_kv_heads=1, dtype="f32")
    W, m, kv = setup(c, B, max_len, seed=81)
    toks = synth.make_prompts(B, n_prefix + q_len, 131, seed=82)
    dtoks = torch.from_numpy(toks.astype(np.int32)).cuda()
    bs().prefill(m, kv, dtoks, n_prefix)
    kvl = torch.full((B,), n_prefix, dtype=torch.int32, device="cuda")
    logits = bs().verify_forward(m, kv, dtoks[:, n_prefix:].contiguous(), kvl)
    for b in range(B):
        ref = forward(c, W, toks[b], storage="f32")
        assert np.max(np.abs(logits[b].cpu().numpy() - ref[n_prefix:])) < TOL["f32"], b


# caches of more than 256 MB: weights and cached keys and values are asked for as non-temporal loads (head_dim 64 and 128, one
# and two row tiles per wavefront, the whole-K projections with one and two row tiles)
@pytest.mark.parametrize("c,B,n_prefix,q_len,max_len", [
    (MID, 1, 100, 5, 36000), (WIDE, 4, 45, 1, 36000), (WIDE, 4, 70, 6, 36000), (ROWS, 1, 33, 9, 16000), (ROWS, 2, 64, 10, 8000)])
def test_streamed_loads(c, B, n_prefix, q_len, max_len):
    W, m, kv = setup(c, B, max_len, seed=51, packed=True)
    assert kv.buf.numel() > 256 << 20
    toks = synth.make_prompts(B, n_prefix + q_len, c["vocab"], seed=52)
    dtoks = torch.from_numpy(toks.astype(np.int32)).cuda()
    bs().prefill(m, kv, dtoks, n_prefix)
    kvl = torch.full((B,), n_prefix, dtype=torch.int32, device="cuda")
    logits = bs().verify_forward(m, kv, dtoks[:, n_prefix:].contiguous(), kvl)
    for b in range(B):
        ref = forward(c, W, toks[b], storage="bf16")
        assert np.max(np.abs(logits[b].cpu().numpy() - ref[n_prefix:])) < TOL["bf16"], b


@pytest.mark.parametrize("B,n_prefix,q_len,max_len", [
    (1, 63, 2, 1100),      # three key splits of one 32-key block each: the two new keys fall into different splits
    (1, 64, 2, 1100), (2, 95, 1, 1100), (1, 1000, 2, 1100), (1, 31, 1, 2100), (1, 1, 1, 600), (2, 300, 1, 4200)])
def test_one_and_two_rows_on_a_narrow_model_with_a_long_cache(B, n_prefix, q_len, max_len):
    """Draft steps: one or two rows against a cache whose full length asks for several key splits, the new keys sitting
    at the edge of a 32-key block or of a split; the second pass reads what the first one put into the cache."""
    W, m, kv = setup(MID, B, max_len, seed=31, packed=True)
    toks = synth.make_prompts(B, n_prefix + 2 * q_len, MID["vocab"], seed=32)
    dtoks = torch.from_numpy(toks.astype(np.int32)).cuda()
    bs().prefill(m, kv, dtoks, n_prefix, want_logits=False)
    kvl = torch.full((B,), n_prefix, dtype=torch.int32, device="cuda")
    first = bs().verify_forward(m, kv, dtoks[:, n_prefix:n_prefix + q_len].contiguous(), kvl)
    kvl += q_len                                      # the second pass reads what the first one put into the cache
    second = bs().verify_forward(m, kv, dtoks[:, n_prefix + q_len:n_prefix + 2 * q_len].contiguous(), kvl)
    torch.cuda.synchronize()
    for b in range(B):
        ref = forward(MID, W, toks[b], storage="bf16")
        e1 = np.max(np.abs(first[b].cpu().numpy() - ref[n_prefix:n_prefix + q_len]))
        e2 = np.max(np.abs(second[b].cpu().numpy() - ref[n_prefix + q_len:n_prefix + 2 * q_len]))
        assert e1 < TOL["bf16"] and e2 < TOL["bf16"], (b, e1, e2)


# 512, 576 and 128 (sequence, head) pairs of 128: one split of the keys and several with a merge kernel; 192 pairs of 64: five splits
@pytest.mark.parametrize("heads,hd,B,n_prefix,q_len,max_len,splits", [
    (32, 128, 16, 1000, 9, 1024, 1), (32, 128, 16, 863, 1, 900, 1), (36, 128, 16, 831, 2, 1700, 2), (16, 128, 8, 1203, 5, 2400, 2),
    (12, 64, 16, 2047, 1, 4200, 5), (12, 64, 16, 1300, 3, 4200, 5)])
def test_key_splits_of_batches(heads, hd, B, n_prefix, q_len, max_len, splits):
    """Sequences of different lengths, their new keys at different places of the last block; the wavefronts of a split walk
    from one to eight blocks, requested ahead."""
    c = synth.cfg(1, 256, heads, hd, 256, 512, dtype="bf16")
    assert bs().attention_splits(c, B, q_len, max_len)[0] == splits and max_len // splits >= 768
    W, m, kv = setup(c, B, max_len, seed=71, packed=True)
    toks = synth.make_prompts(B, n_prefix + q_len, c["vocab"], seed=72)
    dtoks = torch.from_numpy(toks.astype(np.int32)).cuda()
    bs().prefill(m, kv, dtoks, n_prefix, want_logits=False)
    lens = [max(n_prefix - 41 * b, 30) for b in range(B)]
    q = torch.stack([dtoks[b, n:n + q_len] for b, n in enumerate(lens)]).contiguous()
    logits = bs().verify_forward(m, kv, q, torch.tensor(lens, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    for b in (0, 1, 6, B - 1):
        ref = forward(c, W, toks[b][:lens[b] + q_len], storage="bf16", last_rows=q_len)
        assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["bf16"], b


# Splits combined in the kernel by wavefronts that request their next block ahead: one query head per kv head and four, both head_dims
@pytest.mark.parametrize("heads,kv_heads,hd,q_len,max_len,splits,lens", [
    (32, 32, 128, 9, 8192, 8, [5003]), (32, 8, 128, 4, 8192, 8, [4100, 3001, None, 35]), (16, 16, 64, 2, 8192, 8, [4600, 31, 2000, None, 4599, 1, 700, 1025]),
    (32, 32, 128, 5, 4096, 4, [None, 3333])])
def test_splits_combined_in_the_kernel_with_blocks_requested_ahead(heads, kv_heads, hd, q_len, max_len, splits, lens):
    """Up to seven blocks a wavefront; None: a sequence left out."""
    c, B, n = synth.cfg(1, 256, heads, hd, 256, 512, n_kv_heads=kv_heads), len(lens), max(k or 0 for k in lens)
    assert bs().attention_splits(c, B, q_len, max_len) == (splits, splits, True) and max_len // splits >= 768
    W, m, kv = setup(c, B, max_len, seed=77, packed=True)
    toks = synth.make_prompts(B, n + q_len, c["vocab"], seed=78)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    bs().prefill(m, kv, dt, n, want_logits=False)
    kvl = torch.tensor([max_len if k is None else k for k in lens], dtype=torch.int32, device="cuda")
    q = torch.stack([dt[b, (k or 0):(k or 0) + q_len] for b, k in enumerate(lens)]).contiguous()
    ws = torch.zeros(m.forward_workspace_bytes(B, q_len, max_len), dtype=torch.uint8, device="cuda")
    logits = bs().verify_forward(m, kv, q, kvl, workspace=ws)
    assert int(ws[:4].view(torch.int32).cpu()[0]) == (1 if None in lens else 0)
    for b, k in enumerate(lens):
        if k is not None:
            ref = forward(c, W, toks[b][:k + q_len], storage="bf16", last_rows=q_len)
            assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["bf16"], b


# The workgroup of a split combines 256 / head_dim rows side by side: four, two and one of head_dim 64, two and one of 128, with rows left over in
# the last turn, splits without keys, and an even and an odd number of blocks a wavefront
@pytest.mark.parametrize("heads,kv_heads,hd,B,q_len,n,max_len,splits", [
    (8, 8, 64, 1, 16, 1001, 1100, 3), (8, 8, 64, 1, 7, 40, 1100, 3), (8, 2, 64, 1, 4, 640, 1100, 3), (8, 8, 64, 3, 5, 333, 1100, 3), (8, 8, 64, 1, 16, 650, 700, 2),
    (8, 8, 128, 1, 16, 1500, 2100, 5), (8, 8, 128, 1, 16, 129, 1600, 4), (8, 8, 128, 2, 5, 900, 1100, 3), (8, 2, 128, 1, 4, 1900, 2100, 5)])
def test_rows_combined_side_by_side(heads, kv_heads, hd, B, q_len, n, max_len, splits):
    c = synth.cfg(1, 256, heads, hd, 256, 512, n_kv_heads=kv_heads)
    assert bs().attention_splits(c, B, q_len, max_len) == (splits, splits, True)
    W, m, kv = setup(c, B, max_len, seed=81, packed=True)
    toks = synth.make_prompts(B, n + q_len, c["vocab"], seed=82)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    bs().prefill(m, kv, dt, n, want_logits=False)
    logits = bs().verify_forward(m, kv, dt[:, n:].contiguous(), torch.full((B,), n, dtype=torch.int32, device="cuda"))
    for b in range(B):
        ref = forward(c, W, toks[b], storage="bf16", last_rows=q_len)
        assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["bf16"] and off(logits[b], ref) < 5e-4, (b, off(logits[b], ref))


# A batch with sequences much longer than the others: these are cut into more parts, up to `most`, the others into `few`.
@pytest.mark.parametrize("c,B,q_len,max_len,few,most,long_len", [
    (synth.cfg(2, 256, 16, 128, 256, 512), 16, 5, 2304, 1, 4, 1500),                       # parts combined by the last workgroup
    (synth.cfg(1, 256, 32, 128, 256, 512, n_kv_heads=8), 24, 2, 4200, 1, 2, 1100),         # the same with grouped queries
    (synth.cfg(2, 256, 16, 128, 256, 512, n_kv_heads=8), 16, 3, 2304, 2, 4, 1500),         # merge kernel
    (synth.cfg(1, 3328, 26, 128, 6912, 512), 8, 3, 2304, 1, 5, 600),                       # tiled planes for the O projection
    (synth.cfg(1, 3328, 26, 128, 6912, 512), 4, 7, 2304, 2, 5, 600),
    (synth.cfg(2, 256, 16, 64, 256, 512), 40, 1, 2304, 1, 2, 900), (synth.cfg(1, 256, 12, 64, 256, 512), 32, 2, 8300, 2, 3, 900)])
def test_sequences_much_longer_than_the_others(c, B, q_len, max_len, few, most, long_len):
    """One long sequence; another one, with a sequence left out beside it; two long ones; all of one length: four passes in one workspace.
    With the poll limit at 1: these passes wait for nobody."""
    assert bs().attention_splits(c, B, q_len, max_len) == (few, most, False)
    W, m, kv = setup(c, B, max_len, seed=75, packed=True)
    toks = synth.make_prompts(B, long_len + q_len, c["vocab"], seed=76)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    bs().prefill(m, kv, dt, long_len, want_logits=False)
    short = [20 + 7 * b % 50 for b in range(B)]
    n = m.forward_workspace_bytes(B, q_len, max_len)
    ws = torch.zeros(n + 256, dtype=torch.uint8, device="cuda")
    ws[n:] = 77
    for longs, out in (([0], None), ([B - 1], 1), ([0, B // 2], None), (list(range(B)), None)):
        lens = [long_len if b in longs else short[b] for b in range(B)]
        bs().prefill(m, kv, dt, long_len, want_logits=False)
        kvl = torch.tensor(lens, dtype=torch.int32, device="cuda")
        if out is not None:
            kvl[out] = max_len - q_len + 1
        ws[:4] = 0
        q = torch.stack([dt[b, k:k + q_len] for b, k in enumerate(lens)]).contiguous()
        bs().step_poll_limit(1)
        try:
            logits = bs().verify_forward(m, kv, q, kvl, workspace=ws[:n])
        finally:
            bs().step_poll_limit(0)
        assert int(ws[:4].view(torch.int32).cpu()[0]) == (0 if out is None else 1)
        assert bool((ws[n:] == 77).all())
        for b in {longs[0], longs[-1], 2, B - 2}:
            ref = forward(c, W, toks[b][:lens[b] + q_len], storage="bf16", last_rows=q_len)
            assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["bf16"], (longs, b)


# one of the many-row projections in whole rounds of 256 items, finished in the GEMM, and the rest of the last round split along
# K: gate/up is 272 items of 128 columns per block of 256 rows
FFN_WIDE = synth.cfg(1, 1024, 2, 64, 34784, 512, dtype="bf16")


@pytest.mark.parametrize("c,B,n_prefix,q_len,max_len,splits", [
    # 17..32 rows on models with several 16-column units per compute unit: the whole-K projections with two row tiles
    (ROWS, 2, 30, 9, 47, 1), (ROWS, 1, 40, 17, 65, 1), (ROWS, 4, 8, 8, 24, 1), (ROWS_GQA, 3, 21, 6, 35, 1), (ROWS_MANY, 2, 25, 16, 49, 1), (ROWS_MANY, 7, 5, 3, 16, 1),
    # the same against one key split and against several, the O projection on tiled planes in all; with two splits a merge kernel
    # writes them and a wavefront walks up to three blocks
    (WIDE_ROWS, 2, 30, 9, 47, 1), (WIDE_ROWS, 4, 540, 5, 553, 1), (WIDE_ROWS, 4, 540, 5, 1100, 2), (WIDE_ROWS, 2, 540, 9, 2100, 4),
    (FFN_WIDE, 1, 220, 3, 231, 1), (FFN_WIDE, 1, 390, 40, 438, 1)])
def test_projections_with_epilogues_on_more_rows(c, B, n_prefix, q_len, max_len, splits):
    assert bs().attention_splits(c, B, q_len, max_len)[0] == splits
    W, m, kv = setup(c, B, max_len, seed=61, packed=True)
    toks = synth.make_prompts(B, n_prefix + q_len, c["vocab"], seed=62)
    dtoks = torch.from_numpy(toks.astype(np.int32)).cuda()
    last = bs().prefill(m, kv, dtoks, n_prefix, want_logits=True)
    kvl = torch.full((B,), n_prefix, dtype=torch.int32, device="cuda")
    logits = bs().verify_forward(m, kv, dtoks[:, n_prefix:].contiguous(), kvl)
    torch.cuda.synchronize()
    for b in range(B):
        ref = forward(c, W, toks[b], storage="bf16", last_rows=q_len + 1)
        assert np.max(np.abs(last[b].cpu().numpy() - ref[0])) < TOL["bf16"], b
        assert np.max(np.abs(logits[b].cpu().numpy() - ref[1:])) < TOL["bf16"], b


@pytest.mark.parametrize("c,B,n_prefix,q_len", [(MID_GQA, 2, 140, 9), (ODD_BF16, 1, 33, 5), (WIDE, 1, 20, 16)])
def test_packed_weights_give_bit_identical_logits(c, B, n_prefix, q_len):
    """The tiled copy only changes where each weight is read from, not the order of the arithmetic."""
    outs = []
    for packed in (False, True):
        W, m, kv = setup(c, B, 200, seed=11, packed=packed)
        toks = synth.make_prompts(B, n_prefix + q_len, c["vocab"], seed=12)
        dtoks = torch.from_numpy(toks.astype(np.int32)).cuda()
        last = bs().prefill(m, kv, dtoks, n_prefix, want_logits=True)
        kvl = torch.full((B,), n_prefix, dtype=torch.int32, device="cuda")
        logits = bs().verify_forward(m, kv, dtoks[:, n_prefix:n_prefix + q_len].contiguous(), kvl)
        torch.cuda.synchronize()
        outs.append((last.cpu().numpy().copy(), logits.cpu().numpy().copy()))
    assert np.array_equal(outs[0][0], outs[1][0])
    assert np.array_equal(outs[0][1], outs[1][1])


def test_pack_errors():
    b = bs()
    m = b.Model.from_numpy(synth.TINY_TARGET, synth.make_weights(synth.TINY_TARGET, 1))
    assert m.packed_bytes() == 0                      # fp32 models are not packed
    with pytest.raises(RuntimeError):
        m.pack()
    W, m2, _ = setup(MID, 1, 64, seed=2)
    n = m2.packed_bytes()
    assert n >= sum(v.size for k, v in W.items() if not k.endswith("norm") and k != "embed") * 2
    small = torch.empty(n - 256, dtype=torch.uint8, device="cuda")
    assert b.lib.bs_model_pack(m2.h, b.ptr(small), small.numel(), None) == b.BS_EWORKSPACE
    m2.pack()
    again = torch.empty(n, dtype=torch.uint8, device="cuda")
    assert b.lib.bs_model_pack(m2.h, b.ptr(again), n, None) == b.BS_ESTATE


def test_ragged_cache_lengths_and_logit_rows():
    c = MID_GQA
    B, max_len = 3, 160
    W, m, kv = setup(c, B, max_len, seed=5)
    lens = [40, 97, 1]
    toks = synth.make_prompts(B, 120, c["vocab"], seed=6)
    dtoks = torch.from_numpy(toks.astype(np.int32)).cuda()
    # fill each sequence's cache to its own length with single-sequence-valid chunks: prefill to the max, the
    # extra positions of shorter sequences are simply overwritten later
    bs().prefill(m, kv, dtoks, max(lens))
    q_len = 4
    q = torch.stack([dtoks[b, lens[b]:lens[b] + q_len] for b in range(B)]).contiguous()
    kvl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    logits = bs().verify_forward(m, kv, q, kvl, logit_rows=2)
    torch.cuda.synchronize()
    for b in range(B):
        ref = forward(c, W, toks[b, :lens[b] + q_len], storage="bf16")
        assert np.max(np.abs(logits[b].cpu().numpy() - ref[lens[b] + q_len - 2:lens[b] + q_len])) < TOL["bf16"]


def test_one_pass_over_gamma_plus_one_equals_token_by_token():
    # "verify in parallel" (App. A): scoring gamma+1 positions at once must equal gamma+1 single-token passes
    c = MID
    W, m, kv = setup(c, 2, 64, seed=7)
    kv2 = bs().KV(m, 2, 64)
    toks = torch.from_numpy(synth.make_prompts(2, 30, c["vocab"], seed=8).astype(np.int32)).cuda()
    bs().prefill(m, kv, toks, 21); bs().prefill(m, kv2, toks, 21)
    kvl = torch.full((2,), 21, dtype=torch.int32, device="cuda")
    a = bs().verify_forward(m, kv, toks[:, 21:30].contiguous(), kvl)
    rows = []
    for j in range(9):
        rows.append(bs().verify_forward(m, kv2, toks[:, 21 + j:22 + j].contiguous(), kvl + j))
    b = torch.cat(rows, dim=1)
    assert torch.max(torch.abs(a - b)).item() < 2e-3
    assert torch.equal(kv.buf.view(torch.int16)[: kv.buf.numel() // 2], kv2.buf.view(torch.int16)[: kv2.buf.numel() // 2]) or \
        torch.max(torch.abs(kv.buf.view(torch.bfloat16).float() - kv2.buf.view(torch.bfloat16).float())).item() < 0.05


def test_cache_overflow_skips_sequence_and_sets_status():
    c = synth.TINY_DRAFT
    W, m, kv = setup(c, 2, 16, seed=9)
    toks = torch.from_numpy(synth.make_prompts(2, 16, c["vocab"], seed=10).astype(np.int32)).cuda()
    bs().prefill(m, kv, toks, 10)
    before = kv.buf.clone()
    ws = torch.zeros(m.forward_workspace_bytes(2, 4, 16), dtype=torch.uint8, device="cuda")
    kvl = torch.tensor([10, 14], dtype=torch.int32, device="cuda")           # sequence 1 would need 18 > 16
    logits = bs().verify_forward(m, kv, toks[:, 10:14].contiguous(), kvl, workspace=ws)
    torch.cuda.synchronize()
    assert int(ws[:4].view(torch.int32)[0].item()) & 1
    ref = forward(c, W, toks[0, :14].cpu().numpy(), storage="f32")
    assert np.max(np.abs(logits[0].cpu().numpy() - ref[10:14])) < TOL["f32"]
    # nothing of sequence 1 was written to the cache
    es, L = 4, c["n_layers"]
    per_seq = c["n_kv_heads"] * 32 * c["head_dim"] * es          # cache rows are padded to a multiple of 32
    cur = kv.buf.view(L, 2, 2, per_seq); old = before.view(L, 2, 2, per_seq)
    assert torch.equal(cur[:, :, 1], old[:, :, 1]) and not torch.equal(cur[:, :, 0], old[:, :, 0])


def test_argument_errors():
    b = bs()
    c = synth.TINY_DRAFT
    W, m, kv = setup(c, 1, 16, seed=11)
    toks = torch.zeros(1, 4, dtype=torch.int32, device="cuda"); kvl = torch.zeros(1, dtype=torch.int32, device="cuda")
    small = torch.zeros(512, dtype=torch.uint8, device="cuda")
    with pytest.raises(b.BanditSpecError) as e:
        b.verify_forward(m, kv, toks, kvl, workspace=small)
    assert e.value.code == -4
    other = b.KV(b.Model.from_numpy(synth.TINY_TARGET, synth.make_weights(synth.TINY_TARGET, 1)), 1, 16)
    with pytest.raises(b.BanditSpecError) as e:
        b.verify_forward(m, other, toks, kvl)
    assert e.value.code == -5
    with pytest.raises(b.BanditSpecError) as e:
        b.verify_forward(m, kv, torch.zeros(1, 17, dtype=torch.int32, device="cuda"), kvl)
    assert e.value.code == -2


def test_per_launch_timing_refuses_a_stream_capture_and_counts_eager_launches():
    """The measurement hook: with the record on, eager launches of the bf16 GEMM are counted, a pass that is being
    captured into a graph is refused (BS_ESTATE, nothing launched), and switching the record off drops it."""
    b = bs()
    W, m, kv = setup(MID, 1, 64, seed=5, packed=True)
    toks = torch.zeros(1, 9, dtype=torch.int32, device="cuda"); kvl = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(m.forward_workspace_bytes(1, 9, 64), dtype=torch.uint8, device="cuda")
    lg = torch.empty(1, 9, MID["vocab"], dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        b.verify_forward(m, kv, toks, kvl, workspace=ws, logits=lg)
        side.synchronize()
        b.profile_enable(True)
        try:
            b.verify_forward(m, kv, toks, kvl, workspace=ws, logits=lg)
            side.synchronize()
            ms, by, n = b.profile_collect(0)
            assert n >= 4 * MID["n_layers"] and ms > 0 and by > 0
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=side):
                with pytest.raises(b.BanditSpecError) as e:
                    b.verify_forward(m, kv, toks, kvl, workspace=ws, logits=lg)
            assert e.value.code == -5
        finally:
            b.profile_enable(False)
        assert b.profile_collect(0)[2] == 0
        b.verify_forward(m, kv, toks, kvl, workspace=ws, logits=lg)          # and the library still works
        side.synchronize()


def test_resident_step_gives_up_after_its_poll_limit_and_recovers():
    """One row of a small packed bf16 model runs as one resident kernel whose workgroups poll for each other's outputs.
    With the poll limit at 1 every wait runs out at once: the launch must still end (no workgroup waits for ever), report
    it in bit 16 of the status word, and the next pass with the default limit must be right again."""
    b = bs()
    c = MID
    W, m, kv = setup(c, 1, 96, seed=21, packed=True)
    n_prefix = 40
    toks = synth.make_prompts(1, n_prefix + 2, c["vocab"], 22)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    b.prefill(m, kv, dt, n_prefix)
    kvl = torch.full((1,), n_prefix, dtype=torch.int32, device="cuda")
    ws = torch.zeros(m.forward_workspace_bytes(1, 2, 96), dtype=torch.uint8, device="cuda")     # the status word starts at 0
    lg = torch.empty(1, 2, c["vocab"], dtype=torch.float32, device="cuda")
    q = dt[:, n_prefix:n_prefix + 2].contiguous()
    try:
        b.step_poll_limit(1)
        b.verify_forward(m, kv, q, kvl, workspace=ws, logits=lg)
        torch.cuda.synchronize()                      # returns: the launch ended
        assert int(ws[:4].view(torch.int32).cpu()[0]) & 16
    finally:
        b.step_poll_limit(0)
    ws[:4].zero_()                                    # the word is only ever OR-ed into
    b.verify_forward(m, kv, q, kvl, workspace=ws, logits=lg)
    torch.cuda.synchronize()
    assert int(ws[:4].view(torch.int32).cpu()[0]) & 16 == 0
    ref = forward(c, W, toks[0], storage="bf16")
    assert np.max(np.abs(lg[0].cpu().numpy() - ref[n_prefix:n_prefix + 2])) < TOL["bf16"]


def test_fused_and_unfused_schedules_agree_closely():
    """The same wide model packed (five kernels per layer: whole-K projections with fused epilogues, key splits combined in the
    attention kernel) and unpacked (16-row GEMM with split-K, consumer kernels, merge kernel): the two schedules share no
    projection kernel and differ only in the order of fp32 additions, so their logits agree far more closely than either has to
    agree with the fp64 oracle -- a wrong rotation angle, sum-of-squares piece or residual column in one of them shows here."""
    c, B, n_prefix, q_len, max_len = WIDE_ROWS, 2, 30, 7, 2100
    Wd = synth.make_weights_device(c, 51, "cuda", std=0.02 * (4096 / c["d_model"]) ** 0.5)
    toks = synth.make_prompts(B, n_prefix + q_len, c["vocab"], seed=52)
    dtoks = torch.from_numpy(toks.astype(np.int32)).cuda()
    outs = []
    for packed in (False, True):
        m = bs().Model(c, dict(Wd))
        if packed:
            m.pack(release_originals=False)
        kv = bs().KV(m, B, max_len)
        bs().prefill(m, kv, dtoks, n_prefix, want_logits=False)
        kvl = torch.full((B,), n_prefix, dtype=torch.int32, device="cuda")
        first = bs().verify_forward(m, kv, dtoks[:, n_prefix:n_prefix + 3].contiguous(), kvl).cpu().numpy()
        kvl += 3                                       # the second pass reads the cache rows the first one's epilogue wrote
        second = bs().verify_forward(m, kv, dtoks[:, n_prefix + 3:n_prefix + q_len].contiguous(), kvl).cpu().numpy()
        torch.cuda.synchronize()
        outs.append((first, second))
    for a, b_ in zip(outs[0], outs[1]):
        scale = float(np.max(np.abs(a)))
        assert scale > 0.1
        # measured: 1.6e-4 .. 2.8e-4 on logits of magnitude 5..6 (a k or v that rounds to the neighbouring bf16 value in the cache)
        assert np.max(np.abs(a - b_)) < 5e-4 * max(scale, 1.0), (np.max(np.abs(a - b_)), scale)


def test_key_splits_combined_in_the_attention_kernel_with_a_sequence_left_out_and_with_no_patience():
    """Three sequences of five rows against a long cache (several key splits, combined inside the attention kernel through
    exchange cells): sequence 1 has no room and is left out, its workgroups hand nothing over and nobody waits for them;
    the others' logits are right, bit 0 of the status word is set, bit 16 is not.  With a poll limit of one a pass gives up
    (the workgroups of the last splits hold no keys and poll while the others still walk theirs: bit 16, no hang), and the next pass
    with the default limit is right again."""
    b = bs()
    c = MID
    max_len, n_prefix, q_len = 8300, 600, 5
    assert b.attention_splits(c, 3, q_len, max_len) == (17, 17, True)
    W, m, kv = setup(c, 3, max_len, seed=27, packed=True)
    toks = synth.make_prompts(3, n_prefix + q_len, c["vocab"], 28)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    b.prefill(m, kv, dt, n_prefix)
    ws = torch.zeros(m.forward_workspace_bytes(3, q_len, max_len), dtype=torch.uint8, device="cuda")
    kvl = torch.tensor([n_prefix, max_len - 2, n_prefix], dtype=torch.int32, device="cuda")
    q = dt[:, n_prefix:n_prefix + q_len].contiguous()

    def check(expect_bit16):
        lg = b.verify_forward(m, kv, q, kvl, workspace=ws)
        torch.cuda.synchronize()
        status = int(ws[:4].view(torch.int32).cpu()[0])
        assert status & 1 and bool(status & 16) == expect_bit16, status
        if not expect_bit16:
            for i in (0, 2):
                ref = forward(c, W, toks[i], storage="bf16")
                assert np.max(np.abs(lg[i].cpu().numpy() - ref[n_prefix:n_prefix + q_len])) < TOL["bf16"], i

    check(False)
    b.step_poll_limit(1)
    try:
        check(True)
    finally:
        b.step_poll_limit(0)
    ws.zero_()
    check(False)


@pytest.mark.parametrize("c,B,q_len", [(MID, 4, 5), (MID, 1, 17), (MID, 2, 16)])
def test_passes_of_17_to_32_rows_wait_for_nobody(c, B, q_len):
    """Such passes may run beside others on other streams: with the poll limit at 1, where every wait between workgroups runs
    out at once, they give the right logits against several key splits, and report nothing."""
    b, n_prefix, max_len = bs(), 100, 2100
    assert b.attention_splits(c, B, q_len, max_len) == (5, 5, False)
    W, m, kv = setup(c, B, max_len, seed=27, packed=True)
    toks = synth.make_prompts(B, n_prefix + q_len, c["vocab"], 28)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    b.prefill(m, kv, dt, n_prefix)
    kvl = torch.full((B,), n_prefix, dtype=torch.int32, device="cuda")
    ws = torch.zeros(m.forward_workspace_bytes(B, q_len, max_len), dtype=torch.uint8, device="cuda")
    b.step_poll_limit(1)
    try:
        lg = b.verify_forward(m, kv, dt[:, n_prefix:].contiguous(), kvl, workspace=ws)
        torch.cuda.synchronize()
    finally:
        b.step_poll_limit(0)
    assert int(ws[:4].view(torch.int32).cpu()[0]) == 0
    for i in range(B):
        ref = forward(c, W, toks[i], storage="bf16")
        assert np.max(np.abs(lg[i].cpu().numpy() - ref[n_prefix:])) < TOL["bf16"], i


def test_resident_step_with_a_sequence_left_out():
    """Two sequences, one row each, on a small packed bf16 model (the resident one-launch pass): sequence 1 has no room
    in its cache and is left out.  Its attention units have nothing to do in any layer and must still keep in step with
    the others; sequence 0's logits are right, bit 0 of the status word is set and bit 16 is not."""
    b = bs()
    c = MID
    max_len = 48
    W, m, kv = setup(c, 2, max_len, seed=23, packed=True)
    toks = synth.make_prompts(2, 40, c["vocab"], 24)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    b.prefill(m, kv, dt, 30)
    ws = torch.zeros(m.forward_workspace_bytes(2, 1, max_len), dtype=torch.uint8, device="cuda")
    kvl = torch.tensor([30, max_len], dtype=torch.int32, device="cuda")       # sequence 1: position 48 of 48
    for step in range(3):                             # several passes in a row: every layer of every pass hands over in step
        lg = b.verify_forward(m, kv, dt[:, 30 + step:31 + step].contiguous(), kvl, workspace=ws)
        torch.cuda.synchronize()
        status = int(ws[:4].view(torch.int32).cpu()[0])
        assert status & 1 and not status & 16, status
        ref = forward(c, W, toks[0, :31 + step], storage="bf16")
        assert np.max(np.abs(lg[0, 0].cpu().numpy() - ref[30 + step])) < TOL["bf16"], step
        kvl[0] += 1


# Passes of 33 rows and more: tiled activation planes (rows rounded up to 16) in the layers, and in front of the LM head where it has that many rows
# Measured: at most 7.7e-4 (keys and values that round the other way in early tokens), as a rule 1e-4.
@pytest.mark.parametrize("c", [dict(MID_GQA, n_layers=2), synth.cfg(2, 96, 2, 64, 168, 1000, dtype="bf16")], ids=["tiled", "d_ff of 168: row by row"])
@pytest.mark.parametrize("B,q_len,rows", [(11, 3, 3), (9, 5, 4), (9, 5, 1), (35, 1, 1), (3, 16, 16), (29, 9, 9)])
def test_planes_of_33_rows_and_more(c, B, q_len, rows):
    n, max_len = 20, 40
    W, m, kv = setup(c, B, max_len, seed=91, packed=c["d_ff"] % 32 == 0)
    toks = synth.make_prompts(B, n + q_len, c["vocab"], 92)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    bs().prefill(m, kv, dt, n)
    logits = bs().verify_forward(m, kv, dt[:, n:].contiguous(), torch.full((B,), n, dtype=torch.int32, device="cuda"), rows)
    for b in {0, 1, B // 2, B - 1}:
        ref = forward(c, W, toks[b], storage="bf16", last_rows=rows)
        assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["bf16"] and off(logits[b], ref) < 1.2e-3, (b, off(logits[b], ref))


# 129 rows and more: blocks of up to 128 rows, wavefronts in one row (5 to 8 row tiles) or two (6, 8); columns beside 384 and 512, a last block that is not full
@pytest.mark.parametrize("c", [synth.cfg(1, 1024, 16, 64, 2816, 544, n_kv_heads=4), synth.cfg(1, 736, 9, 64, 1472, 1030, n_kv_heads=3),
                               synth.cfg(1, 2048, 16, 128, 6912, 512)], ids=["1024", "736", "2048"])
@pytest.mark.parametrize("B,n", [(1, 129), (3, 53), (1, 191), (1, 225), (1, 257), (1, 384), (2, 321), (9, 128), (4, 1000)])
def test_blocks_of_rows_from_129_rows_on(c, B, n):
    W, m, kv = setup(c, B, n + 8, seed=95, packed=True)
    toks = synth.make_prompts(B, n, c["vocab"], seed=96)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    rows = min(n, 40)                                  # several logit rows a sequence: the LM head has many rows as well
    logits = bs().verify_forward(m, kv, dt, torch.zeros(B, dtype=torch.int32, device="cuda"), rows)
    for b in {0, B - 1}:
        ref = forward(c, W, toks[b], storage="bf16", last_rows=rows)
        assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["bf16"] and off(logits[b], ref) < 5e-4, (b, off(logits[b], ref))      # measured: at most 1.3e-4


# 33 to 256 rows of a model whose weights are more than the memory-side cache holds: eight wavefronts in a row with two, three or four weight tiles
# each, 3 to 8 row tiles full and not, one block of rows and two; the tiled copy of the weights and the weights as they are
@pytest.fixture(scope="module")
def past_cache():
    c = synth.cfg(1, 1024, 16, 64, 28672, 70001, n_kv_heads=4)
    W = synth.make_weights(c, 97, 0.04)
    return c, {k: (v if k.endswith("norm") else synth.to_bf16_grid(v)) for k, v in W.items()}


@pytest.mark.parametrize("B,n,packed", [(1, 33, True), (3, 16, True), (1, 49, False), (2, 40, True), (9, 9, True), (1, 96, True), (1, 97, False),
                                        (1, 128, True), (3, 43, True), (1, 160, True), (2, 128, False), (1, 257, True), (3, 100, False)])
def test_rows_of_a_model_that_streams(past_cache, B, n, packed):
    c, W = past_cache
    m = bs().Model.from_numpy(c, W)
    if packed:
        m.pack(release_originals=True)
    kv = bs().KV(m, B, n + 8)
    toks = synth.make_prompts(B, n, c["vocab"], seed=98)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    rows = min(n, 40)
    logits = bs().verify_forward(m, kv, dt, torch.zeros(B, dtype=torch.int32, device="cuda"), rows)
    for b in {0, B - 1}:
        ref = forward(c, W, toks[b], storage="bf16", last_rows=rows)
        assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["bf16"] and off(logits[b], ref) < 5e-4, (b, off(logits[b], ref))      # measured: at most 1.3e-4


# fp32 projections with the work around them: rows and columns that four and eight do not divide, a vocabulary of an odd size, an embedding, a final norm and an
# LM head at addresses that 16 does not divide, trailing logit rows, a sequence left out; short caches and one in several splits
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("c,B,n,q_len,rows,max_len", [
    (synth.cfg(2, 72, 3, 24, 104, 131, dtype="f32"), 1, 9, 1, 1, 11), (synth.cfg(2, 72, 3, 24, 104, 131, dtype="f32"), 3, 61, 3, 2, 64),
    (synth.cfg(1, 264, 6, 40, 520, 999, n_kv_heads=2, dtype="f32"), 5, 130, 1, 1, 140), (synth.cfg(1, 264, 6, 40, 520, 999, n_kv_heads=2, dtype="f32"), 2, 500, 9, 9, 512),
    (synth.cfg(1, 64, 2, 128, 96, 300, dtype="f32"), 3, 520, 6, 6, 530)])
def test_f32_projections_with_the_work_around_them(c, B, n, q_len, rows, max_len, shift):
    W = synth.make_weights(c, 33)
    dev = {k: torch.from_numpy(v).cuda() for k, v in W.items()}
    for k in ("embed", "lm_head", "final_norm"):
        dev[k] = torch.empty(dev[k].numel() + shift, device="cuda")[shift:].view(dev[k].shape).copy_(dev[k])
    m = bs().Model(c, dev)
    kv = bs().KV(m, B, max_len)
    toks = synth.make_prompts(B, n + q_len, c["vocab"], seed=34)
    dt = torch.from_numpy(toks.astype(np.int32)).cuda()
    bs().prefill(m, kv, dt, n)
    kvl = torch.full((B,), n, dtype=torch.int32, device="cuda")
    if B > 2:
        kvl[1] = max_len                               # no room: left out
    logits = bs().verify_forward(m, kv, dt[:, n:].contiguous(), kvl, rows)
    for b in range(B):
        if B <= 2 or b != 1:
            ref = forward(c, W, toks[b], storage="f32", last_rows=rows)
            assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["f32"], b


@pytest.mark.parametrize("B,q_len", [(1, 47), (3, 16), (1, 130)])
def test_f32_kernel_per_step_under_wide_feed_forward_matrices(B, q_len):
    """48 rows and more of a model whose feed-forward matrices have more than 12 million elements each."""
    c = synth.cfg(1, 1024, 2, 32, 11800, 8201, n_kv_heads=1, dtype="f32")
    W = synth.make_weights(c, 35)
    dev = {k: torch.from_numpy(v).cuda() for k, v in W.items()}
    dev["lm_head"] = torch.empty(8201 * 1024 + 1, device="cuda")[1:].view(8201, 1024).copy_(dev["lm_head"])
    m = bs().Model(c, dev)
    kv = bs().KV(m, B, q_len)
    toks = synth.make_prompts(B, q_len, c["vocab"], seed=36)
    logits = bs().verify_forward(m, kv, torch.from_numpy(toks.astype(np.int32)).cuda(), torch.zeros(B, dtype=torch.int32, device="cuda"))
    for b in range(B):
        ref = forward(c, W, toks[b], storage="f32")
        assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["f32"], b


# QKV: the number of ranges of K decides how the sums round, so two passes that are cut into as many leave the same bits in the first layer's cache,
# whatever blocks of rows and arrangement of wavefronts each of them takes: here one of up to 128 rows or fewer blocks, and one of more
@pytest.mark.parametrize("c,n,fewer", [
    (synth.cfg(1, 4096, 32, 128, 512, 512), 240, 140), (synth.cfg(1, 4096, 32, 128, 512, 512), 490, 400),
    (synth.cfg(1, 4096, 32, 128, 512, 512, n_kv_heads=8), 240, 140), (synth.cfg(1, 768, 12, 64, 512, 512), 240, 100),
    (synth.cfg(1, 768, 12, 64, 512, 512), 1000, 800), (synth.cfg(1, 1024, 8, 128, 512, 512), 240, 100), (synth.cfg(1, 1024, 8, 128, 512, 512), 640, 760)],
    ids=["4096, 240", "4096, 490", "4096 grouped, 240", "768, 240", "768, 1000", "1024, 240", "1024, 640"])
def test_keys_and_values_of_a_pass_have_the_sums_of_a_shorter_one(c, n, fewer):
    m = bs().Model(c, synth.make_weights_device(c, 41, "cuda")).pack(release_originals=True)
    toks = torch.from_numpy(synth.make_prompts(1, max(n, fewer), c["vocab"], seed=42).astype(np.int32)).cuda()
    caches = []
    for rows in (n, fewer):
        kv = bs().KV(m, 1, 1024)
        bs().verify_forward(m, kv, toks[:, :rows].contiguous(), torch.zeros(1, dtype=torch.int32, device="cuda"), 1)
        k, v = kv.buf.view(torch.int16).view(2, c["n_kv_heads"], 1024, c["head_dim"])
        # values: blocks of 32 keys, key 16t + 4q + e of a block at slot 8q + 4t + e
        v = v.reshape(c["n_kv_heads"], 32, c["head_dim"], 4, 2, 4).permute(0, 1, 4, 3, 5, 2).reshape(c["n_kv_heads"], 1024, c["head_dim"])
        caches.append((k[:, :min(n, fewer)], v[:, :min(n, fewer)]))
    for a, b in zip(*caches):
        assert a.ne(0).any() and torch.equal(a, b), int(a.ne(b).sum())


def test_a_row_of_wavefronts_leaves_the_sums_of_squares_of_two():
    """4096 rows take O and down in whole items of 512 columns (eight wavefronts in a row), 2048 rows in items of 256 (four by two): the rows' sums of
    squares, and with them the second layer's keys and values, have the same bits."""
    c = synth.cfg(2, 4096, 32, 64, 2048, 512)
    m = bs().Model(c, synth.make_weights_device(c, 43, "cuda")).pack(release_originals=True)
    toks = torch.from_numpy(synth.make_prompts(4, 1024, c["vocab"], seed=44).astype(np.int32)).cuda()
    caches = []
    for B in (4, 2):
        kv = bs().KV(m, B, 1024)
        bs().verify_forward(m, kv, toks[:B].contiguous(), torch.zeros(B, dtype=torch.int32, device="cuda"), 1)
        caches.append(kv.buf.view(torch.int16).view(2, 2, B, -1)[:, :, :2])
    assert caches[0].ne(0).any() and torch.equal(*caches), int(caches[0].ne(caches[1]).sum())


def test_workspace_of_every_length_is_planned_in_little_time():
    """A workspace query plans the pass of every length up to its limit: 4096 lengths of the 7B shape in under 2 ms of host work."""
    import ctypes
    import time
    c = synth.LLAMA7B_TARGET
    cfg = bs().ModelCfg(c["n_layers"], c["d_model"], c["n_heads"], c["n_kv_heads"], c["head_dim"], c["d_ff"], c["vocab"], 1, c["rope_base"], c["norm_eps"])
    best = 1.0
    for _ in range(10):
        t = time.perf_counter()
        assert bs().lib.bs_forward_workspace_bytes(ctypes.byref(cfg), 1, 4096, 4352) > 0
        best = min(best, time.perf_counter() - t)
    assert best < 2e-3, best


@pytest.mark.parametrize("c,B,q_len,rows", [(synth.cfg(1, 1024, 2, 32, 96, 24001, dtype="f32"), 8, 32, 32), (synth.cfg(1, 1024, 2, 32, 96, 24001, dtype="f32"), 8, 33, 31),
                                            (synth.cfg(1, 1024, 64, 128, 256, 999, dtype="f32"), 2, 256, 3)],
                         ids=["head by itself", "head with the norm", "layers by themselves"])
def test_f32_matrices_of_more_than_24_million_elements(c, B, q_len, rows):
    """Many rows leave the fused projections where a matrix is large: an LM head from 256 logit rows on, a layer from 512 rows on."""
    W = synth.make_weights(c, 37)
    m = bs().Model(c, {k: torch.from_numpy(v).cuda() for k, v in W.items()})
    kv = bs().KV(m, B, q_len)
    toks = synth.make_prompts(B, q_len, c["vocab"], seed=38)
    logits = bs().verify_forward(m, kv, torch.from_numpy(toks.astype(np.int32)).cuda(), torch.zeros(B, dtype=torch.int32, device="cuda"), rows)
    for b in (0, B - 1):
        ref = forward(c, W, toks[b], storage="f32", last_rows=rows)
        assert np.max(np.abs(logits[b].cpu().numpy() - ref)) < TOL["f32"], b
