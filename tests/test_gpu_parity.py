"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by
element at sizes the oracle finishes in seconds (several tiles, ragged tails,
both activation-tile variants, vocabularies that are not a multiple of 4)."""
import numpy as np
import pytest
import torch

import mrp_inputs as mi
import paper_2605_18817_amd as mrp
from harness import (Problem, compare_chain, dev_bits, gpu_chain, io_to_host, lm_head_on_tiles, oracle_chain,
                     small_tile_features)

pytestmark = pytest.mark.gpu


def _free_run(cfg, rcfg, gamma="ones", share_heads=False, seqs=None, max_exempt=0):
    prob = Problem(cfg, gamma=gamma, share_heads=share_heads)
    try:
        z0 = mi.logits0(cfg)
        h = mi.hidden(cfg)
        z_d = torch.from_numpy(z0).cuda()
        io, hrun_d = gpu_chain(prob, cfg.B, cfg.K, z_d, h, rcfg)
        g = io_to_host(io)
        seqs = list(range(cfg.B)) if seqs is None else seqs
        rows = np.concatenate([np.arange(b * cfg.L, (b + 1) * cfg.L) for b in seqs])
        o = oracle_chain(prob, z0[rows], mi.bf16_bits_to_f64(h[rows]), rcfg, cfg.K)
        plain = oracle_chain(prob, z0[rows], mi.bf16_bits_to_f64(h[rows]), rcfg, cfg.K, round_y=0)
        stats = compare_chain(g, z_d.cpu().numpy()[rows], hrun_d.cpu().numpy()[rows], o, seqs, cfg.L, cfg.K,
                              rcfg, plain=plain, max_exempt=max_exempt)
        print(f"\n[{cfg.name or cfg.cid} d={cfg.d} V={cfg.V} M={cfg.M}] {stats}")
        return prob, g, o, stats
    except Exception:
        prob.close()
        raise


def test_pack_weight_layout():
    rng = np.random.default_rng(3)
    for rows, cols in ((32, 16), (70, 48), (129, 256)):
        w = rng.integers(0, 65536, (rows, cols), dtype=np.uint16)
        out = mrp.pack_weight(dev_bits(w)).cpu().numpy().view(np.uint16)
        rpad = (rows + 31) // 32 * 32
        assert out.size == rpad * cols
        wp = np.zeros((rpad, cols), np.uint16); wp[:rows] = w
        # [row block][col block][lane][8] with lane = row % 32 + 32 * ((col % 16) // 8)
        ref = wp.reshape(rpad // 32, 32, cols // 16, 2, 8).transpose(0, 2, 3, 1, 4).reshape(-1)
        np.testing.assert_array_equal(out, ref)


def test_pack_body_weight_converts_to_fp16():
    """Head-body weights: same block layout, every bf16 value as the nearest fp16 (exact in fp16's
    normal range, subnormal below 6.1e-5)."""
    rng = np.random.default_rng(4)
    rows, cols = 70, 48
    vals = rng.normal(0, 0.02, (rows, cols)).astype(np.float32)
    vals[0, :8] = [0.0, 1.0, -2.5, 3e-5, -1e-6, 6.1e-5, 1000.0, -0.0]
    w = mi.f32_to_bf16_bits(vals)
    out = mrp.pack_weight(dev_bits(w), body=True).cpu().numpy().view(np.uint16)
    rpad = (rows + 31) // 32 * 32
    want = np.zeros((rpad, cols), np.uint16)
    want[:rows] = mi.bf16_bits_to_f32(w).astype(np.float16).view(np.uint16)
    ref = want.reshape(rpad // 32, 32, cols // 16, 2, 8).transpose(0, 2, 3, 1, 4).reshape(-1)
    np.testing.assert_array_equal(out, ref)


def test_config0_tiny():
    cfg = mi.config(0)
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=cfg.tau))
    prob.close()
    assert stats["diverged"] == 0


def test_ragged_rows_and_vocab_with_remask():
    # M = 35 (ragged 32-row tile), V = 4100 (ragged 32- and 128-wide vocabulary tiles), d = 384
    cfg = mi.straddling(mi.config(0, d=384, V=4100, B=5, L=7))
    rcfg = mrp.RevealCfg(tau=0.5, tau_remask=0.3)
    prob, g, o, stats = _free_run(cfg, rcfg)
    prob.close()
    assert (o.out.remasked.sum() > 0) and ((o.out.revealed_at == 0).sum() > cfg.B)


def test_scalar_vocab_path_and_max_accept():
    cfg = mi.straddling(mi.config(0, d=128, V=4099, B=3, L=16))
    rcfg = mrp.RevealCfg(tau=0.3, max_accept=1)
    prob, g, o, stats = _free_run(cfg, rcfg)
    prob.close()


@pytest.mark.timeout(600)
def test_maximum_hidden_size_and_block_length():
    """The largest hidden size (d = 8192) and block length (L = 64) the library accepts."""
    cfg = mi.straddling(mi.config(0, d=8192, V=1024, B=2, L=64, K=1))
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=0.9, tau_remask=0.5, max_accept=1))
    prob.close()


def test_block_of_one_position():
    """L = 1: every sequence is a single row; the forced reveal takes it at state 0, later states have
    nothing left to reveal (draft (-1, -1)) and keep the conditioning token."""
    cfg = mi.straddling(mi.config(0, B=9, L=1, K=2))
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=0.9))
    prob.close()
    assert np.all(g.draft_pos[:, 0] == 0) and np.all(g.draft_pos[:, 1:] == -1)
    assert np.all(g.masked == 0)


@pytest.mark.parametrize("B,L", [(12, 64), (40, 7), (112, 7)])
def test_tile_major_partials_with_odd_and_long_blocks(B, L):
    """The GEMM kernels that own whole row tiles write their vocabulary partials tile-major; the merge
    then runs threads over a sequence's rows (block lengths that are not a power of two, and the longest)."""
    cfg = mi.straddling(mi.config(0, d=256, V=4096 + 36, B=B, L=L, K=1))
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=0.9, tau_remask=0.5), seqs=list(range(0, B, max(1, B // 6))))
    prob.close()


def test_many_rows_wide_tile_static_top2():
    # M = 336: the LM head in two row tiles of 192 rows, the second ragged
    cfg = mi.straddling(mi.config(0, d=256, V=2048 + 64, B=21, L=16))
    rcfg = mrp.RevealCfg(tau=1.0, r_min=2)           # static decoding: the two most confident per state
    prob, g, o, stats = _free_run(cfg, rcfg)
    prob.close()
    assert np.all((g.masked.reshape(cfg.B, cfg.L) == 0).sum(1) == 2 * (cfg.K + 1))


def test_tiled_path_ragged_tiles():
    # M = 800 >= 768 selects the tile kernel throughout: 4 row tiles of 224 rows (the last with 128),
    # V = 1000 -> 4 vocabulary tiles (the last with 232 entries, 8 of them in a partial 32-block)
    cfg = mi.straddling(mi.config(0, d=128, V=1000, B=50, L=16))
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=0.5, tau_remask=0.3))
    prob.close()
    # 768 rows (three whole tiles) and a vocabulary that is not a multiple of 4: rows on 8-byte boundaries
    cfg = mi.straddling(mi.config(0, d=256, V=1030, B=48, L=16, K=2))
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=0.5))
    prob.close()


def test_weight_shared_heads_and_alg4_mode():
    # one module applied K times; reveal only at state 0, remask with the same tau (Algorithm 4)
    cfg = mi.straddling(mi.config(0, d=256, V=4096, B=8, L=8, K=2))
    rcfg = mrp.RevealCfg(tau=0.6, tau_remask=0.6, head_reveal=0)
    prob, g, o, stats = _free_run(cfg, rcfg, share_heads=True)
    prob.close()
    assert np.all(g.draft_pos[:, 1:] == -1)


def test_gamma_variants():
    cfg = mi.config(0, B=4, L=4)
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=cfg.tau), gamma="normal")
    prob.close()


def test_zero_residual_bit_exact_and_deterministic():
    cfg = mi.config(0, B=6, L=4, V=4100)
    prob = Problem(cfg, gamma="zeros")
    try:
        z0 = mi.logits0(cfg); h = mi.hidden(cfg)
        z_d = torch.from_numpy(z0).cuda()
        io, _ = gpu_chain(prob, cfg.B, cfg.K, z_d, h, mrp.RevealCfg(tau=cfg.tau))
        g = io_to_host(io)
        np.testing.assert_array_equal(z_d.cpu().numpy(), z0)              # z + 0 == z, bit for bit
        for k in range(1, cfg.K + 1):
            np.testing.assert_array_equal(g.tok[k], g.tok[0])
            np.testing.assert_allclose(g.conf[k], g.conf[0], rtol=1e-5)
    finally:
        prob.close()
    # same inputs twice -> bit-identical outputs (fixed-order split-vocabulary merge)
    cfg = mi.straddling(mi.config(0, d=256, V=8200, B=9, L=16))
    prob = Problem(cfg)
    try:
        z0 = mi.logits0(cfg); h = mi.hidden(cfg)
        outs = []
        for _ in range(2):
            z_d = torch.from_numpy(z0).cuda()
            io, hr = gpu_chain(prob, cfg.B, cfg.K, z_d, h, mrp.RevealCfg(tau=0.5, tau_remask=0.3))
            g = io_to_host(io)
            outs.append((z_d.cpu().numpy(), hr.cpu().numpy(), g))
        np.testing.assert_array_equal(outs[0][0], outs[1][0])
        np.testing.assert_array_equal(outs[0][1], outs[1][1])
        for f in ("tok", "conf", "lse", "masked", "revealed_at", "draft_pos", "draft_tok", "remasked", "cond_tok"):
            np.testing.assert_array_equal(getattr(outs[0][2], f), getattr(outs[1][2], f))
    finally:
        prob.close()


def test_teacher_forced_heads_and_resume():
    """Each head on its own, fed the oracle's previous state (so a flipped decision in one
    head cannot hide errors in the next), and a resumed call equals the tail of a full run."""
    cfg = mi.straddling(mi.config(0, d=256, V=4096, B=6, L=8))
    rcfg = mrp.RevealCfg(tau=0.5, tau_remask=0.3)
    prob = Problem(cfg)
    try:
        z0 = mi.logits0(cfg); h = mi.hidden(cfg)
        seqs = list(range(cfg.B))
        full = oracle_chain(prob, z0, mi.bf16_bits_to_f64(h), rcfg, cfg.K)
        for k in range(1, cfg.K + 1):
            s = full.snaps[k - 1]
            io = mrp.StepIO(cfg.B, cfg.L, 1)
            io.masked.copy_(torch.from_numpy(s.masked)); io.revealed_at.copy_(torch.from_numpy(s.revealed_at))
            io.cond_tok.copy_(torch.from_numpy(s.cond_tok)); io.protect_pos.copy_(torch.from_numpy(s.protect_pos))
            io.x_tok.copy_(torch.from_numpy(s.x_tok))
            z_d = torch.from_numpy(s.z.astype(np.float32)).cuda()
            hrun_d = torch.from_numpy(s.hrun.astype(np.float32)).cuda()
            r1 = mrp.RevealCfg(tau=rcfg.tau, tau_remask=rcfg.tau_remask, fresh_block=0, state_offset=k - 1,
                               run_state0=0)
            io, hrun_d = gpu_chain(prob, cfg.B, 1, z_d, None, r1, io=io, hrun_d=hrun_d, heads=prob.heads_d[k - 1:k])
            g = io_to_host(io)
            o1 = oracle_chain(prob, s.z, s.hrun, r1, 1, masked=s.masked, revealed_at=s.revealed_at,
                              cond_tok=s.cond_tok, protect_pos=s.protect_pos, heads=prob.heads[k - 1:k], x_tok=s.x_tok)
            stats = compare_chain(g, z_d.cpu().numpy(), hrun_d.cpu().numpy(), o1, seqs, cfg.L, 1, r1)
            print(f"\n[teacher-forced head {k}] {stats}")
            np.testing.assert_array_equal(o1.out.tok[1], full.out.tok[k])
    finally:
        prob.close()


def test_sdar_width_vocab_few_rows():
    # real vocabulary and hidden size of the 1.7B-shaped configuration, two sequences
    cfg = mi.config(1, B=2, spike_frac=0.5)
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=cfg.tau))
    prob.close()


def test_empty_batch_and_errors():
    cfg = mi.config(0)
    prob = Problem(cfg)
    try:
        ctx = prob.ctx
        io = mrp.StepIO(1, cfg.L, cfg.K)
        z_d = torch.from_numpy(mi.logits0(cfg)).cuda()
        hrun = torch.zeros((cfg.M, cfg.d), dtype=torch.float32, device="cuda")
        h_d = dev_bits(mi.hidden(cfg))
        rc = mrp.RevealCfg()
        args = (h_d, hrun, prob.E_d, prob.Wp_d, prob.heads_d, z_d, rc, io)
        assert ctx.chain_step(0, cfg.K, *args) == 0                       # empty batch: nothing to do
        assert ctx.chain_step(2, cfg.K, *args, check=False) == -4          # rows beyond the workspace
        assert "max_rows" in ctx.last_error()
        assert ctx.chain_step(1, 17, *args, check=False) == -2             # too many heads
        assert ctx.chain_step(1, cfg.K, h_d, None, *args[2:], check=False) == -1
        zz = torch.zeros(cfg.M * cfg.V + 4, dtype=torch.float32, device="cuda")[1:]  # misaligned view
        with pytest.raises(mrp.MrpError):
            ctx.chain_step(1, cfg.K, h_d, hrun, prob.E_d, prob.Wp_d, prob.heads_d, zz[:cfg.M * cfg.V], rc, io)
        with pytest.raises(mrp.MrpError):
            mrp.MrpContext(100, 4096, 4, 4)                                # d not a multiple of 128
        with pytest.raises(mrp.MrpError):
            mrp.pack_weight(torch.zeros((4, 10), dtype=torch.int16, device="cuda"))
        torch.cuda.synchronize()
    finally:
        prob.close()


@pytest.mark.parametrize("d,B,L,K", [
    (256, 129, 1, 2),    # one row past the persistent kernel's 128-row form: the tile kernel (160-row tiles), five row tiles of the body
    (256, 16, 16, 2),    # 256 rows: the persistent kernel's 256-row form filled exactly
    (256, 257, 1, 1),    # the tile kernel again (two 160-row tiles); nine row tiles of the body: 64-feature tiles
    (256, 32, 16, 1),    # 512 rows: two tiles of 256
    (256, 513, 1, 1),    # one row past: three tiles of 192
    (256, 59, 13, 1),    # 767 rows, the last row count of the small-row head body at this width
    (4096, 25, 8, 2),    # wide model, 200 rows: persistent kernel (17 tiles leave their round empty); 64-feature tiles, 7 row tiles
    (4096, 37, 16, 1),   # wide model, 592 rows: tile kernel with k split for the head body (48 tiles x 4 parts)
])
def test_row_counts_where_the_kernels_change(d, B, L, K):
    """Row counts on both sides of the switches by rows alone (LM head: 128 / 512 rows; head body: 768 rows, 512 for
    d > 2048; 32- against 64-feature tiles), each against the oracle.  The switches that go by width or vocabulary, too:
    the tests below."""
    V = 1028 if d > 256 else 4096 + 36
    cfg = mi.straddling(mi.config(0, d=d, V=V, B=B, L=L, K=K))
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=0.9, tau_remask=0.5), seqs=list(range(0, B, max(1, B // 5))))
    prob.close()


@pytest.mark.parametrize("d,B,L,K", [
    (4096, 8, 16, 1),    # 128 rows: small-row kernels
    (4096, 43, 3, 2),    # 129 rows: the tile kernel, 16 tiles of 160 rows x 16 parts; the second head's two planes
    (4096, 16, 16, 1),   # 256 rows: one row of 256-row tiles
    (4096, 24, 16, 1),   # 384 rows
    (2560, 12, 16, 1),   # 192 rows, a width whose parts leave the tile kernel's round empty: small-row kernels
    (2048, 64, 16, 1),   # 1024 rows: second GEMM on 128-row tiles
    (384, 48, 16, 2),    # 768 rows, a width that ends inside a tile
    (384, 59, 13, 1),    # 767 rows: small-row kernels (24 row tiles)
    (384, 257, 1, 1),    # nine row tiles: 64-feature tiles
])
def test_head_body_on_tiles(d, B, L, K):
    """The MLP head body on both sides of the switch to the tile kernel below 768 rows, and its second GEMM's forms."""
    cfg = mi.straddling(mi.config(0, d=d, V=1028, B=B, L=L, K=K))
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=2.0), seqs=[0, B // 2, B - 1])
    prob.close()


# Vocabularies are chosen by how full they leave the rounds of one tile per CU on 256 CUs
@pytest.mark.parametrize("d,B,L,V,tiles", [
    (256, 160, 1, 1028, True),          # up to 160 rows any vocabulary of one round
    (256, 161, 1, 1028, False),         # from 161 narrow operands stay on the persistent kernel ...
    (128, 257, 1, 35072, False),        # ... and past 256 where 274 tiles leave the second round empty: 256 + 1 rows
    (128, 32, 16, 35072, False),        # 512 rows: two full launches
    (256, 17, 16, 57344, True),         # 272 rows, 448 tiles of 512 slots: seven eighths (d < 1024)
    (256, 17, 16, 57088, False),        # 446
    (1024, 17, 16, 49152, True),        # 384 tiles: three quarters
    (1024, 17, 16, 48896, False),       # 382; two launches
    (2048, 11, 16, 49152, True),        # 176 rows, d = 2048: 192 tiles of 256
    (2048, 11, 16, 48896, False),       # 191
])
def test_lm_head_kernel_by_width_and_vocabulary(d, B, L, V, tiles):
    """129 to 512 rows: both sides of every switch between the tile kernel and the persistent kernel (in one launch up to
    256 rows, in two beyond); first and last sequence compared (first and last row group)."""
    assert lm_head_on_tiles(B * L, d, V) == tiles
    cfg = mi.straddling(mi.config(0, d=d, V=V, B=B, L=L, K=1))
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=2.0), seqs=[0, B - 1])
    prob.close()


@pytest.mark.parametrize("d,B,L", [
    (128, 5, 16), (256, 3, 1), (256, 7, 11), (256, 4, 16),      # one workgroup per sequence
    (256, 300, 4),                                              # more of them than CUs; partials tile by tile
    (256, 512, 1), (256, 513, 1),                               # blocks of one row: two rounds of workgroups, past them the general path
    (128, 1537, 1), (256, 1540, 2),                             # more short blocks than it pays for
    (256, 3, 17), (384, 4, 16),                                 # a longer block, a wider model
])
def test_narrow_head_body(d, B, L):
    """The head body as one workgroup per sequence (d of 128 or 256, blocks of up to 16 rows) and past its limits: three heads
    with remasking, then one head that continues without a state 0 and without the hidden carry."""
    cfg = mi.straddling(mi.config(0, d=d, V=4100, B=B, L=L, K=3))
    rcfg = mrp.RevealCfg(tau=0.5, tau_remask=0.3)
    prob, g, o, stats = _free_run(cfg, rcfg, seqs=list(range(0, B, max(1, B // 5))))
    try:
        s = o.snaps[1]
        h = mi.hidden(cfg)
        full = list(range(0, B, max(1, B // 5)))
        io = mrp.StepIO(len(full), L, 1)
        io.masked.copy_(torch.from_numpy(s.masked)); io.revealed_at.copy_(torch.from_numpy(s.revealed_at))
        io.cond_tok.copy_(torch.from_numpy(s.cond_tok)); io.protect_pos.copy_(torch.from_numpy(s.protect_pos))
        io.x_tok.copy_(torch.from_numpy(s.x_tok))
        rows = np.concatenate([np.arange(b * L, (b + 1) * L) for b in full])
        z_d = torch.from_numpy(s.z.astype(np.float32)).cuda()
        r1 = mrp.RevealCfg(tau=0.5, tau_remask=0.3, fresh_block=0, state_offset=1, run_state0=0, carry_hidden=0)
        io, hrun_d = gpu_chain(prob, len(full), 1, z_d, h[rows], r1, io=io, heads=prob.heads_d[1:2])
        np.testing.assert_array_equal(hrun_d.cpu().numpy(), mi.bf16_bits_to_f64(h[rows]).astype(np.float32))   # not carried
        o1 = oracle_chain(prob, s.z, mi.bf16_bits_to_f64(h[rows]), r1, 1, masked=s.masked, revealed_at=s.revealed_at,
                          cond_tok=s.cond_tok, protect_pos=s.protect_pos, heads=prob.heads[1:2], x_tok=s.x_tok)
        compare_chain(io_to_host(io), z_d.cpu().numpy(), hrun_d.cpu().numpy(), o1, list(range(len(full))), L, 1, r1)
    finally:
        prob.close()


@pytest.mark.parametrize("B,L,V", [
    (9, 16, 32768), (9, 16, 33024),      # 144 rows, tiles of 5 row blocks: 128 tiles are halved (3 + 2 blocks), 129 are not
    (24, 16, 16384), (24, 16, 16640),    # 384 rows, 6 row blocks: 2 x 64, 2 x 65 tiles
    (25, 16, 16384), (25, 16, 16640),    # 400 rows, 7 row blocks (4 + 3; the last half is one row block)
    (32, 16, 16384), (32, 16, 16640),    # 512 rows, 8 row blocks
    (9, 16, 32767), (25, 16, 16383),     # the same where rows end inside a piece, halved
    (9, 16, 33021), (24, 16, 16637), (25, 16, 16638), (32, 16, 16639),      # ... and whole
    (33, 16, 22016),                     # 528 rows: 258 tiles, two of them left over and halved
])
def test_left_over_tiles(B, L, V):
    """LM head on the tile kernel with its left-over tiles halved (up to 128 of them) or whole, at every height; first, middle
    and last sequence compared (every logit of the others, and what lies behind them: below)."""
    cfg = mi.straddling(mi.config(0, d=128, V=V, B=B, L=L, K=1))
    assert B * L > 512 or lm_head_on_tiles(B * L, 128, V)
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=2.0), seqs=[0, B // 2, B - 1])
    prob.close()


@pytest.mark.parametrize("B,L,V", [
    (37, 16, 16640), (37, 16, 8192),     # 592 rows: the last of three 224-row tiles holds 144, five 16-row groups lie past them; halved
    (33, 16, 22016), (33, 16, 16640),    # 528 rows: 144 of 192; halved
    (25, 16, 16384), (25, 16, 16644),    # 400 rows: 176 of 224, halved at 128 rows of a tile; whole, the rows end inside a tile
    (18, 16, 16384), (18, 16, 16640),    # 288 rows: 128 of 160
    (129, 1, 33024), (577, 1, 16640),    # one row in the first group past a whole number of groups; of three 224-row tiles
    (513, 1, 8192), (153, 2, 16388),     # one row in a half; 306 rows: 146 of 160
    (24, 16, 16384), (32, 16, 16640),    # whole tiles only
    (25, 16, 16383), (153, 2, 16641),    # rows that start on any 4-byte boundary
    (65, 2, 4200004),                    # byte offsets of a tile beyond 32 bits
])
def test_every_logit_once_and_nothing_behind_them(B, L, V):
    """The tile kernel's tiles that hold fewer rows than they are high, after a larger batch on the same context (the LM head's
    operand rows past the batch are then not zero): every logit against the same sequences in batches of at most 128 rows,
    which the persistent kernel takes, and a guard of a whole tile's rows behind the matrix."""
    d, M, more = 128, B * L, 256 // L
    assert M > 512 or lm_head_on_tiles(M, d, V)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + V)
    normal = lambda *s, std, dtype=torch.bfloat16: torch.empty(s, dtype=dtype, device="cuda").normal_(0, std, generator=gen)
    E, W = normal(V, d, std=0.02), normal(V, d, std=0.02)
    Wp = mrp.pack_weight(W)
    head = [mrp.Head(mrp.pack_weight(normal(d, 2 * d, std=0.05), body=True), mrp.pack_weight(normal(d, d, std=0.05), body=True),
                     torch.ones(d, dtype=torch.bfloat16, device="cuda"))]
    h, z0 = normal((B + more) * L, d, std=1.0), normal(M, V, std=2.0, dtype=torch.float32)
    rcfg = mrp.RevealCfg(tau=2.0)

    def run(ctx, z, first, n):
        hrun = torch.zeros(n * L, d, device="cuda")
        ctx.chain_step(n, 1, h[first * L:(first + n) * L], hrun, E, Wp, head, z, rcfg, mrp.StepIO(n, L, 1))
        torch.cuda.synchronize()

    ctx = mrp.MrpContext(d, V, (B + more) * L, L)
    run(ctx, torch.zeros((B + more) * L, V, device="cuda"), 0, B + more)
    flat = torch.full(((M + 256) * V,), 7.0, device="cuda")
    z = flat[:M * V].view(M, V)
    z.copy_(z0)
    run(ctx, z, 0, B)
    assert bool((flat[M * V:] == 7.0).all())
    # two orders of summing 128 products, at most 128 roundings each; |w . y| <= |w| |y| with |y| = sqrt(d) from the norm
    w_norm = float(W.float().norm(dim=1).max())
    for b0 in range(0, B, 128 // L):
        n, rows = min(128 // L, B - b0), slice(b0 * L, (b0 + min(128 // L, B - b0)) * L)
        ref = z0[rows].clone()
        run(ctx, ref, b0, n)
        assert bool(((ref - z0[rows]).abs().amax(1) > 0.05).all())        # (the head adds something to every row)
        bound = 2 * 128 * 2.0 ** -24 * w_norm * 1.01 * d ** 0.5 + 2.0 ** -23 * ref.abs()
        assert bool(((z[rows] - ref).abs() <= bound).all()), b0
    ctx.close()


@pytest.mark.parametrize("d,B,L,features", [
    (1024, 4, 4, 16), (1024, 17, 1, 32),                       # 16 rows | 17
    (2048, 4, 4, 16), (2048, 17, 1, 16), (2048, 4, 16, 16),    # one half tile of rows; two, the second with one row; 64 rows
    (2048, 13, 5, 32),                                         # 65 rows: three row tiles of 64 would pass the CU count
    (4096, 8, 4, 16), (4096, 11, 3, 32),                       # 32 rows | 33
])
def test_head_tiles_of_16_features(d, B, L, features):
    """Both sides of the switch between 16- and 32-feature tiles of the head GEMMs, two heads (the second takes both planes
    of the running hidden state), every sequence compared."""
    assert small_tile_features(d, d, B * L) == features
    cfg = mi.straddling(mi.config(0, d=d, V=1028, B=B, L=L, K=2))
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=2.0))
    prob.close()


@pytest.mark.parametrize("B,L,V", [(1, 3, 1001),      # one row block; the last 32-block of the vocabulary holds 9 entries
                                   (15, 4, 4099),     # 60 rows: persistent kernel, two row blocks
                                   (10, 10, 4099),    # 100 rows: four
                                   (25, 8, 4099),     # 200 rows: eight (d < 2048 stays on the persistent kernel to 256 rows)
                                   (9, 16, 4099),     # 144 rows: one 160-row tile
                                   (20, 16, 2049),    # 320 rows: 160-row tiles, the last one holds one entry
                                   (25, 16, 35073),   # 400 rows on the persistent kernel: 276 tiles leave a round half empty
                                   (33, 16, 1002),    # 528 rows on the tile kernel, rows on 8-byte boundaries
                                   (33, 16, 1025),    # ... on 4-byte boundaries, one entry in the last piece
                                   (130, 5, 1031),    # 650 rows, a row ends 3 entries into a piece
                                   (600, 1, 6)])      # a row shorter than two pieces
def test_vocabulary_not_a_multiple_of_four(B, L, V):
    """Rows of the logit state start on any 4-byte boundary: the persistent kernel's forms and the tile kernel at two k steps
    (more of them, and its tallest tiles: below), and nothing written past the end."""
    cfg = mi.straddling(mi.config(0, d=128, V=V, B=B, L=L, K=2))
    prob = Problem(cfg)
    rcfg = mrp.RevealCfg(tau=0.9, tau_remask=0.5)
    z0, h = mi.logits0(cfg), mi.hidden(cfg)
    flat = torch.full((cfg.M * V + 64,), 7.0, device="cuda")
    z_d = flat[:cfg.M * V].view(cfg.M, V)
    z_d.copy_(torch.from_numpy(z0))
    io, hrun_d = gpu_chain(prob, B, cfg.K, z_d, h, rcfg)
    o = oracle_chain(prob, z0, mi.bf16_bits_to_f64(h), rcfg, cfg.K)
    # All sequences are compared, so a decision may fall between two confidences that agree to 1e-3 (relative).  On these
    # fixed inputs one does and comes out the other way, in one of the 130 sequences of 5 positions.
    compare_chain(io_to_host(io), z_d.cpu().numpy(), hrun_d.cpu().numpy(), o, list(range(B)), L, cfg.K, rcfg,
                  max_exempt=1 if B == 130 else 0)
    assert bool((flat[cfg.M * V:] == 7.0).all())
    prob.close()


@pytest.mark.parametrize("d,B,L,V", [
    (384, 9, 16, 1025),       # 144 rows: one tile of five row blocks, 6 k steps
    (640, 24, 16, 1031),      # 384 rows: six row blocks, 10 k steps
    (768, 28, 16, 1030),      # 448 rows: seven, 12 k steps
    (512, 32, 16, 1025),      # 512 rows: eight, 8 k steps
    (640, 32, 16, 1027),      # ... 10
    (768, 32, 16, 1026),      # ... 12: with the two above every remainder of the unrolled k loop
    (512, 64, 16, 1029),      # 1024 rows: four tiles
    (2048, 16, 16, 50257),    # 256 rows: one tile of eight per 256 entries, 197 of them
])
def test_odd_vocabulary_at_every_tile_height(d, B, L, V):
    """The tile kernel's form for rows that start on any 4-byte boundary: every height of its tiles, past the two k steps
    that its last requests are dealt over, against the oracle on the first, a middle and the last sequence.  The threshold
    is out of reach, so a state's decision is its most confident row; in the oracle the two most confident rows of these
    sequences are at least 9e-6 apart, 150 times fp32's resolution there (the next sequence of the 384-row case has two
    that are 9e-8 apart)."""
    cfg = mi.straddling(mi.config(0, d=d, V=V, B=B, L=L, K=1))
    prob, g, o, stats = _free_run(cfg, mrp.RevealCfg(tau=2.0), seqs=[0, B // 2, B - 1])
    prob.close()


@pytest.mark.parametrize("d,L,B,B_big", [(2048, 4, 4, 32), (2048, 16, 4, 8), (1024, 4, 4, 8)])
def test_16_feature_tiles_are_no_further_from_64_bits(d, L, B, B_big):
    """The head GEMMs on 16-feature tiles (16 and 64 rows) and, in a larger batch, on 32-feature tiles, for the same rows:
    both sum the same exact products in fp32, so the half tiles' error of h_run - h against fp64 may not be the larger one
    (a root mean square over at least 16 x 1024 sums, of which each kernel's rounding is a fixed property)."""
    K, V = 2, 4096
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + B)
    normal = lambda *s, std=0.02: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=gen)
    E, W = normal(V, d), normal(V, d)
    w = [(normal(d, 2 * d), normal(d, d)) for _ in range(K)]
    h, z = normal(B_big * L, d, std=1.0), torch.empty(B_big * L, V, device="cuda").normal_(0, 2, generator=gen)
    gamma = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    heads = [mrp.Head(mrp.pack_weight(a, body=True), mrp.pack_weight(b, body=True), gamma) for a, b in w]
    Wp, err = mrp.pack_weight(W), []
    for nb in (B, B_big):
        ctx, io = mrp.MrpContext(d, V, nb * L, L), mrp.StepIO(nb, L, K)
        hrun = torch.zeros(nb * L, d, device="cuda")
        ctx.chain_step(nb, K, h[:nb * L], hrun, E, Wp, heads, z[:nb * L].clone(), mrp.RevealCfg(tau=2.0), io)
        x = h[:B * L].double()
        tok = io.draft_tok.view(nb, K + 1)[:B].long()          # (tau above 1: one reveal per state, the draft)
        for k, (w1, w2) in enumerate(w):
            a = torch.cat([x, E[tok[:, k]].double().repeat_interleave(L, 0)], 1) @ w1.double().t()
            x = x + (a * torch.sigmoid(a)) @ w2.double().t()
        err.append(float((hrun[:B * L].double() - x).norm() / (x - h[:B * L].double()).norm()))
        ctx.close()
    assert err[0] <= err[1] < 1e-6, err
