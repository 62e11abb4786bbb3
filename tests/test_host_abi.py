"""CPU-only checks of the C ABI: the library loads, exports what the header declares, and its host logic
(configuration checks, stash sizing, state machine) behaves without any GPU work being launched."""
import concurrent.futures
import ctypes as C
import os
import random
import re
import subprocess

import pytest

import paper_2405_18047_amd as tbp
import seeded_inputs as si
from gpu_util import PRODUCT_TILES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "tbp.h")).read()
    names = set(re.findall(r"\b(tbp_[a-z0-9_]+)\s*\(", header))
    assert {"tbp_stage_forward", "tbp_stage_backward_p1", "tbp_stage_backward_p2", "tbp_stash_query"} <= names
    L = tbp.lib()
    for n in sorted(names):
        assert hasattr(L, n), n
    assert "gfx950" in tbp.tbp_version()


def _sizes(shape, **kw):
    return tbp.tbp_stash_query(tbp.config_from_shape(shape, **kw))


def test_stash_sizes_follow_the_stash_rule():
    """W class = inputs and output derivatives of the four linear layers (+ fp32 gain partials); A class = the rest."""
    for name in ("llama7b_s1024", "llama13b_s2048", "mlp_bf16"):
        s = si.CONFIGS[name]
        T, d, f, L, M = s.tokens, s.d_model, s.d_ffn, s.n_layers, s.n_microbatches
        if s.n_heads:
            w_el = 8 * d + 3 * f
            a_el = 5 * d + s.n_heads * s.seq + 2 * f
        else:
            w_el = 2 * d + 3 * f
            a_el = d + 2 * f
        got = _sizes(s, attention=tbp.TBP_ATTN_MATERIALISED)
        w_expect = L * M * T * w_el * 2
        # + per norm and micro-batch the fp32 partial rows of the gain gradient, as backward-p1's row kernel leaves them
        n_part = tbp.lib().tbp_rmsnorm_partial_rows(tbp.TBP_BF16, T, d)
        assert 1 <= n_part <= 256
        g_expect = L * 2 * M * n_part * d * 4          # (room for both norms of a layer, used or not)
        assert w_expect + g_expect <= got["w_stash_bytes"] <= w_expect * 1.001 + g_expect + 4096 * L
        assert got["a_stash_bytes"] == L * M * T * a_el * 2
        assert got["arena_bytes"] >= got["w_stash_bytes"] + got["a_stash_bytes"] + got["workspace_bytes"]
        if s.n_heads:     # fused attention keeps a row log-sum-exp (fp32 per token and head) instead of the probabilities
            fused = _sizes(s, attention=tbp.TBP_ATTN_FUSED)
            assert fused["a_stash_bytes"] == L * M * T * ((5 * d + 2 * f) * 2 + s.n_heads * 4)
            assert fused["w_stash_bytes"] == got["w_stash_bytes"]
            assert _sizes(s)["a_stash_bytes"] == fused["a_stash_bytes"]       # AUTO picks it for bf16, head_dim 128
            # dq by a recompute pass, which these stages take by themselves: the same stash, no dS^T workspace
            lean = _sizes(s, attention=tbp.TBP_ATTN_FUSED_RECOMPUTE)
            assert lean["a_stash_bytes"] == fused["a_stash_bytes"] and lean["w_stash_bytes"] == fused["w_stash_bytes"]
            assert fused["workspace_bytes"] == lean["workspace_bytes"]
        # gain gradients computed in p2: each norm's input moves from the forward->p1 slots to slabs kept until p2 and
        # the derivative of its output is kept as well; the fp32 partials disappear
        lit = _sizes(s, gain_grad=tbp.TBP_GAIN_LITERAL)
        n_norms = 2 if s.n_heads else 1
        assert lit["a_stash_bytes"] == _sizes(s)["a_stash_bytes"] - L * M * T * n_norms * d * 2
        w_lit = L * M * T * (w_el + 2 * n_norms * d) * 2
        assert w_lit <= lit["w_stash_bytes"] <= w_lit * 1.001 + 4096 * L
    # fewer activation slots shrink only the forward->p1 part
    s = si.CONFIGS["llama7b_s1024"]
    assert _sizes(s, act_slots=1)["a_stash_bytes"] * 4 == _sizes(s)["a_stash_bytes"]
    assert _sizes(s, act_slots=1)["w_stash_bytes"] == _sizes(s)["w_stash_bytes"]
    # where the backward rebuilds dq on its own account, no dS^T workspace is asked for: at head_dim 64; at 128 on up to 512
    # workgroups of 128 keys (unmasked 128), above 768 keys (unmasked from 512 workgroups on), or 512 from 1024 workgroups on
    for heads, dh, seq, batch, causal, rebuilt in (
            (32, 128, 2048, 2, True, True), (31, 128, 2048, 2, True, True), (32, 128, 512, 8, True, False), (32, 128, 520, 8, True, True),
            (32, 128, 512, 4, True, True), (33, 128, 512, 4, True, False), (33, 128, 520, 6, True, False), (40, 128, 776, 2, True, True),
            (16, 128, 1024, 1, False, True), (17, 128, 1024, 1, False, False), (32, 128, 1024, 2, False, True), (32, 128, 768, 3, False, False),
            (32, 64, 128, 32, True, True), (32, 64, 128, 31, True, True), (32, 64, 512, 8, True, True), (32, 64, 512, 6, False, True)):
        s = si.StageShape("dst", 1, heads * dh, heads, dh, 256, seq, batch, 1, "bf16", 1, causal=causal)
        saved = _sizes(s, attention=tbp.TBP_ATTN_FUSED)["workspace_bytes"] - _sizes(s, attention=tbp.TBP_ATTN_FUSED_RECOMPUTE)["workspace_bytes"]
        assert saved == (0 if rebuilt else batch * heads * seq * ((seq + 127) // 128 * 128) * 2), (heads, dh, seq, batch, causal)
        # the single operation's scratch stays large enough for any smaller call
        assert tbp.lib().tbp_attention_p1_scratch_bytes(batch, heads, seq) >= batch * heads * seq * seq * 2
    # 13B stage: everything fits the 288 GB of one MI355X
    assert _sizes(si.CONFIGS["llama13b_s2048"])["arena_bytes"] < 150 * 2**30


@pytest.mark.parametrize("field,value", [("d_model", 4100), ("d_ffn", 11004), ("seq", 4104), ("head_dim", 120),
                                         ("n_layers", 0), ("dtype", 7), ("d_model", 16384), ("seq", 8192), ("attention", 4),
                                         ("gain_grad", 2)])
def test_bad_configs_are_rejected(field, value):
    cfg = tbp.config_from_shape(si.CONFIGS["llama7b_s1024"])
    setattr(cfg, field, value)
    with pytest.raises(tbp.TbpError) as e:
        tbp.tbp_stash_query(cfg)
    assert e.value.status == 1 and str(e.value)


def test_fused_attention_is_refused_where_it_is_not_built():
    cfg = tbp.config_from_shape(si.CONFIGS["tiny_f32"], attention=tbp.TBP_ATTN_FUSED)       # fp32 storage
    with pytest.raises(tbp.TbpError) as e:
        tbp.tbp_stash_query(cfg)
    assert e.value.status == 1
    cfg = tbp.config_from_shape(si.CONFIGS["llama7b_s1024"], attention=tbp.TBP_ATTN_FUSED)
    cfg.n_heads, cfg.head_dim = 128, 32                                                       # head_dim 32
    with pytest.raises(tbp.TbpError):
        tbp.tbp_stash_query(cfg)
    tbp.tbp_stash_query(tbp.config_from_shape(si.CONFIGS["tiny_f32"]))                       # AUTO falls back


class _FakeStage:
    """A stage over made-up device addresses: valid for every host-side check, never used to launch."""

    def __init__(self, shape, arena_bytes=None, **kw):
        L = tbp.lib()
        self.cfg = tbp.config_from_shape(shape, **kw)
        n = shape.n_layers
        arr = (C.c_void_p * n)(*[0x10000 * (i + 1) for i in range(n)])
        self._keep = arr
        from paper_2405_18047_amd.binding import _tbp_params
        p = _tbp_params()
        for name, _ in p._fields_:
            setattr(p, name, C.cast(arr, C.POINTER(C.c_void_p)))
        need = tbp.tbp_stash_query(self.cfg)["arena_bytes"]
        self.h = C.c_void_p()
        self.status = L.tbp_stage_create(C.byref(self.cfg), C.byref(p), C.c_void_p(0x1000000),
                                         need if arena_bytes is None else arena_bytes, C.byref(self.h))


def test_state_machine_rejects_wrong_order_without_launching():
    L = tbp.lib()
    st = _FakeStage(si.CONFIGS["tiny_f32"])
    assert st.status == 0
    fake = C.c_void_p(0x2000000)
    # p1 before forward, p2 before p1, out-of-range micro-batch, duplicate and non-consecutive sets
    assert L.tbp_stage_backward_p1(st.h, 0, fake, fake, None) == 2
    assert b"forward" in L.tbp_last_error()
    one = (C.c_int * 2)(0, 1)
    assert L.tbp_stage_backward_p2(st.h, one, 1, 0, 1, None) == 2
    assert L.tbp_stage_forward(st.h, 4, fake, fake, None) == 1
    assert L.tbp_stage_forward(st.h, -1, fake, fake, None) == 1
    assert L.tbp_stage_forward(st.h, 0, None, fake, None) == 1
    dup = (C.c_int * 2)(1, 1)
    assert L.tbp_stage_backward_p2(st.h, dup, 2, 0, 1, None) == 1
    assert L.tbp_stage_backward_p2(st.h, one, 0, 0, 1, None) == 1
    assert L.tbp_stage_backward_p2(st.h, one, 2, 5, 1, None) == 1
    from paper_2405_18047_amd.binding import _tbp_stash_stats
    stats = _tbp_stash_stats()
    assert L.tbp_stage_stash_stats(st.h, C.byref(stats)) == 0
    assert (stats.w_live_bytes, stats.a_live_bytes, stats.high_water_bytes) == (0, 0, 0)
    assert L.tbp_stage_reset(st.h) == 0
    L.tbp_stage_destroy(st.h)


def test_create_rejects_small_arena_and_null_pointers():
    L = tbp.lib()
    st = _FakeStage(si.CONFIGS["tiny_f32"], arena_bytes=1024)
    assert st.status == 3 and b"arena" in L.tbp_last_error()
    cfg = tbp.config_from_shape(si.CONFIGS["tiny_f32"])
    h = C.c_void_p()
    assert L.tbp_stage_create(C.byref(cfg), None, C.c_void_p(0x1000), 1 << 40, C.byref(h)) == 1


def test_single_op_argument_checks():
    L = tbp.lib()
    fake = C.c_void_p(0x2000000)
    # bf16 extents must be multiples of 8; accumulate needs fp32 output; unknown layout
    assert L.tbp_gemm(1, 2, 100, 64, 64, 1.0, fake, 100, fake, 64, fake, 64, 1, 0, None, None) == 1
    assert L.tbp_gemm(1, 1, 64, 64, 64, 1.0, fake, 64, fake, 64, fake, 64, 0, 1, None, None) == 1
    assert L.tbp_gemm(1, 3, 64, 64, 64, 1.0, fake, 64, fake, 64, fake, 64, 0, 0, None, None) == 1
    assert L.tbp_gemm(1, 0, 0, 64, 64, 1.0, None, 64, None, 64, None, 64, 0, 0, None, None) == 0   # empty: no-op
    assert L.tbp_rmsnorm_fwd(1, 4, 12, 1e-6, fake, fake, fake, None) == 1
    assert L.tbp_softmax_fwd(1, 1, 8192, 1, fake, fake, None) == 1
    assert L.tbp_rope(1, 4, 8, 2, 24, 48, fake, 0, fake, None) == 1
    assert L.tbp_rmsnorm_p1_scratch_bytes(4096) == 256 * 4096 * 4
    # partial rows of the gain gradient: one per workgroup of the row kernel, never more than 256, none without rows
    assert L.tbp_rmsnorm_partial_rows(1, 4096, 4096) == 256 and L.tbp_rmsnorm_partial_rows(1, 0, 4096) == 0
    assert 1 <= L.tbp_rmsnorm_partial_rows(1, 5, 264) <= 5 and 1 <= L.tbp_rmsnorm_partial_rows(0, 37, 256) <= 37
    assert L.tbp_rmsnorm_p1_partials(1, 4, 12, 1e-6, fake, fake, fake, None, fake, fake, None) == 1
    assert L.tbp_gain_partials_sum(None, 3, 64, 0, fake, None) == 1
    # the variant with the library's static scratch refuses widths its array was not built for, before any device call
    assert L.tbp_rmsnorm_p1_static(1, 4, 8200, 1e-6, fake, fake, fake, None, fake, fake, None) == 1
    assert b"static scratch" in L.tbp_last_error()
    assert L.tbp_rmsnorm_p1_static(0, 4, 4100, 1e-6, fake, fake, fake, None, fake, fake, None) == 1
    assert L.tbp_rmsnorm_p1_static(1, 4, 4096, 1e-6, fake, fake, fake, None, None, fake, None) == 1      # null dx
    # leading dimensions beyond what the kernels' buffer ranges address are refused, not wrapped
    assert L.tbp_gemm(1, 0, 64, 64, 64, 1.0, fake, 1 << 22, fake, 64, fake, 64, 0, 0, None, None) == 1
    assert L.tbp_attention_fwd(1, 1, 2, 4096, 64, 1, fake, 1 << 19, fake, 128, fake, None) == 1
    # dS^T scratch of the fused attention backward: row sums + panels of 128 queries (seq rounded up to 128 on one side)
    assert L.tbp_attention_p1_scratch_bytes(2, 3, 200) == 4864 + 2 * 3 * 2 * 200 * 128 * 2


def test_gemm_workspace_policy_and_checks():
    """tbp_gemm_workspace_bytes is host arithmetic: scratch is asked for only where splitting the contraction pays
    (a bf16 NN / NT product with a storage-type output that neither tile shape can spread over the chip, and a long
    contraction), and it is exactly a head of 1 KiB plus one fp32 partial product per slice."""
    L = tbp.lib()
    need = L.tbp_gemm_workspace_bytes(1, tbp.NT, 1024, 4096, 32768, 0)
    assert need == 1024 + 64 * 4 * 256 * 256 * 4                          # 64 tiles, four slices
    assert L.tbp_gemm_workspace_bytes(1, tbp.NN, 1024, 4096, 32768, 0) == need
    for args in [(1, tbp.TN, 1024, 4096, 32768, 0),      # weight-gradient layout: never split
                 (1, tbp.NT, 1024, 4096, 32768, 1),      # fp32 output
                 (0, tbp.NT, 1024, 4096, 32768, 0),      # fp32 storage
                 (1, tbp.NT, 4096, 4096, 32768, 0),      # 256 large tiles already fill the chip
                 (1, tbp.NT, 2048, 5120, 27648, 0),      # 216 tiles of 256 x 192 do
                 (1, tbp.NT, 1024, 4096, 4096, 0),       # short contraction: the exchange would cost more than it saves
                 (1, tbp.NT, 0, 4096, 32768, 0), (1, 7, 1024, 4096, 32768, 0)]:
        assert L.tbp_gemm_workspace_bytes(*args) == 0, args
    fake = C.c_void_p(0x2000000)
    # a misaligned workspace is refused before anything is launched
    assert L.tbp_gemm_ws(1, tbp.NT, 1024, 4096, 32768, 1.0, fake, 32768, fake, 32768, fake, 4096, 0, 0, None,
                         C.c_void_p(0x3000010), need, None) == 1
    assert "aligned" in L.tbp_last_error().decode()


def test_backward_p2_runs_fit_the_contraction_length(tmp_path):
    """backward-p2 contracts over the rows of a run of consecutive micro-batches in one product, whose length is an int:
    sets of any accepted size are cut into runs that fit (128 micro-batches of 2^24 tokens are 2^31 rows)."""
    src = tmp_path / "runs.cpp"
    src.write_text("""
#include <cstdio>
#include <vector>
#include "kernels.h"
int main() {
  for (int tokens : {1, 2048, 1 << 20, 1 << 24}) {
    for (int n : {1, 4, 127, 128, 300}) {
      std::vector<int> mbs(n);
      for (int k = 0; k < n; k++) mbs[k] = k + (k >= n / 2 ? 1 : 0);          // two runs
      long rows = 0, longest = 0;
      int runs = 0;
      for (int i = 0; i < n;) {
        const int j = tbp::run_end(mbs.data(), n, i, tokens);
        for (int k = i + 1; k < j; k++) if (mbs[k] != mbs[k - 1] + 1) return 1;
        if ((long)(j - i) * tokens > longest) longest = (long)(j - i) * tokens;
        rows += (long)(j - i) * tokens; runs++; i = j;
      }
      if (rows != (long)n * tokens) return 2;
      std::printf("%d %d %d %ld\\n", tokens, n, runs, longest);
    }
  }
}
""")
    exe = tmp_path / "runs"
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2405_18047_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    got = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    got = {tuple(map(int, l.split()[:2])): tuple(map(int, l.split()[2:])) for l in got if l}
    assert all(longest <= 2**31 - 64 for _, longest in got.values())
    assert got[2048, 300] == (2, 150 * 2048) and got[2048, 1] == (1, 2048)          # ordinary sets: the runs themselves
    assert got[1 << 24, 128] == (2, 64 << 24) and got[1 << 24, 300][0] == 6


@pytest.mark.parametrize("layout,mnk,slower", [
    # measured, us: what the slower choice takes, and the faster one
    (tbp.NT, (592, 10616, 10248), (256, 128, 1)),        # 203, 170: two slices of 256 x 256
    (tbp.NN, (2304, 3328, 28416), (256, 128, 1)),        # 392, 365: the same
    (tbp.NT, (24, 584, 3912), (64, 64, 11)),             # 8.4, 6.5: 32 x 32, whole
    (tbp.NN, (72, 2240, 5312), (32, 32, 1)),             # 14.2-21.5, 12.6-18.6 (in steps): six slices of 64 x 64
    (tbp.NN, (176, 9280, 4160), (192, 192, 5)),          # 32.6, 27.2: 128 x 128, whole
    (tbp.NT, (2032, 2624, 848), (256, 128, 1)),          # 18.8, 18.4: 128 x 128, whole
    (tbp.NT, (2496, 1592, 1000), (256, 128, 1)),         # 20.7, 18.5: 128 x 128, whole
    (tbp.NT, (5448, 192, 1248), (128, 64, 1)),           # 13.5, 10.4: 64 x 64, whole
    (tbp.NT, (64, 11928, 11320), (64, 64, 1))])          # 100, 86: two slices of 128 x 128
def test_gemm_plan_avoids_choices_that_measured_slower(layout, mnk, slower):
    rows, cols, per_cu, slices = tbp.tbp_gemm_plan(layout, *mnk)
    assert (rows, cols, slices) != slower
    assert 1 <= per_cu <= 2 and 1 <= slices <= 16
    # without scratch nothing is cut
    assert tbp.tbp_gemm_plan(layout, *mnk, 0)[3] == 1


def test_product_tiles_list_runs_what_it_names():
    """The shapes that the GPU tests run tile by tile: the plan takes the tile and the slices that each is listed for, and every tile
    is there in both layouts, whole and (but for 32 x 32) in slices."""
    for layout, mnk, plan in PRODUCT_TILES:
        assert tbp.tbp_gemm_plan(layout, *mnk, 1024 + plan[3] * mnk[0] * mnk[1] * 4) == plan, (layout, mnk)
    got = {(layout, plan[:3], plan[3] > 1) for layout, _, plan in PRODUCT_TILES}
    tiles = {(64, 64, 2), (128, 64, 1), (128, 128, 1), (128, 128, 2), (128, 192, 1), (256, 128, 1), (192, 192, 1), (256, 192, 1), (256, 256, 1)}
    layouts = (tbp.NN, tbp.NT)
    assert got == {(lo, t, cut) for lo in layouts for t in tiles for cut in (False, True)} | {(lo, (32, 32, 1), False) for lo in layouts}


def test_no_workspace_for_products_that_take_less_than_its_allocation():
    # called in a row, us, with a workspace of its own in slices / whole: 15 / 12.0, 15 / 14.7, 14.2 / 10.9, 13.6 / 9.8, 14.3 / 10.3
    for layout, mnk in ((tbp.NN, (160, 416, 4168)), (tbp.NN, (352, 360, 4552)), (tbp.NN, (176, 928, 4712)), (tbp.NT, (136, 376, 6696)),
                        (tbp.NT, (160, 488, 7112))):
        assert tbp.lib().tbp_gemm_workspace_bytes(tbp.TBP_BF16, layout, *mnk, 0) == 0
        assert tbp.tbp_gemm_plan(layout, *mnk)[3] == 1
        assert tbp.tbp_gemm_plan(layout, *mnk, 1 << 30)[3] > 1          # scratch that is there is used
    # 14.3 / 21.3, 13.9 / 19.8 the other way round
    for layout, mnk in ((tbp.NT, (360, 4096, 11008)), (tbp.NN, (112, 728, 8120)), (tbp.NN, (280, 376, 7048)), (tbp.NN, (312, 616, 6296))):
        assert tbp.lib().tbp_gemm_workspace_bytes(tbp.TBP_BF16, layout, *mnk, 0) > 0


def test_gemm_plan_is_the_same_however_often_and_wherever_it_is_asked_for():
    """Threads keep plans that they have found: many more products than they keep, in several orders and threads."""
    rng = random.Random(5)
    cases = [(rng.choice((tbp.NN, tbp.NT)), 8 * rng.randint(1, 500), 8 * rng.randint(1, 1000), 8 * rng.randint(0, 1000)) for _ in range(900)]
    cases = [c for c in cases if -(-c[1] // 256) * -(-c[2] // 256) <= 256]
    ask = lambda c: (tbp.tbp_gemm_plan(*c), tbp.tbp_gemm_plan(*c, 0), tbp.lib().tbp_gemm_workspace_bytes(tbp.TBP_BF16, *c, 0))
    want = {c: ask(c) for c in cases}
    for c in rng.sample(cases, len(cases)) + cases[::-1]:
        assert ask(c) == want[c], c
    with concurrent.futures.ThreadPoolExecutor(4) as pool:
        assert list(pool.map(ask, cases + cases)) == [want[c] for c in cases + cases]
    for (layout, M, N, K), ((_, _, _, slices), (_, _, _, one), need) in want.items():
        assert one == 1 and (need == 0) == (slices == 1) and need >= (slices > 1) * slices * M * N * 4


def test_gemm_plan_refuses_other_products():
    for layout, M, N, K in ((tbp.TN, 64, 64, 64), (tbp.NN, 0, 64, 64), (tbp.NN, 64, 64, -1), (7, 64, 64, 64), (tbp.NN, 8192, 8192, 64)):
        with pytest.raises(tbp.TbpError):
            tbp.tbp_gemm_plan(layout, M, N, K, 0)
