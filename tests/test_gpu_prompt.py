"""GPU parity: one-shot block-level prompt compression (Section 4.2) through the C ABI against the CPU oracle,
followed by decode steps that start from the state the call leaves."""
import numpy as np
import pytest

from paper_2501_04987_amd import inputs
from tests import parity_harness as ph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    import torch

    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2501_04987_amd import binding as b

    b.load()
    return b


def _run(binding, oracle, *, T, block, steps, B, H, Hkv, d, budget, n_sink, n_recent, seed=0, flags=0, units=None,
         kind="lowrank", dtype="bf16"):
    Q, K, V = inputs.batch_streams(kind, seed, T + steps, B, Hkv, H // Hkv, d, dtype=dtype)
    kv = binding.TreeKV(budget, H, d, kv_heads=Hkv, batch=B, dtype=dtype, n_sink=n_sink, n_recent=n_recent,
                        flags=flags, max_prompt=T)
    st = ph.run_prompt(oracle, kv, Q, K, V, T, block, steps, units=units, dtype=dtype)
    assert st["flagged"] <= max(1, st["decisions"] // 200), st["flagged"]
    print(f"  blocks evicted={st['decisions']} flagged={st['flagged']} token score rel err={st['tok_err']:.2e} "
          f"score_err={st['score_err']:.2e}")
    return kv, st


def test_prompt_layout_ragged_slices(binding, oracle):
    """37 blocks of 16 into 8 block slots (1 sink, 5 tree, 2 recent blocks); the prompt's 592 keys end inside a
    workgroup iteration and inside a wave's tile; 40 decode steps wrap the recent ring."""
    _run(binding, oracle, T=592, block=16, steps=40, B=1, H=2, Hkv=2, d=128, budget=128, n_sink=4, n_recent=20)


def test_prompt_several_slices_and_batches(binding, oracle):
    _run(binding, oracle, T=4096 + 64, block=32, steps=12, B=2, H=2, Hkv=2, d=128, budget=512, n_sink=4, n_recent=100,
         seed=3)


@pytest.mark.parametrize("G,d,block", [(4, 64, 8), (2, 128, 16), (8, 64, 16)])
def test_prompt_grouped_queries(binding, oracle, G, d, block):
    _run(binding, oracle, T=block * 61, block=block, steps=10, B=1, H=2 * G, Hkv=2, d=d, budget=block * 12, n_sink=3,
         n_recent=block + 5, seed=5)


def test_prompt_window_of_128(binding, oracle):
    """block = 128: the window's 128 queries fill all eight operand blocks."""
    _run(binding, oracle, T=128 * 21, block=128, steps=6, B=1, H=2, Hkv=2, d=128, budget=1024, n_sink=4, n_recent=200,
         seed=6)


def test_prompt_pure_algorithm1_single_token_blocks(binding, oracle):
    """block = 1: Algorithm 1 over tokens with the last token's attention as frozen scores."""
    _run(binding, oracle, T=301, block=1, steps=25, B=1, H=2, Hkv=2, d=64, budget=20, n_sink=0, n_recent=0, seed=7)


def test_prompt_tree_region_wider_than_a_wave(binding, oracle):
    """150 tree slots (blocks of 1): the passes over the region take the workgroup-wide path, several passes and a
    partial last one."""
    _run(binding, oracle, T=777, block=1, steps=10, B=1, H=2, Hkv=2, d=64, budget=200, n_sink=10, n_recent=40, seed=8)


def test_prompt_tree_region_of_exactly_a_wave(binding, oracle):
    _run(binding, oracle, T=64 * 9 + 30, block=1, steps=5, B=2, H=2, Hkv=2, d=64, budget=70, n_sink=2, n_recent=4, seed=9)


def test_prompt_that_fits_keeps_everything(binding, oracle):
    kv, st = _run(binding, oracle, T=160, block=32, steps=120, B=1, H=2, Hkv=2, d=128, budget=256, n_sink=4,
                  n_recent=60, seed=8)
    assert st["decisions"] == 0 and st["decode"]["decisions"] == 2 * (160 + 120 - 256)


def test_prompt_keep_left(binding, oracle):
    _run(binding, oracle, T=16 * 50, block=16, steps=8, B=1, H=2, Hkv=2, d=128, budget=160, n_sink=0, n_recent=16,
         flags=binding.TREEKV_KEEP_LEFT, seed=9)


def test_prompt_block_size_that_straddles_slices(binding, oracle):
    """Blocks of 12 do not divide what a workgroup takes per iteration: the block means are then taken by the
    blocks kernel from the token scores."""
    _run(binding, oracle, T=12 * 130, block=12, steps=10, B=1, H=2, Hkv=2, d=128, budget=12 * 9, n_sink=5, n_recent=13,
         seed=14)


def test_prompt_of_700k_tokens_one_head(binding, oracle):
    """One head, 704000 tokens in blocks of 32: 64 slices of 11008 keys (too long for the in-kernel block means),
    22000 blocks through a tree region of 5 blocks."""
    kv, st = _run(binding, oracle, T=32 * 22000, block=32, steps=4, B=1, H=1, Hkv=1, d=64, budget=256, n_sink=4,
                  n_recent=40, seed=15, kind="iid")
    assert st["decisions"] == 22000 - 8


def test_prompt_accumulated_weight_criterion(binding, oracle):
    """With TREEKV_SCORE_ACCUMULATED a token's importance is its summed window attention; the window block's own
    tokens, seen by fewer queries, then weigh less."""
    _run(binding, oracle, T=16 * 45, block=16, steps=30, B=1, H=4, Hkv=2, d=128, budget=160, n_sink=4, n_recent=0,
         flags=binding.TREEKV_SCORE_ACCUMULATED, seed=12)


def test_prompt_replaces_earlier_state(binding, oracle):
    """The call starts from scratch whatever the context held before."""
    import torch

    T, block, B, H, d, budget = 640, 32, 1, 2, 128, 192
    Q, K, V = inputs.batch_streams("lowrank", 11, T + 4, B, H, 1, d, dtype="bf16")
    kv = binding.TreeKV(budget, H, d, kv_heads=H, batch=B, dtype="bf16", n_sink=4, n_recent=40, max_prompt=T)
    out, ret, nret, ev = kv.new_outputs()
    junk = torch.randn(B, H, d, device="cuda").to(torch.bfloat16)
    for _ in range(budget + 30):
        kv.decode_step(junk, junk, junk, out, ret, nret, ev)
    st = ph.run_prompt(oracle, kv, Q, K, V, T, block, 4)
    assert st["decisions"] == H * (T // block - budget // block)


def test_prompt_argument_errors(binding):
    import torch

    kv = binding.TreeKV(64, 2, 128, kv_heads=2, n_sink=4, n_recent=20, max_prompt=256)
    _, ret, nret, _ = kv.new_outputs()
    x = torch.zeros(1, 512, 2, 128, dtype=torch.bfloat16, device="cuda")
    for T, block in [(250, 16), (512, 16), (256, 24), (256, 0), (8, 16), (256, 32)]:   # last: no tree block left
        with pytest.raises(binding.TreeKVError) as e:
            kv.prefill_prompt(x, x, x, T, block, ret, nret)
        assert e.value.status == binding.TREEKV_EINVAL, (T, block)
    none = binding.TreeKV(64, 2, 128, kv_heads=2, n_sink=4, n_recent=20)
    with pytest.raises(binding.TreeKVError):
        none.prefill_prompt(x, x, x, 256, 16, ret, nret)                              # max_prompt = 0
    wide = binding.TreeKV(256, 8, 64, kv_heads=2, n_sink=0, n_recent=0, max_prompt=512)
    _, ret, nret, _ = wide.new_outputs()
    x = torch.zeros(1, 512, 8, 64, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(binding.TreeKVError) as e:
        wide.prefill_prompt(x, x, x, 512, 64, ret, nret)                              # 64 queries x 4 heads > 128 rows
    assert e.value.status == binding.TREEKV_EUNSUPPORTED


def test_prompt_llama_shaped_sampled(binding, oracle):
    """The benchmark's launch configuration: 32 heads x 128, bf16, budget 2048 (4 + 1024 + 1020), a prompt of 32768
    tokens in blocks of 64, then 16 decode steps; the GPU runs all heads, the oracle audits 4 of them (one of the
    heads whose keys sit at byte offset 256 mod 1024 of a token's row among them)."""
    kv, st = _run(binding, oracle, T=32768, block=64, steps=16, B=1, H=32, Hkv=32, d=128, budget=2048, n_sink=4,
                  n_recent=1020, units=[(0, 0), (0, 9), (0, 20), (0, 31)], seed=0)
    assert st["decisions"] == 4 * (32768 // 64 - 2048 // 64)


def test_prompt_chunk_and_step_replay_from_a_hip_graph(binding):
    """A prompt compression, a prefill chunk and a decode step captured in one HIP graph: no host-side state changes
    between calls, so replays with fresh inputs (and eager work in between) give exactly what eager launches give."""
    import torch

    T, block, L, B, H, d, budget, rounds = 512, 16, 48, 1, 4, 128, 96, 4
    n_tok = rounds * (T + L + 1)
    Q, K, V = inputs.batch_streams("lowrank", 33, n_tok, B, H, 1, d, dtype="bf16")
    Qd, Kd, Vd = (ph.to_device(x, "bf16") for x in (Q, K, V))
    mk = lambda x, a, n: x[a:a + n].permute(1, 0, 2, 3).contiguous()

    def make():
        return binding.TreeKV(budget, H, d, kv_heads=H, batch=B, dtype="bf16", n_sink=2, n_recent=20, max_chunk=64,
                              max_prompt=T)

    eager, graph = make(), make()
    # static buffers of the graph
    qw, kp, vp = mk(Qd, T - block, block).clone(), mk(Kd, 0, T).clone(), mk(Vd, 0, T).clone()
    qc, kc, vc = mk(Qd, T, L).clone(), mk(Kd, T, L).clone(), mk(Vd, T, L).clone()
    qs, ks, vs = Qd[T + L].clone(), Kd[T + L].clone(), Vd[T + L].clone()
    tok = torch.empty(B, H, T, dtype=torch.float32, device="cuda")
    oc, rc, nc, ec = graph.new_outputs(L)
    os_, rs, ns, es = graph.new_outputs()
    rp = torch.empty_like(rs)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        graph.prefill_prompt(qw, kp, vp, T, block, rp, None, None, tok)
        graph.prefill_chunk(qc, kc, vc, L, oc, rc, nc, ec)
        graph.decode_step(qs, ks, vs, os_, rs, ns, es)
    torch.cuda.synchronize()
    for r in range(rounds):
        a = r * (T + L + 1)
        qw.copy_(mk(Qd, a + T - block, block)); kp.copy_(mk(Kd, a, T)); vp.copy_(mk(Vd, a, T))
        qc.copy_(mk(Qd, a + T, L)); kc.copy_(mk(Kd, a + T, L)); vc.copy_(mk(Vd, a + T, L))
        qs.copy_(Qd[a + T + L]); ks.copy_(Kd[a + T + L]); vs.copy_(Vd[a + T + L])
        g.replay()
        torch.cuda.synchronize()
        # the same three calls, eagerly, on the other context
        tok_e = torch.empty_like(tok)
        oc_e, rc_e, nc_e, ec_e = eager.new_outputs(L)
        os_e, rs_e, ns_e, es_e = eager.new_outputs()
        rp_e = torch.empty_like(rs_e)
        eager.prefill_prompt(mk(Qd, a + T - block, block), mk(Kd, a, T), mk(Vd, a, T), T, block, rp_e, None, None, tok_e)
        eager.prefill_chunk(mk(Qd, a + T, L), mk(Kd, a + T, L), mk(Vd, a + T, L), L, oc_e, rc_e, nc_e, ec_e)
        eager.decode_step(Qd[a + T + L], Kd[a + T + L], Vd[a + T + L], os_e, rs_e, ns_e, es_e)
        torch.cuda.synchronize()
        for got, want in [(rp, rp_e), (tok, tok_e), (oc, oc_e), (rc, rc_e), (ec, ec_e), (os_, os_e), (rs, rs_e), (es, es_e)]:
            assert torch.equal(got, want), r
        assert torch.equal(graph.scores(), eager.scores()), r
        _ = (Qd[a].float() * 2).sum().item()                             # unrelated eager work between replays


def test_prompt_and_chunked_prefill_share_the_span_structure(binding):
    """The scopes of Algorithm 1 do not depend on the scores, so the one-shot compression with single-token blocks
    and the chunked prefill of the same prompt keep one token of every span each, whatever they score it by (the
    last query's attention / all queries' averaged attention): in position order, the i-th token one of them keeps
    lies before the (i+1)-th token the other keeps.  Sinks and the recent window are the same tokens."""
    import torch

    T, B, H, d, budget, n_sink, n_recent, L = 6000, 1, 4, 128, 256, 4, 60, 250
    Q, K, V = inputs.batch_streams("lowrank", 21, T, B, H, 1, d, dtype="bf16")
    Qd, Kd, Vd = (ph.to_device(x, "bf16").permute(1, 0, 2, 3).contiguous() for x in (Q, K, V))   # [B,T,H,d]
    one = binding.TreeKV(budget, H, d, kv_heads=H, batch=B, dtype="bf16", n_sink=n_sink, n_recent=n_recent, max_prompt=T)
    chk = binding.TreeKV(budget, H, d, kv_heads=H, batch=B, dtype="bf16", n_sink=n_sink, n_recent=n_recent, max_chunk=L)
    _, ret_one, n_one, _ = one.new_outputs()
    one.prefill_prompt(Qd[:, T - 1:T].contiguous(), Kd, Vd, T, 1, ret_one, n_one)
    for t in range(0, T, L):
        out, ret_chk, n_chk, ev = chk.new_outputs(L)
        chk.prefill_chunk(Qd[:, t:t + L].contiguous(), Kd[:, t:t + L].contiguous(), Vd[:, t:t + L].contiguous(), L, out,
                          ret_chk, n_chk, ev)
    torch.cuda.synchronize()
    a, b = ret_one.cpu().numpy()[0], ret_chk.cpu().numpy()[0]
    assert np.all(n_one.cpu().numpy() == budget) and np.all(n_chk.cpu().numpy() == budget)
    same = 0
    for h in range(H):
        assert np.array_equal(a[h, :n_sink], b[h, :n_sink]) and np.array_equal(a[h, -n_recent:], b[h, -n_recent:])
        assert np.all(a[h, :-1] < b[h, 1:]) and np.all(b[h, :-1] < a[h, 1:]), h
        same += int(np.sum(a[h] == b[h]))
    # different criteria: the two must not simply coincide on the tree region
    assert same < H * budget, same
    print(f"  same token kept in {same - H * (n_sink + n_recent)} of {H * (budget - n_sink - n_recent)} spans")


@pytest.mark.parametrize("G,d,block", [(1, 64, 16), (2, 128, 8), (4, 64, 4)])
def test_prompt_fp32_storage(binding, oracle, G, d, block):
    """fp32 storage: the window's scores come from the vector-ALU instance; blocks, hand-over and the decode steps
    that follow are the same kernels."""
    _run(binding, oracle, T=block * 41, block=block, steps=40, B=2, H=2 * G, Hkv=2, d=d, budget=block * 9, n_sink=2,
         n_recent=block + 3, seed=17, kind="iid", dtype="f32")


def test_prompt_fp32_that_fits_and_accumulated(binding, oracle):
    _run(binding, oracle, T=48, block=8, steps=30, B=1, H=2, Hkv=2, d=64, budget=64, n_sink=1, n_recent=10, seed=18,
         kind="iid", dtype="f32")
    _run(binding, oracle, T=320, block=16, steps=20, B=1, H=2, Hkv=1, d=128, budget=96, n_sink=0, n_recent=16, seed=19,
         kind="iid", dtype="f32", flags=binding.TREEKV_SCORE_ACCUMULATED)


@pytest.mark.parametrize("dtype,block", [("bf16", 16), ("bf16", 24), ("f32", 16)])
def test_prompt_token_scores_are_an_output(binding, dtype, block):
    """The state a call leaves does not depend on the buffer its token scores go to: none, one of 4-byte alignment, one
    that something else writes meanwhile (here: the call's own list of evicted blocks).  Block means taken with the
    scores (16) and afterwards (24 does not divide a workgroup's step)."""
    import torch

    B, H, d, T, budget = 2, 2, 64, block * 100, block * 20
    Q, K, V = inputs.batch_streams("lowrank" if dtype == "bf16" else "iid", 51, T, B, H, 1, d, dtype=dtype)
    Qd, Kd, Vd = (ph.to_device(x, dtype).transpose(0, 1).contiguous() for x in (Q, K, V))
    n, N = B * H * T, B * H * (T // block)

    def run(scores, evicted=None):
        kv = binding.TreeKV(budget, H, d, kv_heads=H, batch=B, dtype=dtype, n_sink=4, n_recent=block, max_prompt=T)
        _, ret, nret, _ = kv.new_outputs()
        kv.prefill_prompt(Qd[:, T - block:].contiguous(), Kd, Vd, T, block, ret, nret, evicted, scores)
        snap = kv.export_state()
        torch.cuda.synchronize()
        return ret, snap

    ret, snap = run(None)
    plain, odd, shared = (torch.full((n + 1,), -7.0, device="cuda") for _ in range(3))
    for scores, evicted in ((plain[:n], None), (odd[1:], None), (shared[:n], shared[:N].view(torch.int32))):
        r, s = run(scores, evicted)
        assert torch.equal(r, ret) and torch.equal(s, snap)
    assert torch.equal(plain[:n], odd[1:]) and plain[n] == -7.0 and odd[0] == -7.0
    assert float(plain[:n].min()) >= 0.0
