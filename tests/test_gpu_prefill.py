"""GPU parity: chunked prefill (through the C ABI) against the CPU oracle, mixed with decode steps."""
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


def _run(binding, oracle, schedule, *, B, H, Hkv, d, budget, n_sink, n_recent, seed=0, max_chunk=0, flags=0,
         units=None, kind="lowrank", dtype="bf16", scale=0.0, **gen_kw):
    T = sum(max(L, 1) for L in schedule)
    Q, K, V = inputs.batch_streams(kind, seed, T, B, Hkv, H // Hkv, d, dtype=dtype, **gen_kw)
    kv = binding.TreeKV(budget, H, d, kv_heads=Hkv, batch=B, dtype=dtype, n_sink=n_sink, n_recent=n_recent,
                        max_chunk=max_chunk, flags=flags, softmax_scale=scale)
    st = ph.run_schedule(oracle, kv, Q, K, V, schedule, dtype=dtype, units=units)
    st["score_err"] = ph.compare_scores(kv, st["results"], dtype)
    assert st["flagged"] <= max(2, st["decisions"] // 500), st["flagged"]
    print(f"  flagged={st['flagged']}/{st['decisions']} max_err={st['max_err']:.2e} score_err={st['score_err']:.2e}")
    return kv, st


def test_prefill_fill_then_evict_with_layout(binding, oracle):
    """Chunks that fill the cache, cross the budget, and span several sweeps of the scope index."""
    _run(binding, oracle, [40, 17, 64, 1, 100, 33, 128, 7], B=1, H=2, Hkv=2, d=128, budget=96, n_sink=2, n_recent=30,
         max_chunk=128)


def test_prefill_pure_algorithm1_many_sweeps(binding, oracle):
    """No protected tokens, tree region of 50 slots, chunks of up to 200 tokens: up to 5 sweeps per chunk."""
    _run(binding, oracle, [30, 200, 3, 150, 200, 49, 51], B=1, H=2, Hkv=2, d=128, budget=50, n_sink=0, n_recent=0,
         max_chunk=256, seed=4)


def test_prefill_interleaved_with_decode(binding, oracle):
    _run(binding, oracle, [0, 0, 20, 0, 64, 0, 0, 0, 70, 0, 5, 0], B=2, H=2, Hkv=2, d=128, budget=48, n_sink=1,
         n_recent=15, max_chunk=128, seed=6)


@pytest.mark.parametrize("G,d", [(4, 128), (2, 64), (8, 64)])
def test_prefill_grouped_queries(binding, oracle, G, d):
    _run(binding, oracle, [50, 90, 0, 128, 13], B=2, H=2 * G, Hkv=2, d=d, budget=72, n_sink=3, n_recent=20,
         max_chunk=128, seed=8)


@pytest.mark.parametrize("budget,n_sink,n_recent", [(1, 0, 0), (2, 0, 0), (3, 1, 1), (6, 0, 5), (6, 5, 0)])
def test_prefill_degenerate_budgets(binding, oracle, budget, n_sink, n_recent):
    _run(binding, oracle, [5, 1, 16, 0, 33], B=1, H=1, Hkv=1, d=64, budget=budget, n_sink=n_sink, n_recent=n_recent,
         max_chunk=64, seed=9, kind="iid")


def test_prefill_keep_left(binding, oracle):
    _run(binding, oracle, [64, 64, 10, 64], B=1, H=2, Hkv=2, d=128, budget=40, n_sink=0, n_recent=8, max_chunk=64,
         flags=binding.TREEKV_KEEP_LEFT, seed=10)


def test_prefill_large_budget_runs_in_place(binding, oracle):
    """A budget whose order arrays do not fit in LDS takes the replay kernel's in-place variant."""
    _run(binding, oracle, [1024] * 9 + [700, 0, 0], B=1, H=1, Hkv=1, d=64, budget=9000, n_sink=0, n_recent=0,
         max_chunk=1024, seed=13)


def test_prefill_len1_equals_decode(binding, oracle):
    """A one-token chunk is a decode step: same evictions, same retained list, outputs within tolerance."""
    import torch

    T, B, H, d, budget = 150, 1, 4, 128, 32
    Q, K, V = inputs.batch_streams("lowrank", 12, T, B, H, 1, d, dtype="bf16")
    a = binding.TreeKV(budget, H, d, kv_heads=H, batch=B, dtype="bf16", n_sink=2, n_recent=6, max_chunk=16)
    b = binding.TreeKV(budget, H, d, kv_heads=H, batch=B, dtype="bf16", n_sink=2, n_recent=6, max_chunk=16)
    Qd, Kd, Vd = (ph.to_device(x, "bf16") for x in (Q, K, V))
    oa, ra, na, ea = a.new_outputs()
    ob, rb, nb, eb = b.new_outputs(1)
    for t in range(T):
        a.decode_step(Qd[t], Kd[t], Vd[t], oa, ra, na, ea)
        b.prefill_chunk(Qd[t:t + 1].permute(1, 0, 2, 3).contiguous(), Kd[t:t + 1].permute(1, 0, 2, 3).contiguous(),
                        Vd[t:t + 1].permute(1, 0, 2, 3).contiguous(), 1, ob, rb, nb, eb)
        torch.cuda.synchronize()
        assert torch.equal(ea.flatten(), eb.flatten()) and torch.equal(ra, rb) and torch.equal(na, nb), t
        assert (oa - ob[:, 0]).abs().max().item() < 1e-4
    assert (a.scores() - b.scores()).abs().max().item() < 1e-3


@pytest.mark.parametrize("budget,free", [(400, f) for f in (127, 128, 129, 143, 255, 399)] +
                         [(2600, f) for f in (127, 128, 129, 143, 2559, 2560, 2575, 2599)])
@pytest.mark.parametrize("d", [64, 128])
def test_prefill_free_slot_at_a_tile_edge(binding, oracle, d, budget, free):
    """A full cache whose free slot lies at the edge of a 32-column block, of a 128-column tile or of a wave's 16 columns, in
    the last, partial one, or at the end: two tree slots, the right one of which the decode step frees (keep-left).  400
    slots: logits in registers, blocks of 32; 2600 slots, more than registers hold: two sweeps, tiles of 128."""
    _run(binding, oracle, [budget, 0, 130, 0, 64], B=1, H=2, Hkv=2, d=d, budget=budget, n_sink=free - 1,
         n_recent=budget - free - 1, max_chunk=budget, seed=24, flags=binding.TREEKV_KEEP_LEFT,
         units=None if budget == 400 else [(0, 1)])


@pytest.mark.parametrize("G,budget,n_sink,n_recent,schedule", [
    (8, 72, 3, 20, [50, 90, 0, 128, 13]),              # fewer slots than a 128-column tile
    (4, 130, 2, 40, [1, 63, 64, 65, 0, 127, 128]),     # row tiles of 64, a tile of the cache and two columns of the next
    (2, 127, 0, 0, [127, 1, 129, 0, 33]),
    (1, 400, 127, 271, [400, 0, 130, 0, 64]),          # the free slot at a tile's first column ..
    (1, 400, 142, 256, [400, 0, 130, 0, 64]),          # .. and inside a wave's 16 (keep-left)
])
def test_prefill_two_sweeps_many_heads(binding, oracle, G, budget, n_sink, n_recent, schedule):
    """320 query heads x 64: more row tiles than the kernel with its logits in registers is given at plain head_dim 64, so
    every one of these small caches is swept twice."""
    flags = binding.TREEKV_KEEP_LEFT if budget == 400 else 0
    _run(binding, oracle, schedule, B=2, H=160, Hkv=160 // G, d=64, budget=budget, n_sink=n_sink, n_recent=n_recent,
         max_chunk=max(schedule), seed=25, flags=flags, units=[(0, 0), (1, 160 // G - 1)])


@pytest.mark.parametrize("d,G,flag", [(64, 1, 0), (64, 4, 0), (128, 2, 0), (64, 2, 8), (128, 1, 8)])
def test_prefill_two_sweeps_ragged_chunks(binding, oracle, d, G, flag):
    """Chunk lengths around the 64-row and 128-column tiles into a cache of 2600 slots, nearly empty, at its budget, evicting."""
    assert flag in (0, binding.TREEKV_POSITION_RERANK)
    _run(binding, oracle, [1, 63, 64, 65, 127, 0, 129, 191, 1901, 128, 63, 0, 65, 129, 1], B=1, H=2 * G, Hkv=2, d=d, budget=2600,
         n_sink=3, n_recent=900, max_chunk=1901, seed=26, flags=flag, units=[(0, 1)])


@pytest.mark.parametrize("G", [1, 4])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rerank", [False, True])
def test_prefill_both_attend_kernels_agree(binding, d, rerank, G):
    """The same chunks into 520 slots (logits in registers) and into 2600 (two sweeps) while both fill.  What may differ: a
    probability's exponent (below 2^8) is rounded to 2^-16, a few times that is 1e-4 of its value and of the scores, which
    add them up; for the outputs, the halves of P leave out up to 2^-16 of a probability more on either side."""
    import torch

    lengths = [1, 31, 32, 33, 2, 63, 30, 129, 64, 100, 3, 32]
    assert sum(lengths) == 520
    Q, K, V = (ph.to_device(x, "bf16").transpose(0, 1) for x in
               inputs.batch_streams("lowrank", 27, 520, 2, 3, G, d, dtype="bf16"))
    flags = binding.TREEKV_POSITION_RERANK if rerank else 0
    small, large = (binding.TreeKV(c, 3 * G, d, kv_heads=3, batch=2, dtype="bf16", n_sink=2, n_recent=100, max_chunk=129,
                                   flags=flags) for c in (520, 2600))
    at = 0
    for n in lengths:
        x = [t[:, at:at + n].contiguous() for t in (Q, K, V)]
        a, b = small.new_outputs(n), large.new_outputs(n)
        small.prefill_chunk(*x, n, *a)
        large.prefill_chunk(*x, n, *b)
        at += n
        err = (a[0] - b[0]).abs().max().item()
        assert err <= V.abs().max().item() * (1e-4 + 2.0 ** -15), (n, err)
        torch.testing.assert_close(small.scores()[..., :at], large.scores()[..., :at], rtol=1e-4, atol=1e-9)


@pytest.mark.parametrize("d,rerank,G,budget,schedule", [
    (128, False, 1, 31, [31, 32, 33, 1]),              # blocks and row tiles of 32: exact, one over, one under
    (128, False, 2, 64, [64, 64, 95, 0, 97]),
    (128, True, 1, 96, [40, 56, 33, 0, 31]),
    (64, False, 1, 255, [200, 55, 64, 32, 0, 5]),      # eight waves, one block each and one less
    (64, True, 2, 257, [257, 40, 3]),
    (128, False, 1, 2048, [512, 512, 512, 512, 512, 31]),    # 80 blocks: all that registers hold
    (128, True, 1, 2016, [512, 512, 512, 480, 512, 512]),
    (128, False, 1, 2049, [512, 512, 512, 512, 512, 512]),   # one slot more: the two-sweep kernel, except for a shorter chunk
    (64, False, 1, 2049, [512, 512, 512, 512, 480, 512]),
])
def test_prefill_logits_in_registers(binding, oracle, d, rerank, G, budget, schedule):
    """Edges of the 32-column blocks, of the 32-row tiles and of what a workgroup's registers hold."""
    flags = binding.TREEKV_POSITION_RERANK if rerank else 0
    _run(binding, oracle, schedule, B=1, H=2 * G, Hkv=2, d=d, budget=budget, n_sink=min(2, budget // 4),
         n_recent=budget // 3, max_chunk=512, seed=11, flags=flags, units=[(0, 1)])


@pytest.mark.parametrize("d,dtype,schedule", [
    (128, "bf16", [64, 65, 128, 129, 256, 257]),       # 16-byte pieces of a row times tokens around 1, 2 and 4 x 1024
    (64, "bf16", [128, 129, 256, 257, 512, 511]),
    (64, "f32", [64, 65, 128, 129, 256, 257]),
    (128, "f32", [32, 33, 64, 65, 128, 129]),
])
def test_prefill_rows_copied_by_the_replay(binding, oracle, d, dtype, schedule):
    """Chunk lengths around those at which a thread of the replay holds one more piece, or the scatter kernel takes over."""
    kind = "lowrank" if dtype == "bf16" else "iid"
    _run(binding, oracle, schedule, B=2, H=2, Hkv=2, d=d, budget=150, n_sink=2, n_recent=60, max_chunk=512, seed=3,
         dtype=dtype, kind=kind, units=[(0, 1), (1, 0)])


def test_prefill_argument_errors(binding):
    import torch

    kv = binding.TreeKV(32, 2, 128, max_chunk=64)
    out, ret, nret, ev = kv.new_outputs(8)
    x = torch.zeros(1, 80, 2, 128, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(binding.TreeKVError):
        kv.prefill_chunk(x, x, x, 65, out, ret, nret, ev)          # longer than max_chunk
    with pytest.raises(binding.TreeKVError):
        kv.prefill_chunk(x, x, x, 0, out, ret, nret, ev)
    big = binding.TreeKV(10000, 2, 64, kv_heads=2, dtype="f32", n_sink=0, n_recent=0, max_chunk=512)
    xf = torch.zeros(1, 512, 2, 64, dtype=torch.float32, device="cuda")
    outf, retf, nretf, evf = big.new_outputs(512)
    with pytest.raises(binding.TreeKVError) as e:
        big.prefill_chunk(xf, xf, xf, 512, outf, retf, nretf, evf)  # fp32 storage: more columns than the fp32 path takes
    assert e.value.status == binding.TREEKV_EUNSUPPORTED


def test_prefill_gather_kv_matches_retained(binding, oracle):
    """After chunks and decode steps the compacted cache (treekv_gather_kv) holds exactly the rows of the retained
    positions: surviving chunk rows were scattered into the right freed slots."""
    import torch

    sched = [40, 100, 0, 64, 0, 0, 90]
    T = sum(max(L, 1) for L in sched)
    B, H, d, budget = 2, 2, 128, 56
    Q, K, V = inputs.batch_streams("lowrank", 31, T, B, H, 1, d, dtype="bf16")
    kv = binding.TreeKV(budget, H, d, kv_heads=H, batch=B, dtype="bf16", n_sink=3, n_recent=13, max_chunk=128)
    st = ph.run_schedule(oracle, kv, Q, K, V, sched, dtype="bf16")     # retained lists compared call by call
    Kc, Vc = kv.gather_kv()
    torch.cuda.synchronize()
    for (b, h), res in st["results"].items():
        pos = res["stream"].retained()
        np.testing.assert_array_equal(Kc[b, h, :len(pos)].float().cpu().numpy(), K[pos, b, h])
        np.testing.assert_array_equal(Vc[b, h, :len(pos)].float().cpu().numpy(), V[pos, b, h])


def test_prefill_accumulated_weight_criterion(binding, oracle):
    _run(binding, oracle, [40, 64, 0, 128, 0, 0, 77, 5], B=1, H=4, Hkv=2, d=128, budget=72, n_sink=2, n_recent=20,
         max_chunk=128, flags=binding.TREEKV_SCORE_ACCUMULATED, seed=23)


@pytest.mark.parametrize("G,d", [(1, 64), (2, 128), (4, 64)])
def test_prefill_fp32_storage(binding, oracle, G, d):
    """fp32 storage: the chunk's attention runs on the fp32 matrix instructions and is held to 1e-5;
    chunks that fill, cross the budget and span sweeps, decode steps in between, ragged lengths."""
    _run(binding, oracle, [40, 17, 64, 1, 0, 100, 33, 0, 0, 128, 7], B=2, H=2 * G, Hkv=2, d=d, budget=96, n_sink=2,
         n_recent=30, max_chunk=128, seed=14, kind="iid", dtype="f32")


def test_prefill_fp32_tiny_configuration_in_chunks(binding, oracle):
    """The tiny fp32 configuration (2 heads x 64, budget 64, 512 tokens, K carrying the 1/sqrt(64)) fed as chunks."""
    _run(binding, oracle, [64] * 7 + [63, 1], B=1, H=2, Hkv=2, d=64, budget=64, n_sink=4, n_recent=28, max_chunk=64,
         seed=0, kind="iid", dtype="f32", scale=1.0, k_scale=0.125)


def test_prefill_fp32_degenerate_and_keep_left(binding, oracle):
    _run(binding, oracle, [5, 1, 16, 0, 33], B=1, H=1, Hkv=1, d=64, budget=3, n_sink=1, n_recent=1, max_chunk=64,
         seed=15, kind="iid", dtype="f32")
    _run(binding, oracle, [30, 30, 10, 30], B=1, H=2, Hkv=2, d=128, budget=40, n_sink=0, n_recent=8, max_chunk=32,
         flags=binding.TREEKV_KEEP_LEFT | binding.TREEKV_SCORE_ACCUMULATED, seed=16, kind="iid", dtype="f32")


@pytest.mark.parametrize("d,budget,schedule", [
    (64, 47, [1, 15, 16, 17, 33, 0, 48, 31]),            # row tiles and column blocks of 16, one short, exact, one over
    (128, 127, [127, 1, 2, 129, 0, 16]),                 # fills to one slot short of the budget, then over it
    (64, 2060, [2033, 15, 40, 0, 17]),                   # 2048 columns are parked in LDS; more are formed twice
])
def test_prefill_fp32_tile_edges(binding, oracle, d, budget, schedule):
    _run(binding, oracle, schedule, B=1, H=2, Hkv=1, d=d, budget=budget, n_sink=1, n_recent=budget // 3,
         max_chunk=max(schedule), seed=17, kind="iid", dtype="f32")


@pytest.mark.parametrize("d,n0", [(64, 50), (128, 48), (64, 2060)])
def test_prefill_fp32_non_finite_rows_stay_their_own(binding, d, n0):
    """A token whose v holds an infinity or a NaN reaches the rows that see it and no other, and a query of NaNs spoils
    the scores of the tokens it sees and no other's.  (Column blocks at, inside and past the end of a row tile; at
    2060 cached tokens the logits of the chunk's columns are formed twice.)"""
    import torch

    L, H, inf_at, nan_at, bad_query = 40, 2, 20, 39, 10
    g = torch.Generator(device="cuda").manual_seed(d + n0)
    Q, K, V = (torch.randn(1, n0 + L, H, d, device="cuda", generator=g) for _ in range(3))

    def run(q, v):
        kv = binding.TreeKV(n0 + L + 8, H, d, kv_heads=H, dtype="f32", n_sink=2, n_recent=8, max_chunk=1024)
        for a in list(range(0, n0, 1024)) + [n0]:
            b = min(a + 1024, n0) if a < n0 else n0 + L
            res = kv.new_outputs(b - a)
            kv.prefill_chunk(q[:, a:b].contiguous(), K[:, a:b].contiguous(), v[:, a:b].contiguous(), b - a, *res)
        scores = kv.scores()
        torch.cuda.synchronize()
        return res[0][0].cpu(), scores[0, :, n0:n0 + L].cpu()

    want, want_s = run(Q, V)
    q, v = Q.clone(), V.clone()
    v[:, n0 + inf_at, :, 3] = float("inf")
    v[:, n0 + nan_at, :, 5] = float("nan")
    q[:, n0 + bad_query] = float("nan")
    got, got_s = run(q, v)
    want[inf_at:, :, 3] = float("inf")
    want[nan_at:, :, 5] = float("nan")
    rows = [i for i in range(L) if i != bad_query]
    torch.testing.assert_close(got[rows], want[rows], rtol=1e-5, atol=1e-5, equal_nan=True)
    assert torch.isnan(got[bad_query]).all()
    torch.testing.assert_close(got_s[:, bad_query + 1:], want_s[:, bad_query + 1:], rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rerank", [False, True])
@pytest.mark.parametrize("rise", [0, 20, 40, 60, 100])
@pytest.mark.parametrize("budget", [512, 2600])
def test_prefill_rows_whose_logits_rise(binding, d, rerank, rise, budget):
    """Keys of the second tile lie `rise` (in log2) above those of the first: what a row's sums are taken against changes
    on the way.  One query per head, so a token's score is its probability, and a head's scores add up to one but for the
    error of the normaliser.
    2600 slots, two sweeps: the reference is raised at 2^16 only, the normaliser is log2(sum).  Bound, in log2 units:
    log2(sum) <= 8 is rounded twice (2 * 2^-22, and the same for its own instruction), times ln 2 = 6e-7; the sums' own
    rounding is some 2^-23.  A reference left 40 or 60 below the logits rounds log2(sum) and the exponentials' arguments to
    2^-19.
    512 slots, logits in registers: every block of 32 columns has its own reference and is brought to the row's by one
    exponential, its part of the sum by up to three (from block to block, between the lanes and between the waves), then
    1/sum: five roundings of 2^-23 beside those of the sums, 7e-7."""
    import torch

    H, n0 = 64, 256
    g = torch.Generator(device="cuda").manual_seed(rise)
    logit = torch.rand(n0 + 1, H, device="cuda", generator=g) * 3 - 3
    logit[:128] -= rise
    # all of it in one plane whose angles vanish at this base: re-assigned positions then leave the logits as they are
    K = torch.zeros(1, n0 + 1, H, d, dtype=torch.bfloat16, device="cuda")
    Q = torch.zeros_like(K)
    K[0, :, :, d - 2] = (logit / 8).to(torch.bfloat16)
    Q[..., d - 2] = 8
    V = torch.randn(1, n0 + 1, H, d, device="cuda", generator=g).to(torch.bfloat16)
    scale = 0.7                                               # (not ln 2: with it the exponents would be exact)
    kv = binding.TreeKV(budget, H, d, kv_heads=H, n_sink=2, n_recent=8, softmax_scale=scale, rope_base=1e38,
                        flags=binding.TREEKV_POSITION_RERANK if rerank else 0)
    kv.prefill_chunk(Q[:, :n0].contiguous(), K[:, :n0].contiguous(), V[:, :n0].contiguous(), n0, *kv.new_outputs(n0))
    snap, lay = kv.export_state(), kv.state_layout()
    snap[lay.S:lay.S + H * budget * 4] = 0
    kv.import_state(snap)
    out = kv.new_outputs(1)
    kv.prefill_chunk(Q[:, n0:].contiguous(), K[:, n0:].contiguous(), V[:, n0:].contiguous(), 1, *out)
    got = kv.scores()[0, :, :n0 + 1].double().cpu().numpy()
    s = np.float64(np.float32(scale)) * 8 * K[0, :, :, d - 2].double().cpu().numpy().T
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    np.testing.assert_allclose(got, p, rtol=3e-6, atol=1e-9)
    total = np.abs(got.sum(-1) - 1).max()
    assert total < 1e-6, total
    want = np.einsum("hj,jhd->hd", p, V[0].double().cpu().numpy())
    np.testing.assert_allclose(out[0][0, 0].cpu().numpy(), want, rtol=1e-4, atol=1e-4)
