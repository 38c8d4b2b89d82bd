"""GPU parity of iflow_attn_decode (one decode step of grouped-query attention over an fp16 key/value cache) against the
plain definition in oracle/attention.py."""
import numpy as np
import pytest

from paper_2401_08294_amd import synth
from test_gpu_parity import TOL, gpu, say  # noqa: F401

pytestmark = pytest.mark.gpu


def dev16(torch, a16):
    return torch.from_numpy(np.ascontiguousarray(a16).view(np.int16)).cuda().view(torch.float16)


def rel(got, ref):
    rms = np.sqrt(np.mean(ref ** 2, axis=-1, keepdims=True))
    return float(np.max(np.abs(got - ref) / np.maximum(np.abs(ref), np.maximum(rms, 1e-30))))


def make(n_heads, n_kv, max_seq, seed, q_scale=1.0, d=128):
    rng = np.random.default_rng(seed)
    q = (q_scale * rng.standard_normal((n_heads, d))).astype(np.float16)
    k = rng.standard_normal((n_kv, max_seq, d)).astype(np.float16)
    v = rng.standard_normal((n_kv, max_seq, d)).astype(np.float16)
    return q, k, v


def run(torch, iflow, q, k, v, T, scale, ws=None):
    n_heads, n_kv, max_seq, d = q.shape[0], k.shape[0], k.shape[1], q.shape[1]
    nbytes = iflow.attn_decode_workspace_bytes(n_heads)
    if ws is None:
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")       # scratch: NaN patterns to start with
    out = torch.full((n_heads, d), float("nan"), dtype=torch.float16, device="cuda")
    iflow.attn_decode(dev16(torch, q), dev16(torch, k), dev16(torch, v), n_heads, n_kv, d, T, max_seq, scale, out, ws, nbytes)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64), ws


@pytest.mark.parametrize("n_heads,n_kv,T,max_seq", [(32, 32, 1, 64), (32, 32, 17, 64), (8, 8, 64, 64), (8, 4, 130, 200),
                                                    (32, 32, 1000, 1024), (64, 8, 777, 1024), (16, 4, 4096, 4096), (4, 1, 5000, 8192)])
def test_attention_decode_against_the_definition(gpu, n_heads, n_kv, T, max_seq):
    torch, iflow = gpu
    from oracle import attention as att
    say(f"[case] attention decode heads={n_heads} kv_heads={n_kv} seq_len={T} max_seq={max_seq}")
    q, k, v = make(n_heads, n_kv, max_seq, synth.BASE_SEED + 1500 + T)
    scale = 1.0 / np.sqrt(128.0)
    got, _ = run(torch, iflow, q, k, v, T, scale)
    ref = att.gqa_decode(q.view(np.uint16), k.view(np.uint16), v.view(np.uint16), T, scale)
    e = rel(got, ref)
    say(f"        max rel err {e:.3e}")
    assert np.isfinite(got).all() and e <= TOL


@pytest.mark.parametrize("n_heads,n_kv,d,T,max_seq", [
    (128, 8, 64, 1000, 1024),      # sixteen 64-component query heads per key/value head (the paper's Falcon-40B: Table 3, Table 5)
    (71, 1, 64, 777, 1024),        # multi-query attention: every head shares one key/value head (five pieces of sixteen heads)
    (32, 32, 64, 130, 200),        # multi-head attention at 64 components
    (16, 8, 64, 1, 64), (24, 8, 64, 65, 128), (40, 8, 64, 4096, 4096),       # groups of 2, 3 and 5 at 64 components
    (24, 8, 128, 300, 512), (48, 8, 128, 1000, 1024), (56, 8, 128, 129, 256), (128, 8, 128, 2049, 4096),   # groups of 3, 6, 7 and 16 at 128
    (40, 2, 128, 555, 1024), (33, 1, 128, 64, 64),                           # groups of 20 and 33: several pieces, the last ragged
])
def test_attention_other_head_dimensions_and_group_sizes(gpu, n_heads, n_kv, d, T, max_seq):
    """Section "Grouped-query attention": H heads in G groups, any ratio; head dimension 64 next to 128."""
    torch, iflow = gpu
    from oracle import attention as att
    say(f"[case] attention decode heads={n_heads} kv_heads={n_kv} head_dim={d} seq_len={T} max_seq={max_seq}")
    q, k, v = make(n_heads, n_kv, max_seq, synth.BASE_SEED + 1700 + T + n_heads, d=d)
    scale = 1.0 / np.sqrt(float(d))
    got, _ = run(torch, iflow, q, k, v, T, scale)
    ref = att.gqa_decode(q.view(np.uint16), k.view(np.uint16), v.view(np.uint16), T, scale)
    e = rel(got, ref)
    say(f"        max rel err {e:.3e}")
    assert np.isfinite(got).all() and e <= TOL


def test_attention_peaked_softmax_and_reused_workspace(gpu):
    """Large scores (one position dominates, the running maximum moves a lot) and several launches of different lengths
    on one workspace (left as the previous launch wrote it)."""
    torch, iflow = gpu
    from oracle import attention as att
    n_heads, n_kv, max_seq = 16, 8, 3000
    q, k, v = make(n_heads, n_kv, max_seq, synth.BASE_SEED + 1600, q_scale=6.0)
    ws = None
    for T in (3000, 65, 1, 2049, 3000):
        say(f"[case] attention, peaked scores, seq_len={T}, shared workspace")
        got, ws = run(torch, iflow, q, k, v, T, 0.5, ws)
        ref = att.gqa_decode(q.view(np.uint16), k.view(np.uint16), v.view(np.uint16), T, 0.5)
        e = rel(got, ref)
        assert np.isfinite(got).all() and e <= TOL, f"seq_len {T}: {e}"


def test_attention_one_workspace_for_different_head_counts(gpu):
    """One workspace, sized for the largest head count, serves launches of different head counts, group sizes and lengths
    one after the other with no host synchronization between them: stream order alone keeps a launch's partial results
    apart from the next one's."""
    torch, iflow = gpu
    from oracle import attention as att
    nbytes = iflow.attn_decode_workspace_bytes(64)
    ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
    scale = 1.0 / np.sqrt(128.0)
    cases = [(64, 8, 2000), (32, 32, 900), (8, 4, 1500), (64, 8, 1999), (16, 4, 2048), (32, 32, 901)]
    pending = []
    for n, (n_heads, n_kv, T) in enumerate(cases):
        say(f"[case] attention, shared workspace, heads={n_heads} kv_heads={n_kv} seq_len={T}")
        q, k, v = make(n_heads, n_kv, 2048, synth.BASE_SEED + 1650 + n)
        out = torch.full((n_heads, 128), float("nan"), dtype=torch.float16, device="cuda")
        iflow.attn_decode(dev16(torch, q), dev16(torch, k), dev16(torch, v), n_heads, n_kv, 128, T, 2048, scale, out, ws, nbytes)
        pending.append((q, k, v, T, out))
    torch.cuda.synchronize()
    for q, k, v, T, out in pending:
        ref = att.gqa_decode(q.view(np.uint16), k.view(np.uint16), v.view(np.uint16), T, scale)
        got = out.cpu().numpy().astype(np.float64)
        assert np.isfinite(got).all() and rel(got, ref) <= TOL, f"heads {q.shape[0]}, seq_len {T}"


def test_attention_graph_replay(gpu):
    torch, iflow = gpu
    from oracle import attention as att
    n_heads, n_kv, max_seq, T = 32, 8, 2048, 1500
    say("[case] attention under HIP-graph replay")
    q, k, v = make(n_heads, n_kv, max_seq, synth.BASE_SEED + 1700)
    qd, kd, vd = dev16(torch, q), dev16(torch, k), dev16(torch, v)
    nbytes = iflow.attn_decode_workspace_bytes(n_heads)
    ws = torch.zeros((nbytes,), dtype=torch.uint8, device="cuda")
    out = torch.zeros((n_heads, 128), dtype=torch.float16, device="cuda")
    stream = torch.cuda.Stream()
    scale = 1.0 / np.sqrt(128.0)
    with torch.cuda.stream(stream):
        iflow.attn_decode(qd, kd, vd, n_heads, n_kv, 128, T, max_seq, scale, out, ws, nbytes, stream=stream.cuda_stream)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            iflow.attn_decode(qd, kd, vd, n_heads, n_kv, 128, T, max_seq, scale, out, ws, nbytes, stream=stream.cuda_stream)
    for rep in range(3):
        q2 = make(n_heads, n_kv, 1, synth.BASE_SEED + 1710 + rep)[0]
        qd.copy_(dev16(torch, q2))
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        graph.replay()
        torch.cuda.synchronize()
        ref = att.gqa_decode(q2.view(np.uint16), k.view(np.uint16), v.view(np.uint16), T, scale)
        assert rel(out.cpu().numpy().astype(np.float64), ref) <= TOL


# around a block (16, 32 positions), a range (64), the lengths from which on a head's positions are shared out (256, 320, 352 and 384), and ranges of more than one block a wavefront
EDGES = [1, 15, 16, 17, 31, 33, 63, 64, 65, 96, 127, 129, 255, 256, 257, 319, 320, 321, 351, 352, 353, 383, 384, 385, 449, 2047, 2049, 2113]


@pytest.mark.parametrize("n_heads,n_kv,d", [(32, 32, 128), (8, 4, 128), (3, 1, 128), (32, 4, 128), (32, 2, 128), (5, 5, 64), (16, 2, 64), (18, 1, 64)])
def test_attention_edges(gpu, n_heads, n_kv, d):
    """Lengths at every edge; the cache's rows behind the last position are NaN and reach nothing; an infinite value at the last position makes its component
    infinite in every head, whatever of a block or of the merge's eight ranges lies past it.  Tolerance as above (fp32 sums, probabilities and output rounded to fp16 once: 2^-11 each)."""
    torch, iflow = gpu
    from oracle import attention as att
    q, k, v = make(n_heads, n_kv, max(EDGES) + 40, synth.BASE_SEED + 1800 + n_heads, d=d)
    scale = 1.0 / np.sqrt(float(d))
    for T in EDGES:
        say(f"[case] attention edges heads={n_heads} kv_heads={n_kv} head_dim={d} seq_len={T}")
        kt, vt = k[:, :T + 40].copy(), v[:, :T + 40].copy()
        kt[:, T:], vt[:, T:] = np.nan, np.nan
        got, _ = run(torch, iflow, q, kt, vt, T, scale)
        ref = att.gqa_decode(q.view(np.uint16), k[:, :T + 40].copy().view(np.uint16), v[:, :T + 40].copy().view(np.uint16), T, scale)
        assert np.isfinite(got).all() and rel(got, ref) <= TOL, f"seq_len {T}"
        vt[:, T - 1, 3] = np.inf
        got, _ = run(torch, iflow, q, kt, vt, T, scale)
        assert np.isposinf(got[:, 3]).all() and np.isfinite(np.delete(got, 3, 1)).all(), f"seq_len {T}"


@pytest.mark.parametrize("n_heads,n_kv,d", [(8, 8, 128), (6, 2, 128), (16, 2, 128), (16, 1, 128), (4, 2, 64), (16, 2, 64), (18, 1, 64)])
def test_infinite_value_with_a_small_weight(gpu, n_heads, n_kv, d):
    """An infinite value makes its component infinite as long as its weight is above 2^-25 of the largest so far, wherever the largest is: in the same block, in another wavefront's or
    in another range, before it or after; and it stays infinite where scores 2^120 as large come later.  (Scores are whole in units of log2 but for one rounding of the scale.)"""
    torch, iflow = gpu
    scale = float(np.log(2.0))
    for T in (40, 300, 900):
        rng = np.random.default_rng(synth.BASE_SEED + 1900 + T)
        q, k = np.zeros((n_heads, d), np.float16), np.zeros((n_kv, T, d), np.float16)
        q[:, 0] = 1.0
        v = rng.standard_normal((n_kv, T, d)).astype(np.float16)
        places = [(down, top, at) for down in (1.0, 7.0, 13.5, 20.0, 21.5, 22.25, 23.0, 24.0, 24.75) for top, at in ((0, 1), (T - 1, 3), (5, T - 1), (T // 2, 0))]
        places += [(120.0, T - 1, 3)] + ([(120.0, 261, 3)] if T > 261 else [])
        for down, top, at in places:
            say(f"[case] attention, infinite value heads={n_heads} kv_heads={n_kv} head_dim={d} seq_len={T} weight 2^-{down} at {at}, largest at {top}")
            k[:, :, 0] = 60.0 - down - 12.0 if down > 25 else 40.0
            k[:, top, 0] = 60.0
            k[:, at, 0] = 60.0 - down
            vt = v.copy()
            vt[:, at, 1], vt[:, at, d - 1] = np.inf, -np.inf
            got, _ = run(torch, iflow, q, k, vt, T, scale)
            assert np.isposinf(got[:, 1]).all() and np.isneginf(got[:, d - 1]).all() and np.isfinite(np.delete(got, (1, d - 1), 1)).all(), f"seq_len {T}, weight 2^-{down}"


@pytest.mark.parametrize("n_heads,n_kv,d,lengths", [(24, 8, 128, (129, 300, 9000)), (64, 8, 128, (129, 319, 9000)), (64, 4, 128, (300, 16001)), (10, 1, 128, (320, 20000)), (96, 32, 128, (310, 2113)),
                                                    (32, 8, 64, (129, 384, 9000)), (16, 1, 64, (300, 20000)), (6, 2, 128, (300, 6000)), (32, 32, 128, (200, 2000))])
def test_attention_scores_that_climb(gpu, n_heads, n_kv, d, lengths):
    """Scores that climb along the positions, block after block of a wavefront (128 positions apart) and inside a block, by 0 to 40 in units of log2 and by another step for every head, with
    the largest last, first and in the middle: the reference the sums are kept to follows in some heads of a block and not in others, lags by just less and just more than what it
    may (8: a block's maximum 15 above a reference that was 7 below the first one), and wavefronts and ranges are merged from references far apart.  Every third head has no noise, so that whole
    blocks share one score.  Tolerance as above: scores of up to 1500 (n_kv = 1) are rounded at 2^-24 of that, 1e-4 of a probability."""
    torch, iflow = gpu
    from oracle import attention as att
    q, k, v = make(n_heads, n_kv, max(lengths), synth.BASE_SEED + 2100 + n_heads + d, d=d)
    scale = 1.0 / np.sqrt(float(d))
    steps = np.array([0.0, 6.0, 7.9, 8.0, 8.1, 10.0, 14.9, 15.1, 20.0, 40.0, -6.0, -20.0, 3.0])
    q[::3] = 0.0
    for T in lengths:
        positions = np.arange(max(lengths))
        climbs = {"blocks of a wavefront": positions // 128, "blocks": positions // 32, "the middle": -np.abs(positions - T // 2) // 128, "positions": positions / 8.0}
        for name, climb in climbs.items():
            most = float(np.abs(climb[:T]).max())
            # (steps scaled down where the score would leave what 16 bits of key and query hold: 40 per block over 600 blocks)
            per = np.resize(steps, n_heads) * min(1.0, 1500.0 / (40.0 * max(most, 1.0))) if most * 40.0 > 1500.0 else np.resize(steps, n_heads)
            q[:, 0] = (per * np.log(2.0) / scale).astype(np.float16)
            k[:, :, 0] = climb.astype(np.float16)
            say(f"[case] attention, climbing scores ({name}) heads={n_heads} kv_heads={n_kv} head_dim={d} seq_len={T}")
            got, _ = run(torch, iflow, q, k[:, :T].copy(), v[:, :T].copy(), T, scale)
            ref = att.gqa_decode(q.view(np.uint16), k[:, :T].copy().view(np.uint16), v[:, :T].copy().view(np.uint16), T, scale)
            e = rel(got, ref)
            assert np.isfinite(got).all() and e <= TOL, f"{name}, seq_len {T}: {e:.2e}"
