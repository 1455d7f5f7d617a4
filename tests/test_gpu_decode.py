"""Parity of the decode-side consumer (nkv_decode_attention, through the C ABI) against oracle/decode.py.

The cache a test feeds to both sides never comes from the HIP path: small cases take the CPU oracle's own
compression of a seeded workload, the full-size case a synthetic ragged cache drawn by nkv_inputs.

Bar: |out - oracle| <= DECODE_TOL * max(1, max|V|) and |lse - oracle| <= DECODE_TOL * max(1, |lse|).  The
kernel forms <q, k> from exact bf16 products accumulated in fp32 (d terms, rounding ~ sqrt(d) ulp of the
logit, logits of a few tens at most -> ~1e-5 absolute in the exponent at worst), uses the hardware's base-2
exponential (1 ulp) and fp32 running sums over the rows; the output is a convex combination of value rows,
so a relative weight error e gives at most e * max|V|.
"""
import numpy as np
import pytest
import torch

import nkv_inputs
import oracle
from oracle.decode import decode_attention as oracle_decode
import paper_2605_26678_amd as nkv
from parity_util import oracle_params, shape_of

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
DECODE_TOL = 1e-5


def _f64(t):
    return t.detach().to(torch.float32).cpu().numpy().astype(np.float64)


def _run(w, q, pk, pv, head_off, rows, Hq, scale, want_lse=True):
    shape, params = shape_of(w), nkv.params_default()
    P = len(w.prompt_lens)
    ws = torch.empty(max(nkv.decode_workspace_bytes(shape, Hq, rows), 256), dtype=torch.uint8, device=DEV)
    out = torch.full((P, w.L, Hq, w.d_v), float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full((P, w.L, Hq), float("nan"), dtype=torch.float32, device=DEV) if want_lse else None
    nkv.decode_attention(q, pk, pv, head_off, rows, shape, params, Hq, scale, out, lse, ws)
    torch.cuda.synchronize()
    return out, lse


def _records(w, q, pk, pv, head_off, rows, G, scale):
    """Which partial results a call of the kernels with scratch leaves there, by number: nothing else is written behind the
    units' words in front.  The call's output too."""
    n = len(w.prompt_lens) * w.L * w.H
    shape = shape_of(w)
    front = (4 * (n + 1) + 255) // 256 * 256
    record = G * (w.d + 2)
    ws = torch.full((nkv.decode_workspace_bytes(shape, G * w.H, rows),), 255, dtype=torch.uint8, device=DEV)
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full(q.shape[:3], float("nan"), dtype=torch.float32, device=DEV)
    nkv.decode_attention(q, pk, pv, head_off, rows, shape, nkv.params_default(), G * w.H, scale, out, lse, ws)
    torch.cuda.synchronize()
    words = ws[front:].view(torch.int32)
    words = words[:words.numel() // record * record].reshape(-1, record)
    return (words[:, 0] != -1).nonzero()[:, 0].cpu().numpy(), out, lse


def _check(out, lse, o_out, o_lse, vmax, what):
    err = np.abs(out.cpu().numpy().astype(np.float64) - o_out).max()
    assert err <= DECODE_TOL * max(1.0, vmax), f"{what}: out off by {err:.3e}"
    if lse is not None:
        g = lse.cpu().numpy().astype(np.float64)
        fin = np.isfinite(o_lse)
        assert np.array_equal(np.isneginf(g), np.isneginf(o_lse)), what
        e2 = np.abs(g[fin] - o_lse[fin]) / np.maximum(1.0, np.abs(o_lse[fin]))
        assert e2.size == 0 or e2.max() <= DECODE_TOL, f"{what}: lse off by {e2.max():.3e}"
    return err


CASES = [
    # name, L, H, d, dv, lens, dtype, Hq, r
    ("qwen_like_g4", 2, 2, 128, 0, [1500, 300], "bf16", 8, 0.5),
    ("llama1b_like_d64_g4", 1, 2, 64, 0, [1100], "bf16", 8, 0.5),
    ("llama3b_like_g3", 1, 2, 128, 0, [900], "bf16", 6, 0.75),
    ("mha_g1", 1, 3, 128, 0, [700], "bf16", 3, 0.5),
    ("g8", 1, 1, 64, 0, [800], "bf16", 8, 0.25),
    ("keep_all", 1, 2, 128, 0, [513, 256], "bf16", 4, 0.0),
    ("keep_none", 1, 2, 128, 0, [300], "bf16", 4, 1.0),
    ("generic_fp32", 1, 2, 64, 0, [400], "fp32", 4, 0.5),
    ("generic_dv_differs", 1, 2, 128, 64, [500], "bf16", 4, 0.5),
    ("generic_d40", 1, 2, 40, 24, [300], "fp32", 2, 0.5),
    ("generic_g12", 1, 1, 64, 0, [300], "bf16", 12, 0.5),
    ("fp16_g4", 1, 2, 128, 0, [1500, 300], "fp16", 8, 0.5),
    ("fp16_d64_g2", 1, 2, 64, 0, [600], "fp16", 4, 0.5),
    ("generic_fp16_dv", 1, 2, 128, 64, [600], "fp16", 4, 0.5),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_decode_over_the_oracles_compressed_cache(case):
    name, L, H, d, dv, lens, dtype, Hq, r = case
    w = nkv_inputs.small_workload(name, L, H, d, lens, dtype=dtype, dv=dv)
    K, V = nkv_inputs.make_kv(w, "cpu")
    raw = torch.int32 if dtype == "fp32" else torch.int16
    comp = oracle.compress(K.float().numpy(), K.view(raw).numpy(), V.view(raw).numpy(), w.cu_seqlens,
                           [r] * len(lens), oracle_params(nkv.params_default()))
    pk = torch.from_numpy(comp.packed_k).view(K.dtype)
    pv = torch.from_numpy(comp.packed_v).view(V.dtype)
    head_off = torch.from_numpy(comp.head_off)
    rows = int(head_off[-1])
    q = nkv_inputs.make_queries(w, Hq, K)
    scale = 1.0 / np.sqrt(d)
    o_out, o_lse = oracle_decode(_f64(q), _f64(pk), _f64(pv), comp.head_off, H, scale)
    if rows == 0:                                        # nothing kept: the buffers may be empty
        pk, pv = torch.zeros(1, d, dtype=K.dtype), torch.zeros(1, w.d_v, dtype=V.dtype)
    out, lse = _run(w, q.to(DEV), pk.to(DEV), pv.to(DEV), head_off.to(DEV), rows, Hq, scale)
    err = _check(out, lse, o_out, o_lse, float(_f64(pv).__abs__().max()), name)
    print(f"\n[{name}] rows {rows}, worst |out - oracle| {err:.2e}")


def test_chunk_boundaries_empty_units_and_clamped_offsets():
    """Unit lengths around the 256-row chunk size, an empty unit in the middle, and a cache that holds fewer
    rows than head_off claims (entries are clamped to `rows`)."""
    lens = [1, 255, 256, 257, 0, 512, 513, 3]
    w = nkv_inputs.small_workload("edges", 2, 4, 128, [600])
    K, V = nkv_inputs.make_kv(w, "cpu")
    L = torch.tensor(lens, dtype=torch.int64).reshape(1, 2, 4)
    pk, pv, head_off = nkv_inputs.synthetic_cache(w, K, V, L)
    q = nkv_inputs.make_queries(w, 16, K)
    for rows in (int(head_off[-1]), 1000):
        ho = head_off.numpy().clip(max=rows)
        o_out, o_lse = oracle_decode(_f64(q), _f64(pk[:rows]), _f64(pv[:rows]), ho, 4, 0.1)
        out, lse = _run(w, q.to(DEV), pk[:rows].to(DEV).contiguous(), pv[:rows].to(DEV).contiguous(),
                        head_off.to(DEV), rows, 16, 0.1)
        _check(out, lse, o_out, o_lse, float(_f64(pv).__abs__().max()), f"edges rows={rows}")
    out2, _ = _run(w, q.to(DEV), pk.to(DEV), pv.to(DEV), head_off.to(DEV), int(head_off[-1]), 16, 0.1, want_lse=False)
    assert torch.isfinite(out2).all()


def test_decode_is_deterministic():
    w = nkv_inputs.small_workload("det", 1, 2, 128, [3000])
    K, V = nkv_inputs.make_kv(w, DEV)
    lens = nkv_inputs.synthetic_head_lengths(w, 0.5)
    pk, pv, head_off = nkv_inputs.synthetic_cache(w, K, V, lens)
    q = nkv_inputs.make_queries(w, 8, K)
    a, la = _run(w, q, pk, pv, head_off, pk.shape[0], 8, 0.09)
    b, lb = _run(w, q, pk, pv, head_off, pk.shape[0], 8, 0.09)
    assert torch.equal(a, b) and torch.equal(la, lb)


def test_headline_size_cache_sampled_units():
    """The launch configuration the benchmark times (36 x 8 heads, 32k-token prompt, a quarter retained,
    32 query heads): every output is computed, the oracle checks sampled (layer, query head) pairs."""
    w = nkv_inputs.WORKLOADS["qwen4b_32k"]
    K, V = nkv_inputs.make_kv(w, DEV)
    lens = nkv_inputs.synthetic_head_lengths(w, 0.75)
    assert int(lens.sum()) == w.L * w.H * 8192 and int(lens.min()) < int(lens.max())
    pk, pv, head_off = nkv_inputs.synthetic_cache(w, K, V, lens)
    Hq, G = 32, 4
    q = nkv_inputs.make_queries(w, Hq, K)
    scale = 1.0 / np.sqrt(w.d)
    out, lse = _run(w, q, pk, pv, head_off, pk.shape[0], Hq, scale)
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
    ho = head_off.cpu().numpy()
    rng = np.random.default_rng(0)
    worst = 0.0
    for l, j in [(0, 0), (35, 31)] + [(int(rng.integers(36)), int(rng.integers(32))) for _ in range(10)]:
        u = l * w.H + j // G
        a, b = int(ho[u]), int(ho[u + 1])
        o_out, o_lse = oracle_decode(_f64(q[:, l:l + 1, j:j + 1]), _f64(pk[a:b]), _f64(pv[a:b]), np.array([0, b - a]),
                                     1, scale)
        worst = max(worst, _check(out[:, l:l + 1, j:j + 1], lse[:, l:l + 1, j:j + 1], o_out, o_lse,
                                  float(pv[a:b].abs().max()), f"layer {l} query head {j}"))
    print(f"\n[decode qwen4b_32k] rows {pk.shape[0]}, sampled worst |out - oracle| {worst:.2e}")


@pytest.mark.parametrize("d,G,dtype", [(64, 8, "bf16"), (128, 3, "fp16"), (64, 1, "fp16"), (128, 5, "bf16")])
@pytest.mark.parametrize("lens", [[63, 64, 65, 0], [255, 256, 257, 1], [8000, 3, 0, 0], [20000, 20000, 20000, 65536]])
def test_chunk_sizes_of_few_and_many_rows(d, G, dtype, lens):
    """Units around the chunk lengths of a call with few rows (64) and with many (256, the last case), empty units at
    either end; and the same call with scratch for chunks of 256 rows only, as an earlier size query may have given."""
    H = 2
    w = nkv_inputs.small_workload(f"chunks_{d}_{G}", 1, H, d, [1] * (len(lens) // H), dtype=dtype, n_out=0)
    g = torch.Generator().manual_seed(sum(lens) + d)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    rows = sum(lens)
    off = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64)
    pk, pv = (torch.randn(rows, d, generator=g).to(dt).to(DEV) for _ in range(2))
    q = torch.randn(len(w.prompt_lens), 1, H * G, d, generator=g).to(dt).to(DEV)
    scale = 1.0 / float(np.sqrt(d))
    want, want_lse = oracle_decode(_f64(q), _f64(pk), _f64(pv), off.numpy(), H, scale)
    shape, p = shape_of(w), nkv.params_default()
    part_off = (4 * (len(lens) + 1) + 255) // 256 * 256
    least = part_off + (rows // 256 + len(lens)) * G * (d + 2) * 4
    for nbytes in (max(nkv.decode_workspace_bytes(shape, H * G, rows), 256), least):
        ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        out = torch.full(want.shape, float("nan"), dtype=torch.float32, device=DEV)
        lse = torch.full(want_lse.shape, float("nan"), dtype=torch.float32, device=DEV)
        nkv.decode_attention(q, pk, pv, off.to(DEV), rows, shape, p, H * G, scale, out, lse, ws)
        torch.cuda.synchronize()
        assert np.abs(_f64(out) - want).max() <= DECODE_TOL * max(1.0, float(pv.abs().max()))
        got, has = _f64(lse), np.isfinite(want_lse)
        assert np.array_equal(np.isfinite(got), has)
        assert (np.abs(got[has] - want_lse[has]) <= DECODE_TOL * np.maximum(1.0, np.abs(want_lse[has]))).all()


@pytest.mark.parametrize("units,G,rows", [(1, 1, 2000), (1, 8, 40000), (8, 8, 8192), (256, 1, 300), (256, 8, 16), (256, 5, 130),
                                          (257, 3, 70), (128, 8, 300), (64, 3, 2000)])
def test_both_chunk_lengths_and_both_ways_to_combine(units, G, rows):
    """Calls on either side of the rules for the chunks' length (few units, few rows, as many workgroups as the chip holds for
    G query heads) and for the threads that combine a unit's chunks; uneven units, one of them empty."""
    H, d = (8, 64) if units % 8 == 0 else (1, 128)
    w = nkv_inputs.small_workload(f"combine_{units}_{G}_{rows}", units // H, H, d, [64], n_out=0)
    g = torch.Generator().manual_seed(units * 1000 + rows)
    lens = (torch.rand(units, generator=g) * 2.0 * rows).long()
    lens[units // 2] = 0 if units > 1 else rows
    off = torch.zeros(units + 1, dtype=torch.int64)
    off[1:] = lens.cumsum(0)
    n = int(off[-1])
    pk, pv = (torch.randn(n, d, generator=g).to(torch.bfloat16).to(DEV) for _ in range(2))
    q = torch.randn(1, units // H, H * G, d, generator=g).to(torch.bfloat16).to(DEV)
    scale = 1.0 / float(np.sqrt(d))
    want, want_lse = oracle_decode(_f64(q), _f64(pk), _f64(pv), off.numpy(), H, scale)
    shape = shape_of(w)
    out = torch.full(want.shape, float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full(want_lse.shape, float("nan"), dtype=torch.float32, device=DEV)
    ws = torch.empty(max(nkv.decode_workspace_bytes(shape, H * G, n), 256), dtype=torch.uint8, device=DEV)
    nkv.decode_attention(q, pk, pv, off.to(DEV), n, shape, nkv.params_default(), H * G, scale, out, lse, ws)
    torch.cuda.synchronize()
    assert np.abs(_f64(out) - want).max() <= DECODE_TOL * max(1.0, float(pv.abs().max()))
    got, has = _f64(lse), np.isfinite(want_lse)
    assert np.array_equal(np.isfinite(got), has)
    assert (np.abs(got[has] - want_lse[has]) <= DECODE_TOL * np.maximum(1.0, np.abs(want_lse[has]))).all()


UNIT_COST = 128                                                       # rows' room that a unit takes in a stretch


def _stretch_length(rows, units, d, G):
    """Rows of a stretch, and how many stretches a call of that many rows and units is cut into."""
    resident = 256 * ((8 if d == 128 else 4) if G == 1 else 4 if G == 2 else 3 if G <= 5 else 2)
    room = rows + UNIT_COST * units
    most = resident * min(max(room // (1024 * resident), 1), 4)
    return min(max(-(-(-(-room // most)) // 16) * 16, 192), 1 << 20), most


def _stretch_records(off, run):
    """The partial results that stretches of `run` rows leave: what stretch i holds of unit u is i + u."""
    found = set()
    for u in range(len(off) - 1):
        at, n = int(off[u] - off[0]) + UNIT_COST * (u + 1), int(off[u + 1] - off[u])
        if n > 0:
            found |= set(range(at // run + u, (at + n - 1) // run + u + 1))
    return found


def _piece_records(off, piece):
    return {int(off[u]) // piece + u + k for u in range(len(off) - 1) for k in range(-(-int(off[u + 1] - off[u]) // piece))}


def _ends_around_stretches(units, run, stretches):
    """Lengths of units whose first and last rows lie just before, at and behind multiples of `run`, units of 1 and no rows among them;
    the last unit takes the rest of `stretches` stretches."""
    lens, at = [], 0
    for u in range(units - 1):
        if u % 4 == 3:
            n = u // 4 % 2
        else:
            edge = ((at + UNIT_COST) // run + 1 + 3 * u % 5) * run + (u % 3 - 1)          # where the unit's last row ends ...
            n = edge - at - UNIT_COST * (1 + (u % 4 == 1))                              # ... or the next unit's first row lies
        lens.append(n)
        at += UNIT_COST + n
    return lens + [run * stretches - at - UNIT_COST]


@pytest.mark.parametrize("d,G,dtype,lens,piece", [
    (64, 8, "bf16", [70000, 0, 70001], 0),                           # units far longer than a stretch
    (64, 8, "bf16", _ends_around_stretches(120, 320, 512), 0),       # the first and last rows around a stretch's
    (128, 8, "fp16", _ends_around_stretches(150, 336, 512), 0),
    (128, 5, "fp16", _ends_around_stretches(170, 304, 768), 0),
    (64, 2, "fp16", _ends_around_stretches(200, 304, 1024), 0),
    (128, 1, "bf16", _ends_around_stretches(300, 288, 2048), 0),
    (64, 7, "fp16", [800] * 305 + [0, 1], 0),                        # three units to five workgroups: the last call by stretches
    (64, 7, "fp16", [800] * 308, 256),                               # and the first by pieces
    (64, 8, "fp16", [769] * 200, 0),                                 # more than three pieces a unit: the first call by stretches
    (64, 8, "fp16", [768] * 200, 256),                               # and the last by pieces
    (128, 6, "bf16", [1024] * 130 + [1] * 3, 0),
    (128, 3, "fp16", [0, 131072, 131071, 130, 1], 0),
    (64, 4, "bf16", [700] * 300, 256),
])
def test_stretches_across_units(d, G, dtype, lens, piece):
    """Calls large enough that every workgroup takes a stretch of the cache whichever units it holds, and calls on the other side of the
    lines that take pieces of 256 rows: which partial results there are (a stretch's are not those of pieces), and the oracle's results.  Once
    more with offsets that claim more rows than the cache has."""
    w = nkv_inputs.small_workload(f"stretch_{d}_{G}_{len(lens)}", len(lens), 1, d, [1], dtype=dtype, n_out=0)
    g = torch.Generator().manual_seed(len(lens) + d)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    off = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64)
    full = int(off[-1])
    pk, pv = (torch.randn(full, d, generator=g).to(dt).to(DEV) for _ in range(2))
    q = torch.randn(1, len(lens), G, d, generator=g).to(dt).to(DEV)
    scale = 1.0 / float(np.sqrt(d))
    for rows in (full, full - 37 if lens[-1] > 300 and piece == 0 and lens[0] != 769 else full):
        ho = off.numpy().clip(max=rows)
        want, want_lse = oracle_decode(_f64(q), _f64(pk[:rows]), _f64(pv[:rows]), ho, 1, scale)
        records, out, lse = _records(w, q, pk[:rows], pv[:rows], off.to(DEV), rows, G, scale)
        _check(out, lse, want, want_lse, float(pv.abs().max()), f"stretches d={d} G={G} rows={rows}")
        expected = _piece_records(ho, piece) if piece else _stretch_records(ho, _stretch_length(rows, len(lens), d, G)[0])
        assert set(records.tolist()) == expected


def test_the_lengths_above_end_around_stretches():
    """The units that _ends_around_stretches makes do begin and end on both sides of a stretch's end, at the lengths that the call uses."""
    for units, run, stretches, d, G in ((120, 320, 512, 64, 8), (150, 336, 512, 128, 8), (170, 304, 768, 128, 5), (200, 304, 1024, 64, 2),
                                        (300, 288, 2048, 128, 1)):
        lens = _ends_around_stretches(units, run, stretches)
        assert min(lens) == 0 and 1 in lens and _stretch_length(sum(lens), units, d, G) == (run, stretches)
        ends = np.cumsum(np.array(lens) + UNIT_COST)
        firsts = ends - np.array(lens)
        assert {-1 % run, 0, 1} <= set((ends % run).tolist()) and {-1 % run, 0, 1} <= set((firsts % run).tolist())


@pytest.mark.parametrize("lens,G", [([40000] * 8, 4), ([300] * 300, 5), ([200] * 8, 2)])
def test_decode_captured_in_a_hip_graph(lens, G):
    """Long units, many short ones and a small call, recorded without a call in front and replayed with eager work in between:
    every replay gives the eager call's results bit for bit."""
    w = nkv_inputs.small_workload(f"decode_graph_{len(lens)}", len(lens), 1, 64, [1], dtype="fp16", n_out=0)
    g = torch.Generator().manual_seed(len(lens))
    rows = sum(lens)
    off = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64).to(DEV)
    pk, pv = (torch.randn(rows, 64, generator=g).to(torch.float16).to(DEV) for _ in range(2))
    q = torch.randn(1, len(lens), G, 64, generator=g).to(torch.float16).to(DEV)
    shape, p = shape_of(w), nkv.params_default()
    out = torch.zeros(1, len(lens), G, 64, dtype=torch.float32, device=DEV)
    lse = torch.zeros(1, len(lens), G, dtype=torch.float32, device=DEV)
    ws = torch.empty(max(nkv.decode_workspace_bytes(shape, G, rows), 256), dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        nkv.decode_attention(q, pk, pv, off, rows, shape, p, G, 0.125, out, lse, ws)
    want, want_lse = _run(w, q, pk, pv, off, rows, G, 0.125)
    for rep in range(3):
        out.zero_(), lse.zero_(), ws.fill_(255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(lse, want_lse), f"replay {rep}"


@pytest.mark.parametrize("G,d,dtype", [(4, 128, "bf16"), (8, 64, "fp16"), (1, 128, "fp16"), (3, 64, "bf16")])
def test_buffers_with_room_for_many_more_rows(G, d, dtype):
    """288 units of about 512 rows in buffers that hold 16 times as many (the rows behind them are not numbers): the oracle's
    results, and the work in stretches of a length that follows from the rows that are there."""
    lens = [448 + 128 * (u % 2) for u in range(288)]
    w = nkv_inputs.small_workload(f"room_{G}_{d}", 36, 8, d, [1], dtype=dtype, n_out=0)
    g = torch.Generator(device=DEV).manual_seed(G)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    off = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64)
    rows = int(off[-1])
    pk, pv = (torch.full((16 * rows, d), float("nan"), dtype=dt, device=DEV) for _ in range(2))
    for t in (pk, pv):
        t[:rows] = torch.randn(rows, d, generator=g, device=DEV).to(dt)
    q = torch.randn(1, 36, 8 * G, d, generator=g, device=DEV).to(dt)
    scale = 1.0 / float(np.sqrt(d))
    want, want_lse = oracle_decode(_f64(q), _f64(pk[:rows]), _f64(pv[:rows]), off.numpy(), 8, scale)
    spare, out, lse = _records(w, q, pk, pv, off.to(DEV), 16 * rows, G, scale)
    _check(out, lse, want, want_lse, float(pv[:rows].abs().max()), f"spare rows, G={G}")
    assert set(spare.tolist()) == _stretch_records(off.numpy(), _stretch_length(rows, len(lens), d, G)[0])


@pytest.mark.parametrize("d,G,dtype", [(128, 8, "bf16"), (64, 3, "fp16"), (128, 1, "fp16")])
def test_short_units_beside_a_long_one(d, G, dtype):
    """511 units of one row and one of 600 000: the oracle's results, and no workgroup takes more than 16 of the short units.  What
    stretch i holds of unit u is partial result i + u, and a unit of one row has one."""
    lens = [1] * 511 + [600000]
    w = nkv_inputs.small_workload(f"short_{G}_{d}", 64, 8, d, [1], dtype=dtype, n_out=0)
    g = torch.Generator(device=DEV).manual_seed(G)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    off = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64)
    rows = int(off[-1])
    pk, pv = (torch.randn(rows, d, generator=g, device=DEV).to(dt) for _ in range(2))
    q = torch.randn(1, 64, 8 * G, d, generator=g, device=DEV).to(dt)
    scale = 1.0 / float(np.sqrt(d))
    want, want_lse = oracle_decode(_f64(q), _f64(pk), _f64(pv), off.numpy(), 8, scale)
    records, out, lse = _records(w, q, pk, pv, off.to(DEV), rows, G, scale)
    _check(out, lse, want, want_lse, float(pv.abs().max()), f"short units, G={G}")
    assert len(records) > 512                                         # (pieces of 256 rows would number 511 + 2344)
    stretch = records[:511] - np.arange(511)
    assert stretch.min() == 0 and (np.diff(stretch) >= 0).all()
    assert np.bincount(stretch).max() <= 16


@pytest.mark.parametrize("rows_first", [0, 77])
@pytest.mark.parametrize("units,lens", [(1, [1000]), (8, [8192]), (63, [300, 0, 64, 1]), (64, [256, 0, 255]), (65, [257, 1, 0]),
                                        (255, [300, 0, 64, 1]), (256, [63, 65, 128, 0, 1]), (257, [256, 0, 255, 257, 1, 512]),
                                        (1024, [256]), (1024, [300, 0, 1]), (1025, [256, 511, 0, 513]), (2600, [256, 20])])
def test_every_piece_of_a_unit_is_some_workgroups(units, lens, rows_first):
    """Pieces of 64 and 256 rows that wavefronts (up to 64 units) or workgroups (up to 1024) find by counting all units' pieces or, of
    more units, by their numbers, behind rows that are no unit's: as many partial results as there are pieces, and the oracle's results."""
    lens = (lens * units)[:units]
    w = nkv_inputs.small_workload(f"pieces_{units}_{len(lens)}", units, 1, 64, [1], dtype="fp16", n_out=0)
    g = torch.Generator(device=DEV).manual_seed(units)
    off = torch.tensor(rows_first + np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int64)
    rows = int(off[-1])
    pk, pv = (torch.randn(rows, 64, generator=g, device=DEV).to(torch.float16) for _ in range(2))
    q = torch.randn(1, units, 2, 64, generator=g, device=DEV).to(torch.float16)
    want, want_lse = oracle_decode(_f64(q), _f64(pk), _f64(pv), off.numpy(), 1, 0.125)
    records, out, lse = _records(w, q, pk, pv, off.to(DEV), rows, 2, 0.125)
    _check(out, lse, want, want_lse, float(pv.abs().max()), f"{units} units")
    assert len(records) in [sum((n + piece - 1) // piece for n in lens) for piece in (64, 256)]


@pytest.mark.parametrize("units", [1024, 2560])
def test_units_of_whole_pieces_keep_every_xcd_busy(units):
    """Units of 256 rows, one piece each and room for two, take about as long as units of 255 (1.6 times as long where four of the
    eight XCDs had all the pieces).  The least of many replays of a graph of ten calls."""
    w = nkv_inputs.small_workload(f"xcds_{units}", units // 8, 8, 128, [1], n_out=0)
    g = torch.Generator(device=DEV).manual_seed(units)
    pk, pv = (torch.randn(256 * units, 128, generator=g, device=DEV).to(torch.bfloat16) for _ in range(2))
    q = torch.randn(1, units // 8, 64, 128, generator=g, device=DEV).to(torch.bfloat16)
    shape, p, took = shape_of(w), nkv.params_default(), {}
    out = torch.empty(q.shape, dtype=torch.float32, device=DEV)
    for n in (255, 256):
        rows, off = n * units, n * torch.arange(units + 1, dtype=torch.int64, device=DEV)
        ws = torch.empty(nkv.decode_workspace_bytes(shape, 64, rows), dtype=torch.uint8, device=DEV)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(10):
                nkv.decode_attention(q, pk[:rows], pv[:rows], off, rows, shape, p, 64, 0.1, out, None, ws)
        for _ in range(25):
            start, stop = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            graph.replay()
            stop.record()
            torch.cuda.synchronize()
            took[n] = min(took.get(n, 1e9), start.elapsed_time(stop))
    print(f"{units} units of 255 rows {100 * took[255]:.1f} us, of 256 {100 * took[256]:.1f}")
    assert took[256] < 1.25 * took[255]
