"""GPU: sizes at the edges of the kernels' dispatch rules and of their inner blocking, against
the fp64 oracle and, where two routes must agree bit for bit, against each other."""
import numpy as np
import pytest
import torch

import paper_2604_16395_amd as s2l
import workloads
from tests.gpu_util import DEV, SCALE, Setup, assert_attention_close, to_bf16

pytestmark = pytest.mark.gpu


def _call(case, opts, fused):
    s = Setup(case)
    T, hq, hkv = case.total_tokens, case.num_q_heads, case.num_kv_heads
    ws = torch.empty(s2l.s2l_attn_workspace_bytes(s.batch, hq, hkv, opts), dtype=torch.uint8, device=DEV)
    s.plan = plan = s2l.s2l_attn_plan(s.batch, hq, hkv, ws, opts)
    out = torch.full((T, hq, 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    lse = torch.full((T, hq), float("nan"), dtype=torch.float32, device=DEV)
    if fused:
        assert s2l.s2l_append_chunk_prefill_attn(s.cache, s.batch, to_bf16(s.k_new), to_bf16(s.v_new), s.q, hq, SCALE,
                                                 out, lse, plan, ws)
    else:
        s.append()
        s2l.s2l_chunk_prefill_attn(s.cache, s.batch, s.q, hq, SCALE, out, lse, plan, ws)
    torch.cuda.synchronize()
    return s, out, lse


@pytest.mark.parametrize("layout", [(256, 1), (128, 1), (128, 2)])
@pytest.mark.parametrize("hq,hkv", [(2, 2), (7, 1), (96, 1)])
def test_fused_append_of_wide_tiles_and_odd_groups(hq, hkv, layout):
    """Tiles of up to 256 tokens (one head per kv head: more rows to append than a workgroup holds
    in flight), and group sizes that do not divide the tile (its last columns belong to no token),
    with the last tile one token long."""
    tq = layout[0] // (hq // hkv)
    case = workloads.make_case("append", [0, 64, 1024], [tq + 1, tq, 1], hq, hkv, seed=51)
    opts = s2l.plan_opts(tile_cols=layout[0], key_halves=layout[1])
    a, oa, la = _call(case, opts, True)
    b, ob, lb = _call(case, opts, False)
    for x, y in ((a.cache.k_pages, b.cache.k_pages), (a.cache.v_pages, b.cache.v_pages), (oa, ob)):
        assert torch.equal(x.view(torch.int16), y.view(torch.int16))
    assert torch.equal(la, lb)
    assert_attention_close(case, oa, la, b.oracle(), what=f"G={hq // hkv} {layout}")


@pytest.mark.parametrize("pieces", [2, 4, 5, 8, 9, 16, 31, 33, 64])
def test_merge_of_few_and_many_pieces(pieces):
    """The split merge on both sides of its limits (four pieces: loaded by every lane; eight in
    flight; 32 a half wave), for three heads (a half wave without a row), with requests that are
    not split and a request index past the first 64 among the rows it has to find."""
    P = [64 * pieces - 3] + [0] * 70 + [64 * pieces - 40]
    C = [3] + [1] * 70 + [5]
    case = workloads.make_case("merge", P, C, 3, 1, seed=52)
    s = Setup(case)
    s.append()
    for tc in (16, 128):
        opts = s2l.plan_opts(tile_cols=tc, target_items=1 << 20, min_split_keys=64, max_splits=pieces)
        out, lse = s.attention(opts)
        assert s.plan.num_split_reqs == 2
        assert_attention_close(case, out, lse, s.oracle(), what=f"{pieces} pieces, {tc} columns")


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("hq,hkv", [(4, 4), (12, 4), (64, 8)])
def test_decode_tiles_at_their_edges(hq, hkv, kv_dtype):
    """One-token rows whose key counts lie around the tiles of one wave (32 keys bf16, 64 fp8), of
    the four waves, and the default piece length, unsplit, in the planner's pieces and in 64-key
    pieces (waves without a tile)."""
    P = [n - 1 + d for n in (32, 64, 128, 256, 512) for d in (-1, 0, 1)]
    case = workloads.make_case("dec_edges", P, [1] * len(P), hq, hkv, seed=53, kv_dtype=kv_dtype)
    s = Setup(case)
    s.append()
    for opts in (s2l.plan_opts(target_items=1), None, s2l.plan_opts(target_items=1 << 20, min_split_keys=64)):
        out, lse = s.attention(opts)
        assert s.plan.tile_cols == 16
        assert_attention_close(case, out, lse, s.oracle(), what=f"{kv_dtype} G={hq // hkv}")


def test_allocation_free_call_keeps_to_its_scratch():
    """Decode rows whose default plan (pieces of up to 4096 keys) needs more than the library's
    scratch: the allocation-free call plans them unsplit instead of refusing them.  Two rows are three
    times as long as the others: unsplit they would end long after them (which is what makes the
    planner cut), and with 255 rows for 256 workgroups one round has no room to split both."""
    R, hq, hkv, pool = 255, 16, 1, 64
    P = [131071] * (R - 2) + [3 * 131072 - 1] * 2
    gen = torch.Generator(device=DEV).manual_seed(54)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device=DEV).to(torch.bfloat16)
    cache = s2l.PagedKVCache(rnd(pool, hkv, 16, 128), rnd(pool, hkv, 16, 128))
    tables = torch.randint(0, pool, (R, max(P) // 16 + 1), generator=torch.Generator().manual_seed(54), dtype=torch.int32)
    batch = s2l.Batch(P, [1] * R, tables.numpy())
    assert s2l.s2l_attn_workspace_bytes(batch, hq, hkv) > s2l.NOALLOC_SCRATCH_BYTES
    q, out, ref = rnd(R, hq, 128), torch.empty_like(rnd(R, hq, 128)), torch.empty_like(rnd(R, hq, 128))
    info = s2l.s2l_chunk_prefill_attn_noalloc(cache, batch, q, hq, SCALE, out, None)
    assert info.num_split_reqs == 0
    ws = torch.empty(s2l.s2l_attn_workspace_bytes(batch, hq, hkv), dtype=torch.uint8, device=DEV)
    plan = s2l.s2l_attn_plan(batch, hq, hkv, ws)
    assert plan.num_split_reqs == R
    s2l.s2l_chunk_prefill_attn(cache, batch, q, hq, SCALE, ref, None, plan, ws)
    # Each result is sum(p v) / sum(p) over probabilities rounded to bf16 (2^-9 each, in the sum and
    # in its divisor: 2^-8 A, A = sum(p |v|) / sum(p)), rounded to bf16 (2^-9 |O|).  The two differ by
    # at most twice that; A comes from the same call over |V|, itself good to 2^-6.
    a = torch.empty_like(ref)
    s2l.s2l_chunk_prefill_attn(s2l.PagedKVCache(cache.k_pages, cache.v_pages.abs()), batch, q, hq, SCALE, a, None,
                               plan, ws)
    bound = 2.0 ** -7 * (1 + 2.0 ** -6) * a.float() + 2.0 ** -8 * ref.float().abs()
    assert torch.all((out.float() - ref.float()).abs() <= bound)


@pytest.mark.parametrize("R,hkv", [(1, 1), (1, 8), (2, 1), (3, 5), (63, 2), (65, 1), (256, 4), (257, 1), (1024, 1), (1025, 1)])
def test_device_plan_equals_the_host_plan(R, hkv):
    """The item records the device wrote (in any order, padding aside) are the host planner's, and so
    are the request arrays that the merge reads, with partials that tile the planned floats, at the
    request counts where the plan kernel changes its way: one, a wave, the ranked and binned limit
    (256), requests kept in LDS (1024)."""
    rng = np.random.default_rng(55 + R)
    P, C = rng.integers(0, 900, R), rng.integers(0, 90, R)
    C[0] = 5
    hq = 4 * hkv
    batch = s2l.Batch(P, C, np.zeros((R, 64), np.int32))
    for opts in (None, s2l.plan_opts(target_items=1 << 20, min_split_keys=64)):
        ws = torch.zeros(s2l.s2l_attn_workspace_bytes(batch, hq, hkv, opts), dtype=torch.uint8, device=DEV)
        plan = s2l.s2l_attn_plan(batch, hq, hkv, ws, opts)
        assert s2l.plan_status(ws).item() == 0
        _, items = s2l.s2l_plan_host(P, C, hq, hkv, opts, num_cus=torch.cuda.get_device_properties(0).multi_processor_count,
                                     with_items=True)
        assert len(items) == plan.num_items
        # after the header int32 item_off [R + 1], ns [R], c [R], cu [R + 1], int64 part_off [R]; then
        # the records, 64 bytes each
        raw, off = ws.cpu().numpy(), 256 + 4 * (R + 1)
        ns, c, dev_cu = np.split(raw[off:off + 4 * (3 * R + 1)].view(np.int32), [R, 2 * R])
        off = -(-(off + 4 * (3 * R + 1)) // 8) * 8
        part_off = raw[off:off + 8 * R].view(np.int64)
        off = (off + 8 * R + 63) // 64 * 64
        rec = raw[off:off + 64 * plan.num_items].view(np.int32).reshape(-1, 16)
        cu = np.concatenate([[0], np.cumsum(C)])
        real = rec[rec[:, 0] >= 0]
        got = sorted(map(tuple, real[:, :8].tolist()))
        # host rows: request, kv head, i0, i1, lo, hi, piece, pieces: the record's own order
        assert got == sorted(map(tuple, items[items[:, 0] >= 0].tolist()))
        r = real[:, 0]
        assert np.array_equal(real[:, 8], P[r]) and np.array_equal(real[:, 9], C[r]) and np.array_equal(real[:, 10], cu[r])
        host_ns = np.ones(R, np.int32)
        host_ns[items[items[:, 0] >= 0, 0]] = items[items[:, 0] >= 0, 7]
        assert np.array_equal(ns, host_ns) and np.array_equal(c, C) and np.array_equal(dev_cu, cu)
        assert np.array_equal(np.ascontiguousarray(real[:, 12:14]).view(np.int64)[:, 0], part_off[r])
        split = np.flatnonzero((ns > 1) & (C > 0))
        split = split[np.argsort(part_off[split])]
        ends = np.cumsum(ns[split].astype(np.int64) * C[split] * hq * 132)
        assert np.array_equal(part_off[split], np.concatenate([[0], ends])[:-1]) and plan.part_floats == (ends[-1] if len(ends) else 0)
        assert len(split) == plan.num_split_reqs
        pad = rec[rec[:, 0] < 0]
        assert len(pad) == (items[:, 0] < 0).sum() and np.all(pad[:, 0] == -1)


@pytest.mark.parametrize("R", [257, 1025])
def test_split_rows_of_many_requests(R):
    """Split attention and merge where the plan kernel leaves requests in their order (more than 256)
    and keeps their offsets in the workspace (more than 1024), in decode and in wide tiles."""
    rng = np.random.default_rng(R)
    case = workloads.make_case("many", rng.integers(0, 300, R), rng.integers(0, 4, R), 3, 1, seed=60)
    s = Setup(case)
    s.append()
    for tc in (16, 128):
        out, lse = s.attention(s2l.plan_opts(tile_cols=tc, target_items=1 << 20, min_split_keys=64))
        assert s.plan.num_split_reqs > R // 4
        assert_attention_close(case, out, lse, s.oracle(), what=f"{R} requests, {tc} columns")


def test_native_and_ctypes_marshalling_agree():
    """The per-step calls through the native marshalling (plain arguments) and through ctypes (here
    because the stream is a numpy integer, which only that path takes): the same launches, so the
    same bits; on a side stream given as an object, a number or the current one; and arguments that
    neither path takes raise the same errors."""
    case = workloads.make_case("marshal", [512, 64], [40, 100], 32, 8, seed=56)
    outs = []
    side = torch.cuda.Stream()
    for stream in (None, side, side.cuda_stream, np.int64(0)):
        with torch.cuda.stream(side if stream is side else torch.cuda.current_stream()):
            s = Setup(case)
            k, v = to_bf16(s.k_new), to_bf16(s.v_new)
            ws = torch.empty(s2l.s2l_attn_workspace_bytes(s.batch, 32, 8), dtype=torch.uint8, device=DEV)
            out = torch.zeros((case.total_tokens, 32, 128), dtype=torch.bfloat16, device=DEV)
            lse = torch.zeros((case.total_tokens, 32), dtype=torch.float32, device=DEV)
            torch.cuda.synchronize()
            plan = s2l.s2l_attn_plan(s.batch, 32, 8, ws, None, stream)
            s2l.s2l_kv_append(s.cache, s.batch, k, v, stream)
            s2l.s2l_chunk_prefill_attn(s.cache, s.batch, s.q, 32, SCALE, out, lse, plan, ws, stream)
            torch.cuda.synchronize()
            res = [out.clone(), lse.clone(), s.cache.k_pages]
            out.zero_()
            torch.cuda.synchronize()   # the stream of the fill need not be the one of the calls
            assert s2l.s2l_append_chunk_prefill_attn(s.cache, s.batch, k, v, s.q, 32, SCALE, out, lse, plan, ws, stream)
            torch.cuda.synchronize()
            res.append(out.clone())
            out.zero_()
            torch.cuda.synchronize()
            s2l.s2l_attn_main(s.cache, s.batch, s.q, 32, SCALE, out, None, plan, ws, stream)
            s2l.s2l_split_reduce(s.batch, 32, out, None, plan, ws, stream)
            torch.cuda.synchronize()
            res.append(out.clone())
            outs.append(res)
    assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for o in outs[1:] for a, b in zip(outs[0], o))
    assert torch.equal(outs[0][0], outs[0][3]) and torch.equal(outs[0][0], outs[0][4])
    for bad in (k.float(), torch.empty((200, 8, 128), dtype=torch.bfloat16, device=DEV)[::2]):
        with pytest.raises(ValueError, match="k_new must be a contiguous"):
            s2l.s2l_kv_append(s.cache, s.batch, bad, v)
    with pytest.raises(s2l.S2LError, match="NULL"):
        s2l.s2l_kv_append(s.cache, s.batch, None, v)
    with pytest.raises(s2l.S2LError, match="workspace"):
        s2l.s2l_chunk_prefill_attn(s.cache, s.batch, s.q, 32, SCALE, out, lse, plan, ws[:100])


@pytest.mark.parametrize("q8", [False, True])
@pytest.mark.parametrize("hq,hkv", [(2, 2), (7, 1), (64, 8)])
def test_split_e4m3_pieces_of_256_columns(hq, hkv, q8):
    """256-column tiles over e4m3 pages in many pieces (their partial rows are staged through LDS
    and stored as whole rows): full tiles, one token more, a single token, and group sizes that
    leave columns of a tile unused."""
    tq = 256 // (hq // hkv)
    case = workloads.make_case("f8split", [500, 64, 1000], [tq + 1, tq, 1], hq, hkv, seed=57, kv_dtype="fp8")
    s = Setup(case)
    s.append()
    opts = s2l.plan_opts(tile_cols=256, key_halves=1, target_items=1 << 20, min_split_keys=64, max_splits=16)
    out, lse = s.attention(opts, q8=q8)
    assert_attention_close(case, out, lse, s.oracle(q8=q8), what="f8split")


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("cols,halves", [(16, 1), (128, 1), (128, 2), (256, 1)])
def test_a_nan_key_reaches_every_output_that_sees_it(cols, halves, kv_dtype):
    """A NaN in one key of one kv head makes the scores, and so every output, of the rows that see it
    NaN, however their key range is cut: left whole, in the planner's pieces, and in a few and many
    small ones, where the piece that holds the key has a NaN row sum that the merge must not take
    for an empty piece.  Earlier rows and the other kv head stay as they are."""
    hq, hkv, P, C, bad = 4, 2, 700, 5, 702
    case = workloads.make_case("nan_key", [P, 64], [C, 3], hq, hkv, seed=58, kv_dtype=kv_dtype)
    s = Setup(case)
    s.append()
    plans = [dict(target_items=1), dict(), dict(target_items=1 << 20, min_split_keys=256),
             dict(target_items=1 << 20, min_split_keys=64, max_splits=64)]
    for key in (300, bad):
        for tc in [None] * (cols == 16) + [cols]:
            clean = [s.attention(s2l.plan_opts(**o, **({} if tc is None else dict(tile_cols=tc, key_halves=halves))))
                     for o in plans]
            page, slot = int(case.block_tables[0][key // 16]), key % 16
            old = s.cache.k_pages[page, 1, slot, 7].clone()
            s.cache.k_pages[page, 1, slot, 7] = 0x7f if kv_dtype == "fp8" else float("nan")
            seen = max(0, key - P)
            for o, (out0, lse0) in zip(plans, clean):
                out, lse = s.attention(s2l.plan_opts(**o, **({} if tc is None else dict(tile_cols=tc, key_halves=halves))))
                what = f"key {key}, {o}, {s.plan.num_split_reqs} split requests"
                assert torch.isnan(out[seen:C, 2:]).all() and torch.isnan(lse[seen:C, 2:]).all(), what
                for x, y in ((out, out0), (lse, lse0)):
                    assert torch.equal(x[:, :2], y[:, :2]) and torch.equal(x[C:], y[C:]) and torch.equal(x[:seen], y[:seen]), what
            s.cache.k_pages[page, 1, slot, 7] = old


@pytest.mark.parametrize("offset", [1, 4])
@pytest.mark.parametrize("cols,halves", [(16, 1), (128, 1), (128, 2), (256, 1)])
def test_q_and_out_of_a_view_between_16_byte_boundaries(cols, halves, offset):
    """Contiguous views that start 2 or 8 bytes into a buffer give the bits of aligned tensors, with
    full tiles, a tile of one token and group sizes that leave columns unused."""
    for hq, hkv in ((2, 2), (7, 1)):
        tq = cols // (hq // hkv)
        case = workloads.make_case("views", [100, 0], [tq + 1, tq], hq, hkv, seed=59)
        s = Setup(case)
        s.append()
        T = case.total_tokens
        opts = s2l.plan_opts(tile_cols=cols, key_halves=halves)
        ref, ref_lse = s.attention(opts)
        n = T * hq * 128
        q = torch.empty(n + offset, dtype=torch.bfloat16, device=DEV)[offset:].view(T, hq, 128).copy_(s.q)
        out = torch.full((n + offset,), float("nan"), dtype=torch.bfloat16, device=DEV)[offset:].view(T, hq, 128)
        lse = torch.empty_like(ref_lse)
        s2l.s2l_chunk_prefill_attn(s.cache, s.batch, q, hq, SCALE, out, lse, s.plan, s._ws)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16)) and torch.equal(lse, ref_lse)


def test_decode_reference_covers_the_first_64_keys_of_each_wave():
    """One-token rows whose weight lies on a single key: within the first 256 keys (64 for each of the
    four waves) that key sets the reference, its probability is 1 without rounding, and the
    log-sum-exp is good to fp32 (the score 2^-23 * 30, the other keys' sum 1000 e^-19 * 2^-8).  Rounded
    against another reference, each of these four scores would be off by 5e-4 or more."""
    keys, n, hq = [0, 31, 40, 100, 127, 128, 150, 200, 255], 1000, 4
    cache = s2l.PagedKVCache(torch.zeros((63 * len(keys), 1, 16, 128), dtype=torch.bfloat16, device=DEV),
                             torch.ones((63 * len(keys), 1, 16, 128), dtype=torch.bfloat16, device=DEV))
    tables = np.arange(63 * len(keys), dtype=np.int32).reshape(len(keys), 63)
    for r, j in enumerate(keys):
        cache.k_pages[63 * r + j // 16, 0, j % 16, 0] = 28.25
    q = torch.zeros((len(keys), hq, 128), dtype=torch.bfloat16, device=DEV)
    q[:, :, 0] = torch.tensor([8.0, 8.25, 8.5, 8.75], device=DEV)
    score = q[:, :, 0].double().cpu() * 28.25 * SCALE
    exact = score + torch.log1p((n - 1) * torch.exp(-score))
    batch = s2l.Batch([n - 1] * len(keys), [1] * len(keys), tables)
    opts = s2l.plan_opts(target_items=1)
    ws = torch.empty(s2l.s2l_attn_workspace_bytes(batch, hq, 1, opts), dtype=torch.uint8, device=DEV)
    plan = s2l.s2l_attn_plan(batch, hq, 1, ws, opts)
    out, lse = torch.empty_like(q), torch.empty(q.shape[:2], device=DEV)
    s2l.s2l_chunk_prefill_attn(cache, batch, q, hq, SCALE, out, lse, plan, ws)
    assert plan.tile_cols == 16 and plan.num_split_reqs == 0
    err = (lse.double().cpu() - exact).abs()
    assert err.max() < 3e-5, [(j, e.tolist()) for j, e in zip(keys, err)]
