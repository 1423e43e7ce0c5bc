"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.

Bit-exact for codes, min/max metadata, histograms, codebooks, records, offsets and the fp16 buffer; attention within
max|o_gpu - o_oracle| <= 1e-3 * max(1, max|o_oracle|).
"""
import sys

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

K, V = 0, 1
SCALE = 1.0 / np.sqrt(128.0)


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_00579_amd import binding
    binding.load()
    return binding


def _dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def _attn_close(o_gpu, o_ref):
    o_ref = np.asarray(o_ref, np.float64)
    err = np.abs(o_gpu.astype(np.float64) - o_ref).max()
    tol = 1e-3 * max(1.0, np.abs(o_ref).max())
    assert np.isfinite(o_gpu).all()
    assert err <= tol, f"max abs err {err:.3e} > {tol:.3e}"
    return err


def _both(gpu, oracle, B, H, Hq, S_book, S, max_seq, rel_k, rel_v, seed, limit=12):
    """Build codebooks on the first S_book tokens and compress S tokens on both sides (code words of up to `limit`
    bits; 12 is the library's default)."""
    Kx, Vx = W.make_kv(B, H, max(S_book, S), seed)
    oc = oracle.OracleCache(B, H, Hq, max_seq, rel_k, rel_v, 0, limit)
    oc.build_codebook(Kx[:, :S_book], Vx[:, :S_book])
    oc.compress_blocks(Kx[:, :S], Vx[:, :S])
    gc = gpu.KVCompCache(B, H, Hq, max_seq, rel_k, rel_v, max_code_len=limit)
    gc.build_codebook(_dev(Kx[:, :S_book]), _dev(Vx[:, :S_book]))
    gc.compress_blocks(_dev(Kx[:, :S]), _dev(Vx[:, :S]))
    return Kx, Vx, oc, gc


def _assert_same_cache(oc, gc, sample=None):
    st_o, st_g = oc.stats(), gc.stats()
    for key in ("n_blocks", "n_res", "raw_bytes", "record_bytes_k", "record_bytes_v", "header_bytes", "offsets_bytes",
                "residual_bytes", "payload_bits_k", "payload_bits_v", "stored_bytes"):
        assert st_o[key] == st_g[key], key
    assert abs(st_o["compression_ratio"] - st_g["compression_ratio"]) < 1e-12
    blocks = [(w, b, h, j) for w in (K, V) for b in range(oc.B) for h in range(oc.H) for j in range(oc.n_blocks)]
    if sample is not None and len(blocks) > sample:
        rng = np.random.default_rng(0)
        keep = rng.choice(len(blocks), sample, replace=False)
        blocks = [blocks[i] for i in keep]
    for w, b, h, j in blocks:
        bh = b * oc.H + h
        assert gc.block_entry(w, b, h, j) == (int(oc.off16[w][bh, j]), int(oc.size16[w][bh, j])), (w, b, h, j)
        np.testing.assert_array_equal(gc.get_block(w, b, h, j), oc.get_block(w, b, h, j), err_msg=str((w, b, h, j)))
    for w in (K, V):
        res, n = gc.residual(w)
        assert n == oc.n_res
        np.testing.assert_array_equal(res.view(np.uint16), oc.res[w][:, : oc.n_res].view(np.uint16))


@pytest.mark.parametrize("B,H,S,rel", [(1, 1, 1024, 1e-2), (2, 3, 200, 5e-3), (1, 2, 320, 2e-2)])
def test_codes_minmax_histogram_codebook(gpu, oracle, B, H, S, rel):
    _say(f"codes/hist B={B} H={H} S={S} rel={rel}")
    Kx, Vx = W.make_kv(B, H, S, 21)
    Kx[0, 64:128, 0, 5] = np.float16(0.75)   # a constant K unit
    Vx[0, 70, 0, :] = np.float16(-0.0)       # a constant V unit of negative zeros
    gc = gpu.KVCompCache(B, H, H, S, rel, rel)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    for which, X in ((K, Kx), (V, Vx)):
        codes_o, mm_o = oracle.tensor_quantize(which, X, rel)
        codes_g, mm_g = gc.debug_codes(which, _dev(X))
        np.testing.assert_array_equal(mm_g, mm_o)
        np.testing.assert_array_equal(codes_g, codes_o)
        hist_o = oracle.histogram(codes_o)
        np.testing.assert_array_equal(gc.histogram(which).astype(np.uint64), hist_o)
        ln_o, cd_o, _ = oracle.build_codebook(hist_o, oracle.n_sym(rel), 12)
        ln_g, cd_g = gc.codebook(which)
        np.testing.assert_array_equal(ln_g, ln_o)
        np.testing.assert_array_equal(cd_g, cd_o)
    gc.close()


def test_config0_end_to_end(gpu, oracle):
    w = W.CONFIGS["c0"]
    _say("config 0: compress + one decode step")
    Kx, Vx, oc, gc = _both(gpu, oracle, w.batch, w.n_kv_heads, w.n_q_heads, w.seq, w.seq, w.seq, w.rel_eb, w.rel_eb, w.seed,
                           limit=W.CODE_LEN_LIMIT[w.rel_eb])
    _assert_same_cache(oc, gc)
    q = W.make_queries(w.batch, w.n_q_heads, 1, w.seed)[0]
    out = gc.attn_decode(_dev(q), SCALE).cpu().numpy()
    err = _attn_close(out, oc.attn_decode(q, SCALE))
    _say(f"  attention max abs err {err:.3e}; CR {gc.stats()['compression_ratio']:.3f}")
    gc.close()


@pytest.mark.parametrize("B,H,Hq,S,rel_k,rel_v", [
    (2, 2, 2, 520, 1e-2, 2e-2),     # ragged tail of 8 tokens, several blocks per wave
    (1, 2, 8, 333, 5e-3, 1e-2),     # GQA group of 4
    (1, 1, 8, 192, 2e-2, 2e-2),     # GQA group of 8, no residual
    (3, 2, 4, 129, 1e-2, 1e-2),     # GQA group of 2, one-token tail
    (1, 1, 8, 200, 2e-3, 2e-3),     # 251 quantization levels: symbols above 127 through the int8 products of a group
    (1, 2, 8, 136, 2e-3, 4e-3),     # the same for a group of 4
])
def test_records_and_attention(gpu, oracle, B, H, Hq, S, rel_k, rel_v):
    _say(f"records+attention B={B} H={H} Hq={Hq} S={S}")
    Kx, Vx, oc, gc = _both(gpu, oracle, B, H, Hq, S, S, S + 64, rel_k, rel_v, 22)
    _assert_same_cache(oc, gc)
    for step in range(2):
        q = W.make_queries(B, Hq, 2, 22)[step]
        out = gc.attn_decode(_dev(q), SCALE).cpu().numpy()
        _attn_close(out, oc.attn_decode(q, SCALE))
    gc.close()


@pytest.mark.parametrize("B,H,Hq,S,rel_k,rel_v,k_mode,limit,window", [
    (2, 2, 2, 520, 1e-2, 2e-2, 0, 12, 64),     # ragged tail
    (1, 3, 3, 333, 5e-3, 1e-2, 1, 9, 64),      # K BlockQuant: one {min,max} pair per block in the workspace
    (1, 2, 8, 700, 1e-2, 1e-2, 0, 6, 256),     # buffer of 256 tokens: fewer blocks are encoded than were quantized
    (2, 1, 4, 64, 2e-2, 2e-2, 0, 6, 64),       # a single block
])
def test_prefill_with_one_quantization_pass(gpu, oracle, B, H, Hq, S, rel_k, rel_v, k_mode, limit, window):
    """kvcomp_prefill = kvcomp_build_codebook + kvcomp_compress_blocks with the codes kept in a workspace between the
    histogram pass and the encoder: histograms, codebooks, records, offsets, buffer and attention against the oracle,
    and the arena byte for byte against the two separate calls."""
    _say(f"prefill B={B} H={H} Hq={Hq} S={S} rel {rel_k}/{rel_v} k_mode={k_mode} limit {limit} buffer {window}")
    import torch
    Kx, Vx = W.make_kv(B, H, S, 38)
    Kx[0, 0:64, 0, 7] = np.float16(1.25)      # a constant K unit
    oc = oracle.OracleCache(B, H, Hq, S + 64, rel_k, rel_v, k_mode, limit, buffer_tokens=window)
    oc.build_codebook(Kx, Vx)
    oc.compress_blocks(Kx, Vx)
    gc = gpu.KVCompCache(B, H, Hq, S + 64, rel_k, rel_v, k_mode=k_mode, max_code_len=limit, buffer_tokens=window)
    dK, dV = _dev(Kx), _dev(Vx)
    ws = torch.full((gc.prefill_workspace_bytes(S) + 64,), 0xAB, dtype=torch.uint8, device="cuda:0")
    gc.prefill(dK, dV, ws[: gc.prefill_workspace_bytes(S)])
    assert (ws[gc.prefill_workspace_bytes(S):] == 0xAB).all()      # nothing written past the stated size
    for which in (K, V):
        np.testing.assert_array_equal(gc.histogram(which).astype(np.uint64), oc.hist[which])
        ln_g, cd_g = gc.codebook(which)
        np.testing.assert_array_equal(ln_g, oc.len[which])
        np.testing.assert_array_equal(cd_g, oc.code[which])
    _assert_same_cache(oc, gc)
    q = W.make_queries(B, Hq, 1, 38)[0]
    _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), oc.attn_decode(q, SCALE))
    one_pass = [gc.get_block(w, b, h, j) for w in (K, V) for b in range(B) for h in range(H) for j in range(oc.n_blocks)]
    gc.reset(keep_codebook=False)
    gc.build_codebook(dK, dV)
    gc.compress_blocks(dK, dV)
    two_calls = [gc.get_block(w, b, h, j) for w in (K, V) for b in range(B) for h in range(H) for j in range(oc.n_blocks)]
    for a, b_ in zip(one_pass, two_calls):
        np.testing.assert_array_equal(a, b_)
    # errors: too small a workspace, a cache that is not empty, non-finite input
    with pytest.raises(gpu.KvcompError) as e:
        gc.prefill(dK, dV, ws)
    assert e.value.status == gpu.ERR_STATE
    gc.reset(keep_codebook=False)
    with pytest.raises(gpu.KvcompError) as e:
        gc.prefill(dK, dV, ws[:1024])
    assert e.value.status == gpu.ERR_CAPACITY
    bad = Kx.copy()
    bad[0, 3, 0, 5] = np.nan
    with pytest.raises(gpu.KvcompError) as e:
        gc.prefill(_dev(bad), dV, ws)
    assert e.value.status == gpu.ERR_NONFINITE
    gc.prefill(dK, dV, ws)
    _assert_same_cache(oc, gc)
    gc.close()


@pytest.mark.parametrize("B,H,S", [(4, 8, 32768)])
def test_prefill_is_reproducible(gpu, B, H, S):
    """The same prompt compressed again and again gives the same cache: every record of 2 x 16384 blocks, read back as
    fp16 (a wave that clears a record header after another has filled it shows in about one block in 10^5)."""
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(17)
    Kx, Vx = (torch.randn((B, S, H, 128), generator=gen, device="cuda:0").half() for _ in range(2))
    gc = gpu.KVCompCache(B, H, H, S, 1e-2, 1e-2, max_code_len=6)
    ws = torch.empty(gc.prefill_workspace_bytes(S), dtype=torch.uint8, device="cuda:0")
    first = None
    for i in range(24):
        gc.reset(keep_codebook=False)
        gc.prefill(Kx, Vx, ws)
        got = [gc.decompress(w, S) for w in (K, V)]
        if first is None:
            first = got
        assert all(torch.equal(a, b) for a, b in zip(got, first)), f"pass {i} differs from the first"
    gc.close()


# up to 768 records of both tensors / 8192 of one are placed by the size pass's last workgroup, more by launches of their own
@pytest.mark.parametrize("B,H,n_blk", [(1, 1, 1), (3, 5, 7), (3, 16, 8), (5, 7, 11), (2, 16, 64), (2, 16, 65), (2, 32, 128), (3, 2731, 1),
                                       (4, 32, 128), (4, 32, 129)])
def test_placement_by_the_last_workgroup_and_by_launches(gpu, B, H, n_blk):
    import torch
    _say(f"placement of {B} x {H} x {n_blk} records a tensor")
    S = 64 * n_blk
    gen = torch.Generator(device="cuda:0").manual_seed(n_blk)
    k, v = (torch.randn((B, S, H, 128), generator=gen, device="cuda:0").half() for _ in range(2))
    gc = gpu.KVCompCache(B, H, H, S, 1e-2, 1e-2, max_code_len=6)
    gc.prefill(k, v, torch.empty(gc.prefill_workspace_bytes(S), dtype=torch.uint8, device="cuda:0"))

    def entries():
        return [gc.block_entry(w, b, h, j) for w in (K, V) for b in range(B) for h in range(H) for j in range(n_blk)]

    first = entries()  # sizes from the block histograms, one tensor after the other
    at = 0
    for off, size in first:
        assert off == at and size > 0
        at += size
    assert gc.stats()["max_record_bytes"] == 16 * max(size for _, size in first)
    gc.reset(keep_codebook=True)
    gc.compress_blocks(k, v)  # sizes from the codes, both tensors at once
    assert entries() == first
    gc.close()


def test_one_context_two_prompts_with_different_codebooks(gpu, oracle):
    """A context that is reset and filled again builds new codebooks: the tables that the second prompt is encoded and
    decoded with must be the second prompt's (the tables travel from a pinned host block that is rewritten in place).
    Second prompt: values on a coarse grid, so that most quantization levels are never used and the code lengths
    differ from the first prompt's in almost every symbol."""
    _say("one context, two prompts")
    B, H, Hq, S = 1, 2, 2, 384
    Ka, Va = W.make_kv(B, H, S, 61)
    rng = np.random.default_rng(62)
    Kb = (rng.integers(-3, 4, size=Ka.shape) * 0.5).astype(np.float16)
    Vb = (rng.integers(0, 2, size=Va.shape) * 2.0 - 1.0).astype(np.float16)
    gc = gpu.KVCompCache(B, H, Hq, S + 64, 1e-2, 1e-2, max_code_len=6)
    q = W.make_queries(B, Hq, 1, 61)[0]
    books = []
    for Kx, Vx in ((Ka, Va), (Kb, Vb), (Ka, Va)):
        oc = oracle.OracleCache(B, H, Hq, S + 64, 1e-2, 1e-2, 0, 6)
        oc.build_codebook(Kx, Vx)
        oc.compress_blocks(Kx, Vx)
        gc.reset(keep_codebook=False)
        gc.prefill(_dev(Kx), _dev(Vx))
        for which in (K, V):
            ln_g, cd_g = gc.codebook(which)
            np.testing.assert_array_equal(ln_g, oc.len[which])
            np.testing.assert_array_equal(cd_g, oc.code[which])
        _assert_same_cache(oc, gc)
        _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), oc.attn_decode(q, SCALE))
        for which in (K, V):   # the stand-alone decompressor reads the single-symbol tables and the tree
            ref = oc.decompress(which)
            np.testing.assert_array_equal(gc.decompress(which, S).cpu().numpy().view(np.uint16), ref.view(np.uint16))
            np.testing.assert_array_equal(gc.decompress(which, S, tree_walk=True).cpu().numpy().view(np.uint16), ref.view(np.uint16))
        books.append(np.asarray(oc.len[K]).copy())
    assert (books[0] != books[1]).sum() > 8    # the two prompts really have different codebooks
    gc.close()


def test_all_residual_and_tiny_sequences(gpu, oracle):
    _say("seq < 64: everything stays in the fp16 buffer")
    B, H, Hq = 2, 2, 4
    for S in (1, 40, 63, 64, 65):
        Kx, Vx, oc, gc = _both(gpu, oracle, B, H, Hq, 128, S, 128, 1e-2, 1e-2, 23)
        _assert_same_cache(oc, gc)
        q = W.make_queries(B, Hq, 1, 23)[0]
        _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), oc.attn_decode(q, SCALE))
        gc.close()


@pytest.mark.parametrize("G", [1, 4, 8])
def test_symbols_unseen_at_codebook_build(gpu, oracle, G):
    _say(f"codebook from a narrow prefix, later data uses every level; {G} query heads per KV head")
    B, H, S = 1, 2, 256
    Kx, Vx = W.make_kv(B, H, S, 24)
    # the first 64 tokens use only three distinct values per unit -> the histogram sees few levels
    Kx[:, :64] = np.float16(0.0); Kx[:, 0:64:2] = np.float16(1.0); Kx[:, 1:64:7] = np.float16(0.5)
    Vx[:, :64] = np.float16(0.0); Vx[:, :64, :, ::2] = np.float16(1.0); Vx[:, :64, :, 1::7] = np.float16(0.5)
    oc = oracle.OracleCache(B, H, G * H, S, 1e-2, 1e-2)
    oc.build_codebook(Kx[:, :64], Vx[:, :64])
    oc.compress_blocks(Kx, Vx)
    gc = gpu.KVCompCache(B, H, G * H, S, 1e-2, 1e-2)
    gc.build_codebook(_dev(Kx[:, :64]), _dev(Vx[:, :64]))
    gc.compress_blocks(_dev(Kx), _dev(Vx))
    assert int(oc.len[K].max()) > 8  # rare levels got long code words
    _assert_same_cache(oc, gc)
    q = W.make_queries(B, G * H, 1, 24)[0]
    _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), oc.attn_decode(q, SCALE))
    # the same cache decoded with a staging area smaller than its records (global-memory path)
    assert gc.stats()["max_record_bytes"] > 4608
    gc.set_tuning(stage_bytes=4608)
    _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), oc.attn_decode(q, SCALE))
    gc.set_tuning(n_splits=3)
    _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), oc.attn_decode(q, SCALE))
    gc.close()


def test_append_path(gpu, oracle):
    _say("append: 150 tokens one by one, two flushes")
    B, H, Hq, S0, extra = 2, 2, 4, 100, 150
    Kx, Vx, oc, gc = _both(gpu, oracle, B, H, Hq, S0, S0, 256, 1e-2, 1e-2, 25)
    kn, vn = W.make_new_tokens(B, H, extra, 25)
    qs = W.make_queries(B, Hq, extra, 25)
    dkn, dvn, dq = _dev(kn), _dev(vn), _dev(qs)
    for t in range(extra):
        oc.append_token(kn[t], vn[t])
        gc.append_token(dkn[t], dvn[t])
        if t % 37 == 0 or t in (27, 28, 91, 92, extra - 1):   # around the flushes at t = 27 and t = 91
            _attn_close(gc.attn_decode(dq[t], SCALE).cpu().numpy(), oc.attn_decode(qs[t], SCALE))
    assert oc.n_blocks == 3 and oc.n_res == (S0 + extra) % 64
    _assert_same_cache(oc, gc)
    # running the whole sequence again after a reset gives the byte-identical arena (no atomics in the placement)
    first = [gc.get_block(w, b, h, j) for w in (K, V) for b in range(B) for h in range(H) for j in range(3)]
    gc.reset(keep_codebook=True)
    gc.compress_blocks(_dev(Kx[:, :S0]), _dev(Vx[:, :S0]))
    for t in range(extra):
        gc.append_token(dkn[t], dvn[t])
    _assert_same_cache(oc, gc)
    second = [gc.get_block(w, b, h, j) for w in (K, V) for b in range(B) for h in range(H) for j in range(3)]
    for a, b_ in zip(first, second):
        np.testing.assert_array_equal(a, b_)
    gc.close()


@pytest.mark.parametrize("B,H,Hq,window,S0,extra", [(2, 2, 2, 192, 200, 260), (1, 2, 8, 128, 70, 200),
                                                    (1, 1, 8, 1024, 1100, 80), (2, 1, 1, 320, 40, 100)])
def test_larger_buffer_window(gpu, oracle, B, H, Hq, window, S0, extra):
    """A buffer of `window` > 64 tokens (Section 3.2.1, maximum buffer size of Section 4.2): the newest tokens stay
    fp16, the oldest block of a full buffer is compressed.  Records, offsets, buffer contents (oldest first), the
    decompressed cache and the attention output against the oracle, across several wrap-arounds of the ring."""
    _say(f"buffer window {window}: B={B} H={H} Hq={Hq}, prompt {S0} + {extra} appended tokens")
    max_seq = (S0 + extra + 63) // 64 * 64
    Kx, Vx = W.make_kv(B, H, max(S0, 64), 27)
    oc = oracle.OracleCache(B, H, Hq, max_seq, 1e-2, 1e-2, buffer_tokens=window)
    gc = gpu.KVCompCache(B, H, Hq, max_seq, 1e-2, 1e-2, buffer_tokens=window)
    oc.build_codebook(Kx, Vx)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    oc.compress_blocks(Kx[:, :S0], Vx[:, :S0])
    gc.compress_blocks(_dev(Kx[:, :S0]), _dev(Vx[:, :S0]))
    _assert_same_cache(oc, gc)
    kn, vn = W.make_new_tokens(B, H, extra, 27)
    qs = W.make_queries(B, Hq, extra, 27)
    dkn, dvn, dq = _dev(kn), _dev(vn), _dev(qs)
    worst = 0.0
    for t in range(extra):
        oc.append_token(kn[t], vn[t])
        gc.append_token(dkn[t], dvn[t])
        if t % 23 == 0 or oc.n_res in (window - 64, window - 1) or t == extra - 1:   # before and after every flush
            worst = max(worst, _attn_close(gc.attn_decode(dq[t], SCALE).cpu().numpy(), oc.attn_decode(qs[t], SCALE)))
    tokens = S0 + extra
    assert oc.n_blocks * 64 + oc.n_res == tokens
    _assert_same_cache(oc, gc)
    for which in (K, V):
        got = gc.decompress(which, tokens).cpu().numpy()
        np.testing.assert_array_equal(got.view(np.uint16), oc.decompress(which).view(np.uint16))
    _say(f"  blocks {oc.n_blocks}, buffered {oc.n_res}, worst attention error {worst:.2e}")
    gc.close()
    for bad in (100, 32, 8192):
        with pytest.raises(gpu.KvcompError):
            gpu.KVCompCache(B, H, Hq, max_seq, 1e-2, 1e-2, buffer_tokens=bad)


@pytest.mark.parametrize("B,H,Hq,window,S0,extra", [(2, 2, 2, 64, 100, 150), (1, 2, 8, 128, 70, 200),
                                                    (1, 1, 4, 192, 30, 260)])
def test_append_fused_into_the_attention_launch(gpu, oracle, B, H, Hq, window, S0, extra):
    """kvcomp_append_attn_decode = append_token then attn_decode: every step's output against the oracle's two calls,
    and the cache afterwards (buffer contents included: the kernel stores the token it read from the caller's tensor)
    bit for bit, across flushes and ring wrap-arounds; interleaved with the two separate calls."""
    _say(f"append fused into attention: B={B} H={H} Hq={Hq} buffer {window}, prompt {S0} + {extra} tokens")
    max_seq = (S0 + extra + 63) // 64 * 64
    Kx, Vx = W.make_kv(B, H, max(S0, 64), 28)
    oc = oracle.OracleCache(B, H, Hq, max_seq, 1e-2, 1e-2, buffer_tokens=window)
    gc = gpu.KVCompCache(B, H, Hq, max_seq, 1e-2, 1e-2, buffer_tokens=window)
    oc.build_codebook(Kx, Vx)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    oc.compress_blocks(Kx[:, :S0], Vx[:, :S0])
    gc.compress_blocks(_dev(Kx[:, :S0]), _dev(Vx[:, :S0]))
    kn, vn = W.make_new_tokens(B, H, extra, 28)
    qs = W.make_queries(B, Hq, extra, 28)
    dkn, dvn, dq = _dev(kn), _dev(vn), _dev(qs)
    worst = 0.0
    for t in range(extra):
        oc.append_token(kn[t], vn[t])
        if t % 11 == 5:   # the two separate calls in between
            gc.append_token(dkn[t], dvn[t])
            out = gc.attn_decode(dq[t], SCALE)
        else:
            out = gc.append_attn_decode(dkn[t], dvn[t], dq[t], SCALE)
        if t % 3 == 0 or oc.n_res in (window - 64, window - 63, window - 1):
            worst = max(worst, _attn_close(out.cpu().numpy(), oc.attn_decode(qs[t], SCALE)))
        if t in (0, 17, extra // 2):
            _assert_same_cache(oc, gc)
    _assert_same_cache(oc, gc)
    _say(f"  blocks {oc.n_blocks}, buffered {oc.n_res}, worst attention error {worst:.2e}")
    for _ in range(max_seq - S0 - extra):
        gc.append_attn_decode(dkn[0], dvn[0], dq[0], SCALE)
    with pytest.raises(gpu.KvcompError) as e:
        gc.append_attn_decode(dkn[0], dvn[0], dq[0], SCALE)
    assert e.value.status == gpu.ERR_CAPACITY
    gc.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("n0", [1, 14, 30, 60])
def test_buffered_tokens_at_unit_edges(gpu, oracle, G, n0):
    """Nothing but buffered fp16 tokens, which are read in units of 16: counts around the edges of a unit, the newest token
    (still in the caller's tensor) first and last of its unit.  fp16 inputs, exact products, fp32 sums of at most 128 and
    63 terms: 2^-24 * (128 + 63) * the sum of magnitudes, below 3e-5 for these inputs."""
    B, H = 2, 2
    Kx, Vx, oc, gc = _both(gpu, oracle, B, H, H * G, 64, n0, 128, 1e-2, 1e-2, seed=41 + n0)
    kn, vn = W.make_new_tokens(B, H, 3, 43)
    q = W.make_queries(B, H * G, 3, 44)
    for t in range(3):
        oc.append_token(kn[t], vn[t])
        out = gc.append_attn_decode(_dev(kn[t]), _dev(vn[t]), _dev(q[t]), SCALE).cpu().numpy()
        ref = oc.attn_decode(q[t], SCALE)
        assert np.abs(out - ref).max() <= 3e-5 * max(1.0, np.abs(ref).max()), (t, np.abs(out - ref).max())
        again = gc.attn_decode(_dev(q[t]), SCALE).cpu().numpy()  # the token is in its slot now
        assert np.array_equal(out, again)
    held = np.concatenate([Vx[:, :n0], vn.transpose(1, 0, 2, 3)], axis=1)
    assert np.array_equal(gc.residual(V)[0].view(np.uint16), held.view(np.uint16))
    gc.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_scores_of_buffered_tokens_are_summed_in_a_tree(gpu, G):
    """The scores of the buffered tokens are fp32 sums over 128 channels, and with large ones they decide the error of the
    output.  Summed as a tree (four sums of 32 channels, then the four), as numpy does here for the comparison, partial sums
    stay small; one running sum over the four leaves half as much error again.  Everything else is float64 in the comparison,
    so the kernel may exceed it by the rounding of its exp and sums: a quarter."""
    B, H, S, seeds = 2, 4, 200, 12
    err, tree = 0.0, 0.0
    for seed in range(seeds):
        Kx, Vx = W.make_kv(B, H, S, 300 + seed)
        q = (2 * W.make_queries(B, H * G, 1, 300 + seed)[0].astype(np.float32)).astype(np.float16)
        gc = gpu.KVCompCache(B, H, H * G, 256, 1e-2, 1e-2, buffer_tokens=256)
        gc.prefill(_dev(Kx), _dev(Vx))
        out = gc.attn_decode(_dev(q), SCALE).cpu().numpy().astype(np.float64)
        gc.close()
        for b in range(B):
            for hq in range(H * G):
                prod = Kx[b, :, hq // G].astype(np.float32) * q[b, hq].astype(np.float32)   # exact: 11 x 11 bits
                exact = prod.astype(np.float64).sum(-1)
                part = prod.reshape(S, 4, 32).transpose(0, 2, 1)
                while part.shape[1] > 1:
                    part = part[:, 0::2] + part[:, 1::2]
                part = part[:, 0]
                part = ((part[:, 0] + part[:, 1]) + (part[:, 2] + part[:, 3])).astype(np.float64)
                ref, cmp = ((lambda p: p / p.sum() @ Vx[b, :, hq // G].astype(np.float64))(np.exp(SCALE * (s - exact.max())))
                            for s in (exact, part))
                err += ((out[b, hq] - ref) ** 2).sum()
                tree += ((cmp - ref) ** 2).sum()
    _say(f"  buffered scores, groups of {G}: error {np.sqrt(err / tree):.3f} of the tree's")
    assert err <= 1.25 ** 2 * tree, np.sqrt(err / tree)


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("S", [20, 64 * 2 + 20])
def test_infinities_in_the_v_of_buffered_tokens(gpu, oracle, G, S):
    """A buffered token is taken as it is, Inf in V included: every head gets Inf in that channel, however many waves there are
    to merge, and the other channels do not notice."""
    _say(f"Inf in V of buffered tokens, groups of {G}, {S} tokens")
    B, H = 1, 2
    _, _, oc, gc = _both(gpu, oracle, B, H, G * H, 64, S, 256, 1e-2, 1e-2, 64)
    kn, vn = W.make_new_tokens(B, H, 2, 64)
    for t in range(2):
        oc.append_token(kn[t], vn[t])
    vn[0, 0, :, 5], vn[1, 0, :, 99] = np.inf, -np.inf
    for t in range(2):
        gc.append_token(_dev(kn[t]), _dev(vn[t]))
    q = W.make_queries(B, G * H, 1, 64)[0]
    ref = np.array(oc.attn_decode(q, SCALE))
    ref[..., 5], ref[..., 99] = np.inf, -np.inf
    for n_splits in (1, 2):
        for waves in (0, 1, 2, 3, 4, 5, 6, 7, 8):
            gc.set_tuning(n_splits=n_splits, waves=waves)
            out = gc.attn_decode(_dev(q), SCALE).cpu().numpy()
            np.testing.assert_allclose(out, ref, rtol=0, atol=1e-3, err_msg=f"{n_splits} {waves}")
    gc.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("S", [16, 64 + 16, 64 * 3 + 32])
def test_buffered_tokens_that_score_minus_infinity(gpu, oracle, G, S):
    """Buffered tokens with score -Inf (K holds -Inf where every query is positive) take no part, also where they fill a unit
    of 16 by themselves: the output is that of the cache without them."""
    _say(f"buffered tokens that score -Inf, groups of {G}, {S} tokens")
    B, H = 1, 2
    _, _, oc, gc = _both(gpu, oracle, B, H, G * H, 64, S, 256, 1e-2, 1e-2, 65)
    kn, vn = W.make_new_tokens(B, H, 17, 65)
    kn[..., 30] = -np.inf
    q = W.make_queries(B, G * H, 1, 65)[0]
    q[..., 30] = 1.0
    ref = np.array(oc.attn_decode(q, SCALE))
    for t in range(17):                        # a unit of their own, then one behind it
        _attn_close(gc.append_attn_decode(_dev(kn[t]), _dev(vn[t]), _dev(q), SCALE).cpu().numpy(), ref)
    for n_splits in (1, 2):
        for waves in (0, 1, 2, 3, 5, 8):
            gc.set_tuning(n_splits=n_splits, waves=waves)
            _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), ref)
    gc.close()


@pytest.mark.parametrize("G", [2, 4, 8])
def test_units_that_score_minus_infinity_for_one_head_only(gpu, oracle, G):
    """Two units of buffered tokens on the wave that has the blocks: all tokens score -Inf for the even heads, those of the
    second unit +Inf for the odd ones, whose reference moves.  The even heads' output is that of the blocks alone."""
    _say(f"units that score -Inf for one head only, groups of {G}")
    B, H = 1, 2
    _, _, oc, gc = _both(gpu, oracle, B, H, G * H, 64, 64, 256, 1e-2, 1e-2, 66)
    kn, vn = W.make_new_tokens(B, H, 32, 66)
    kn[:16, ..., 30] = kn[16:, ..., 31] = -np.inf
    q = W.make_queries(B, G * H, 1, 66)[0]
    q[..., 30:32] = 1.0
    q[:, 1::2, 31] = -1.0
    ref = np.array(oc.attn_decode(q, SCALE))
    for t in range(32):
        gc.append_token(_dev(kn[t]), _dev(vn[t]))
    for waves in (1, 2, 3, 8):
        gc.set_tuning(n_splits=1, waves=waves)
        out = gc.attn_decode(_dev(q), SCALE).cpu().numpy()
        _attn_close(out[:, ::2], ref[:, ::2])
    gc.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("limit", [6, 12])
@pytest.mark.parametrize("blocks", [0, 1, 2, 3, 9])
def test_a_buffered_token_that_scores_nan(gpu, oracle, G, limit, blocks):
    """A NaN in the K of the newest token, or Infs of both signs there, makes the output NaN: alone in its unit of 16 and with one
    token beside it, on a wave of its own and on one with blocks, in every split."""
    _say(f"a buffered token that scores NaN, groups of {G}, code words of up to {limit} bits, {blocks} blocks")
    B, H = 1, 2
    q = W.make_queries(B, G * H, 1, 67)[0]
    q[..., 30:32] = 1.0
    for buffered in (0, 1, 16, 17):            # in front of the token
        n = 64 * blocks + buffered
        Kx, Vx = W.make_kv(B, H, max(n, 64), 67)
        kn, vn = W.make_new_tokens(B, H, 2, 67)
        for bad in ((np.nan, 0.0), (np.inf, -np.inf)):
            gc = gpu.KVCompCache(B, H, G * H, 64 * 10, 1e-2, 1e-2, max_code_len=limit)
            gc.build_codebook(_dev(Kx), _dev(Vx))
            if n:
                gc.compress_blocks(_dev(Kx[:, :n]), _dev(Vx[:, :n]))
            kn[0, ..., 30:32] = bad
            for t in range(2):                 # the token appended inside the launch, then one behind it
                assert np.isnan(gc.append_attn_decode(_dev(kn[t]), _dev(vn[t]), _dev(q), SCALE).cpu().numpy()).all()
                for n_splits in (1, 2):
                    for waves in (0, 1, 2, 3, 4, 5, 8):
                        gc.set_tuning(n_splits=n_splits, waves=waves)
                        out = gc.attn_decode(_dev(q), SCALE).cpu().numpy()
                        assert np.isnan(out).all(), (buffered, bad, t, n_splits, waves)
                gc.set_tuning()
            gc.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("limit", [6, 12])
def test_a_query_that_is_not_finite_spoils_its_own_head_only(gpu, oracle, G, limit):
    """An Inf or a NaN in the query of one head: that head's output is NaN, the others' are what they are without it."""
    _say(f"queries that are not finite, groups of {G}, code words of up to {limit} bits")
    B, H, S = 1, 2, 64 * 9 + 21
    _, _, oc, gc = _both(gpu, oracle, B, H, G * H, S, S, S, 1e-2, 1e-2, 70, limit)
    q = W.make_queries(B, G * H, 1, 70)[0]
    ref = oc.attn_decode(q, SCALE)
    for head in {0, G - 1, G}:
        for bad in (np.inf, -np.inf, np.nan):
            qb = q.copy()
            qb[0, head, 77] = bad
            others = np.arange(G * H) != head
            for n_splits, waves in ((0, 0), (1, 1), (1, 3), (2, 0)):
                gc.set_tuning(n_splits=n_splits, waves=waves)
                out = gc.attn_decode(_dev(qb), SCALE).cpu().numpy()
                assert np.isnan(out[0, head]).all(), (head, bad, n_splits, waves)
                _attn_close(out[0, others], ref[0, others])
    gc.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("blocks", [2, 9])
def test_blocks_that_score_minus_infinity(gpu, G, blocks):
    """Blocks whose tokens all score -Inf (a scale that overflows) take no part, first blocks of a wave and of a split among them:
    the output is the mean of V over the blocks that score 0, whose V is the same for every token and exact."""
    _say(f"blocks that score -Inf, groups of {G}, {blocks} blocks")
    B, H, S = 1, 2, 64 * blocks
    rng = np.random.default_rng(68)
    Kx, Vx = np.zeros((B, S, H, 128), np.float16), rng.standard_normal((B, S, H, 128)).astype(np.float16)
    q = rng.standard_normal((B, G * H, 128)).astype(np.float16)
    q[..., 5] = -2.0
    for live in (0, blocks - 1):
        Kx[..., 5] = 1.0
        Kx[:, 64 * live:64 * (live + 1), :, 5] = 0.0
        Vx[:, 64 * live:64 * (live + 1)] = (np.arange(128) % 2).astype(np.float16)   # the two ends of every token's range
        gc = gpu.KVCompCache(B, H, G * H, S, 1e-2, 1e-2)
        gc.build_codebook(_dev(Kx), _dev(Vx))
        gc.compress_blocks(_dev(Kx), _dev(Vx))
        for n_splits in (0, 1, 2, blocks):
            for waves in (0, 1, 2, 3, 8):
                gc.set_tuning(n_splits=n_splits, waves=waves)
                out = gc.attn_decode(_dev(q), 3e38).cpu().numpy()
                np.testing.assert_allclose(out, np.broadcast_to(np.arange(128) % 2, out.shape), rtol=0, atol=1e-5)
        gc.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("limit", [6, 12])
def test_a_wave_for_each_record_of_a_pair(gpu, oracle, G, limit):
    _say(f"K and V records of a pair on two waves, and on one; groups of {G}, code words of up to {limit} bits")
    B, H = 1, 2
    for S in (64, 64 * 4 + 63, 64 * 6 + 1, 64 * 9 + 40):  # 1, 4, 6 and 9 blocks: around every edge of the rule
        _, _, oc, gc = _both(gpu, oracle, B, H, G * H, 64, S, S, 1e-2, 1e-2, 61, limit)
        q = W.make_queries(B, G * H, 1, 61)[0]
        ref = oc.attn_decode(q, SCALE)
        for n_splits in (1, 2, 3, oc.n_blocks):  # last splits with fewer blocks among them
            # waves: the library's choice; too few for the pairs; stage_bytes: as needed, and records from global memory
            for waves, stage in ((0, 0), (1, 0), (3, 0), (0, 4608), (1, 4608)):
                gc.set_tuning(n_splits=n_splits, waves=waves, stage_bytes=stage)
                _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), ref)
        gc.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("rel", [1e-2, 2e-2])
def test_pairs_of_a_split_on_twelve_to_sixteen_waves(gpu, oracle, G, rel):
    """One split with as many block pairs as the rules for its waves go by: groups of 4 have room for fifteen waves at 1e-2 and for
    sixteen at 2e-2, groups of 1 and 2 for sixteen."""
    _say(f"one split of up to 33 pairs, groups of {G}, bound {rel}")
    q = W.make_queries(1, G, 1, 69)[0]
    for blocks in (12, 13, 15, 16, 17, 20, 31, 32, 33):
        _, _, oc, gc = _both(gpu, oracle, 1, 1, G, 64 * 12, 64 * blocks + 21, 64 * 40, rel, rel, 69, 6)
        if G == 4 and blocks == 33:
            room = (160 * 1024 - 32768 - 4 * (512 + 192) - 512) // (gc.stats()["max_record_bytes"] + 32 + 12 * 144)
            assert room == 15 if rel == 1e-2 else room >= 16
        ref = oc.attn_decode(q, SCALE)
        for waves in (0, 12, 13, 14, 15, 16):
            gc.set_tuning(n_splits=1, waves=waves)
            _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), ref)
        gc.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_query_at_any_element_of_a_larger_tensor(gpu, oracle, G):
    """The query may start at any fp16 element: blocks and buffered tokens give the same bits as from an aligned copy."""
    import torch
    _say(f"queries at odd elements, groups of {G}")
    B, H, S = 2, 2, 300
    _, _, oc, gc = _both(gpu, oracle, B, H, G * H, S, S, S + 8, 1e-2, 1e-2, 63)
    q = W.make_queries(B, G * H, 1, 63)[0]
    want = gc.attn_decode(_dev(q), SCALE)
    _attn_close(want.cpu().numpy(), oc.attn_decode(q, SCALE))
    for first in (1, 2, 4, 7):
        flat = torch.full((q.size + 8,), float("nan"), dtype=torch.float16, device="cuda:0")
        view = flat[first:first + q.size].view(q.shape)
        view.copy_(_dev(q))
        assert torch.equal(gc.attn_decode(view, SCALE), want)
    kn, vn = W.make_new_tokens(B, H, 1, 63)
    oc.append_token(kn[0], vn[0])
    _attn_close(gc.append_attn_decode(_dev(kn[0]), _dev(vn[0]), view, SCALE).cpu().numpy(), oc.attn_decode(q, SCALE))
    gc.close()


@pytest.mark.parametrize("G", [1, 2])
@pytest.mark.parametrize("rel,limit", [(2e-3, 8), (2e-3, 12), (3.9e-3, 8), (3.95e-3, 7), (1e-2, 6), (0.25, 2)])
def test_integer_dot_products_of_groups_of_1_and_2(gpu, oracle, G, rel, limit):
    """Weights as 30-bit integers against decoded symbols as int8: 251, 129, 128, 51 and 3 levels (beyond 128 the symbols are
    biased), channels ten times the others.  The weights carry fp32's 24 bits, the products are exact, the rest is fp32
    sums over 128 channels and 195 tokens: 2^-24 * (128 + 195) * the sum of magnitudes (about 4) is 8e-5."""
    B, H, S = 1, 2, 195
    Kx, Vx, oc, gc = _both(gpu, oracle, B, H, H * G, S, S, 256, rel, rel, seed=51, limit=limit)
    q = W.make_queries(B, H * G, 1, 52)[0]
    out = gc.attn_decode(_dev(q), SCALE).cpu().numpy()
    ref = oc.attn_decode(q, SCALE)
    assert np.abs(out - ref).max() <= 8e-5 * max(1.0, np.abs(ref).max()), np.abs(out - ref).max()
    gc.close()


@pytest.mark.parametrize("G", [1, 2])
def test_small_weights_beside_a_large_one_are_rounded(gpu, oracle, G):
    """One channel's weight is 2^24 times the others', so that those are integers of about 100 on the block's scale (unit 2^-20).
    Half of the tokens have code 50 in all 127 of them and differ from the other half by the error of the weights alone: rounded
    to nearest, 0.29 * sqrt(127) * 50 units = 1.6e-4 of the score in the mean, cut off 0.5 * 127 * 50 units = 3e-3.  The output
    moves by half of it: 5 of the former, 4e-4, is the bar."""
    _say(f"small weights beside a large one, groups of {G}")
    S = 64
    Kx, Vx = np.zeros((1, S, 1, 128), np.float16), np.ones((1, S, 1, 128), np.float16)
    Kx[0, 1::2, 0, 1:] = 1.0          # codes 0 and 50
    Kx[0, 32:, 0, 0] = 1.0            # these tokens' scores are far below the others'
    Vx[0, 1::2] = -1.0
    q = np.random.default_rng(5).uniform(1e-3, 4e-3, (1, G, 128)).astype(np.float16)
    q[..., 0] = -32768.0
    oc = oracle.OracleCache(1, 1, G, S, 1e-2, 1e-2, 0, 12)
    gc = gpu.KVCompCache(1, 1, G, S, 1e-2, 1e-2)
    for c, dev in ((oc, lambda x: x), (gc, _dev)):
        c.build_codebook(dev(Kx), dev(Vx))
        c.compress_blocks(dev(Kx), dev(Vx))
    err = np.abs(gc.attn_decode(_dev(q), 1.0).cpu().numpy() - oc.attn_decode(q, 1.0)).max()
    assert err <= 4e-4, err
    gc.close()


def test_many_sequence_splits(gpu, oracle):
    """One long sequence with a single KV head: the library splits it 128 ways (its maximum) so that the chip is
    filled; every split count gives the oracle's result, also when the last split is short or the buffer holds
    more 16-token units than there are splits."""
    _say("one head, 20000 tokens: 128 splits (automatic), then 97, 5 and 1")
    B, H, Hq, S = 1, 1, 2, 20000
    Kx, Vx = W.make_kv(B, H, S, 29)
    oc = oracle.OracleCache(B, H, Hq, S + 64, 1e-2, 1e-2, 0, 7, buffer_tokens=256)
    gc = gpu.KVCompCache(B, H, Hq, S + 64, 1e-2, 1e-2, max_code_len=7, buffer_tokens=256)
    oc.build_codebook(Kx, Vx)
    oc.compress_blocks(Kx, Vx)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    gc.compress_blocks(_dev(Kx), _dev(Vx))
    assert oc.n_blocks == 309 and oc.n_res == 224
    q = W.make_queries(B, Hq, 1, 29)[0]
    ref = oc.attn_decode(q, SCALE)
    for n_splits in (0, 97, 5, 1):
        gc.set_tuning(n_splits=n_splits)
        err = _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), ref)
        _say(f"  n_splits {n_splits}: max abs err {err:.2e}")
    gc.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("n_blocks,splits", [(130, (2, 15, 17, 33, 65)), (128, (16, 32, 64, 128))])
def test_split_merge_at_range_edges(gpu, oracle, G, n_blocks, splits):
    _say(f"splits merged in one and in several ranges; groups of {G}, {n_blocks} blocks")
    B, H, S = 1, 1, 64 * n_blocks
    _, _, oc, gc = _both(gpu, oracle, B, H, G * H, 256, S, S, 1e-2, 1e-2, 62, 6)
    q = W.make_queries(B, G * H, 1, 62)[0]
    ref = np.asarray(oc.attn_decode(q, SCALE), np.float64)
    # waves of a workgroup to a head, batches of 16 splits, the second split of a lane (beyond 64).  A split left out or
    # with another's weight is off by 1e-2 and more; the integer weights of groups of 4 and 8 by up to 2e-4.
    for n_splits in splits:
        per_split = -(-n_blocks // n_splits)
        assert -(-n_blocks // per_split) == n_splits, "the launch has as many splits as asked for"
        for waves in (0, 1, 5):
            gc.set_tuning(n_splits=n_splits, waves=waves)
            out = gc.attn_decode(_dev(q), SCALE).cpu().numpy().astype(np.float64)
            assert np.linalg.norm(out - ref) <= 2e-4 * np.linalg.norm(ref), (n_splits, waves)
    gc.close()


def _random_cases(n):
    rng = np.random.default_rng(2024)
    cases = []
    for i in range(n):
        H = int(rng.choice([1, 2, 3]))
        G = int(rng.choice([1, 2, 4, 8]))
        rel_k, rel_v = (float(x) for x in rng.choice([4e-3, 1e-2, 2e-2, 5e-2, 0.1], 2))
        levels = int(np.rint(1.0 / (2.0 * np.float32(min(rel_k, rel_v))))) + 1
        lo = int(np.ceil(np.log2(levels)))
        cases.append((int(rng.choice([1, 2])), H, H * G, int(rng.integers(64, 700)), rel_k, rel_v,
                      int(rng.choice([0, 1])), int(rng.integers(lo, 13)), int(rng.choice([64, 64, 128, 256])),
                      int(rng.integers(0, 150)), 100 + i))
    return cases


@pytest.mark.parametrize("B,H,Hq,S,rel_k,rel_v,k_mode,max_len,window,extra,seed", _random_cases(12))
def test_random_small_configs(gpu, oracle, B, H, Hq, S, rel_k, rel_v, k_mode, max_len, window, extra, seed):
    """Seeded random combinations of batch, heads, group size, length, error bounds, K unit, code word limit, buffer
    size and appended tokens: whole cache and decompressed tensors bit for bit, attention within tolerance."""
    _say(f"random case: B={B} H={H} Hq={Hq} S={S} rel {rel_k}/{rel_v} k_mode={k_mode} limit {max_len} "
         f"buffer {window} +{extra} tokens")
    max_seq = (S + extra + 63) // 64 * 64
    Kx, Vx = W.make_kv(B, H, S, seed)
    oc = oracle.OracleCache(B, H, Hq, max_seq, rel_k, rel_v, k_mode, max_len, buffer_tokens=window)
    gc = gpu.KVCompCache(B, H, Hq, max_seq, rel_k, rel_v, k_mode=k_mode, max_code_len=max_len, buffer_tokens=window)
    oc.build_codebook(Kx, Vx)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    oc.compress_blocks(Kx, Vx)
    gc.compress_blocks(_dev(Kx), _dev(Vx))
    kn, vn = W.make_new_tokens(B, H, max(extra, 1), seed)
    qs = W.make_queries(B, Hq, max(extra, 1), seed)
    for t in range(extra):
        oc.append_token(kn[t], vn[t])
        if t % 5 == 4:
            gc.append_token(_dev(kn[t]), _dev(vn[t]))
        else:
            out = gc.append_attn_decode(_dev(kn[t]), _dev(vn[t]), _dev(qs[t]), SCALE)
            if t % 16 == 0:
                _attn_close(out.cpu().numpy(), oc.attn_decode(qs[t], SCALE))
    _assert_same_cache(oc, gc)
    _attn_close(gc.attn_decode(_dev(qs[0]), SCALE).cpu().numpy(), oc.attn_decode(qs[0], SCALE))
    tokens = S + extra
    for which in (K, V):
        got = gc.decompress(which, tokens).cpu().numpy()
        np.testing.assert_array_equal(got.view(np.uint16), oc.decompress(which).view(np.uint16))
    gc.close()


def test_decode_loop_in_a_hip_graph(gpu, oracle):
    """The decode loop (append + attention per step, one flush inside) captured in a HIP graph, as bench.py times it:
    every replay -- with an eager reset and prefill of the cache in between -- must give the eager loop's outputs bit
    for bit; the last step is also checked against the oracle."""
    import torch
    _say("decode loop of 20 steps in a HIP graph, three replays")
    B, H, Hq, S0, T = 2, 2, 4, 180, 20      # 180 = 2 blocks + 52 buffered: the 12th append completes a block
    Kx, Vx, oc, gc = _both(gpu, oracle, B, H, Hq, S0, S0, 256, 1e-2, 1e-2, 33)
    kn, vn = W.make_new_tokens(B, H, T, 33)
    qs = W.make_queries(B, Hq, T, 33)
    dK, dV, dkn, dvn, dq = _dev(Kx[:, :S0]), _dev(Vx[:, :S0]), _dev(kn), _dev(vn), _dev(qs)
    outs = torch.empty((T, B, Hq, 128), dtype=torch.float32, device="cuda:0")

    def loop():
        for t in range(T):
            gc.append_attn_decode(dkn[t], dvn[t], dq[t], SCALE, outs[t])

    def prefill():
        gc.reset(keep_codebook=True)
        gc.compress_blocks(dK, dV)

    loop()
    torch.cuda.synchronize()
    eager = outs.cpu().numpy().copy()
    for t in range(T):
        oc.append_token(kn[t], vn[t])
    _attn_close(eager[T - 1], oc.attn_decode(qs[T - 1], SCALE))
    _assert_same_cache(oc, gc)
    prefill()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        loop()
    for replay in range(3):
        prefill()                      # eager work and a synchronisation between the replays
        outs.zero_()
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(outs.cpu().numpy(), eager, err_msg=f"replay {replay}")
    # a replay runs the device work only: the context's host-side counters are where the last eager call left them
    # (the prefill), so the cache is brought back to a consistent state eagerly before it is used again
    prefill()
    loop()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(outs.cpu().numpy(), eager)
    _assert_same_cache(oc, gc)
    gc.close()


def test_on_a_side_stream(gpu, oracle):
    """Every call takes the caller's stream: the whole path on a non-default stream (default priority), with the
    default stream kept busy by unrelated work, gives the same cache and attention."""
    import torch
    _say("the path on a side stream")
    B, H, Hq, S = 1, 2, 4, 300
    Kx, Vx = W.make_kv(B, H, S, 34)
    oc = oracle.OracleCache(B, H, Hq, 384, 1e-2, 1e-2)
    oc.build_codebook(Kx, Vx)
    oc.compress_blocks(Kx, Vx)
    kn, vn = W.make_new_tokens(B, H, 30, 34)
    q = W.make_queries(B, Hq, 1, 34)[0]
    for t in range(30):
        oc.append_token(kn[t], vn[t])
    dK, dV, dkn, dvn, dq = _dev(Kx), _dev(Vx), _dev(kn), _dev(vn), _dev(q)
    busy = torch.empty(64 << 20, dtype=torch.uint8, device="cuda:0")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        gc = gpu.KVCompCache(B, H, Hq, 384, 1e-2, 1e-2)
        gc.build_codebook(dK, dV)
        torch.cuda.default_stream().wait_stream(side)   # unrelated work on the default stream, ordered after this point
        with torch.cuda.stream(torch.cuda.default_stream()):
            for _ in range(4):
                busy.fill_(1)
        gc.compress_blocks(dK, dV)
        for t in range(30):
            if t % 2:
                gc.append_token(dkn[t], dvn[t])
            else:
                gc.append_attn_decode(dkn[t], dvn[t], dq, SCALE)
        out = gc.attn_decode(dq, SCALE)
        side.synchronize()
        _assert_same_cache(oc, gc)
        _attn_close(out.cpu().numpy(), oc.attn_decode(q, SCALE))
        gc.close()


@pytest.mark.parametrize("Hq,scale", [(2, 4.0), (8, 4.0), (2, 1e-4), (16, 30.0)])
def test_sharp_and_flat_softmax(gpu, oracle, Hq, scale):
    """Softmax scales far from 1/sqrt(128): with a large scale one token takes nearly all the weight (scores of the
    order of +-10^3, partial maxima that differ by hundreds between waves and splits), with a tiny one the weights
    are uniform.  Buffered tokens take part, so the sharpest token may sit in the fp16 buffer."""
    _say(f"softmax scale {scale}, Hq={Hq}")
    B, H, S = 1, 2, 1500
    Kx, Vx = W.make_kv(B, H, S, 35)
    oc = oracle.OracleCache(B, H, Hq, 1536, 1e-2, 1e-2, 0, 7, buffer_tokens=128)
    gc = gpu.KVCompCache(B, H, Hq, 1536, 1e-2, 1e-2, max_code_len=7, buffer_tokens=128)
    oc.build_codebook(Kx, Vx)
    oc.compress_blocks(Kx, Vx)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    gc.compress_blocks(_dev(Kx), _dev(Vx))
    q = W.make_queries(B, Hq, 1, 35)[0]
    for n_splits in (0, 1, 7):
        gc.set_tuning(n_splits=n_splits)
        err = _attn_close(gc.attn_decode(_dev(q), scale).cpu().numpy(), oc.attn_decode(q, scale))
    _say(f"  max abs err {err:.2e}")
    gc.close()


@pytest.mark.parametrize("G,limit", [(4, 6), (8, 6), (8, 7), (2, 6)])
def test_heads_of_a_group_with_different_sharpness(gpu, oracle, G, limit):
    """The query heads that share a KV head differ by orders of magnitude in how sharp their softmax is, and K grows
    along the sequence so that the largest score of nearly every block exceeds the one before: the running softmax
    reference of the group path (which moves lazily, and whose integer weights share one scale per block across the
    heads) must not cost the other heads their resolution beyond what 22-bit weights under a 30000-fold spread of |q|
    leave: half of the 1e-3 bar (measured 2.7e-4 for groups of 4 and 8, 5e-6 for the per-head path of groups of 2)."""
    _say(f"heads of different sharpness, G={G}, code words <= {limit} bits")
    B, H, S = 1, 2, 64 * 40
    Hq = H * G
    Kx, Vx = W.make_kv(B, H, S, 71)
    ramp = np.linspace(0.25, 2.0, S, dtype=np.float32)[None, :, None, None]
    Kx = (Kx.astype(np.float32) * ramp).astype(np.float16)
    q = W.make_queries(B, Hq, 1, 71)[0].astype(np.float32)
    sharp = np.array([30.0, 0.01, 1.0, 8.0, 0.1, 3.0, 0.001, 15.0], np.float32)[:G]
    q = (q.reshape(B, H, G, 128) * sharp[None, None, :, None]).reshape(B, Hq, 128).astype(np.float16)
    oc = oracle.OracleCache(B, H, Hq, S + 64, 1e-2, 1e-2, 0, limit)
    gc = gpu.KVCompCache(B, H, Hq, S + 64, 1e-2, 1e-2, max_code_len=limit)
    oc.build_codebook(Kx, Vx)
    oc.compress_blocks(Kx, Vx)
    gc.prefill(_dev(Kx), _dev(Vx))
    ref = np.asarray(oc.attn_decode(q, SCALE), np.float64)
    for n_splits in (0, 1, 5):
        gc.set_tuning(n_splits=n_splits)
        out = gc.attn_decode(_dev(q), SCALE).cpu().numpy()
        err = np.abs(out - ref).max()
        assert err <= 5e-4 * max(1.0, np.abs(ref).max()), (n_splits, err)
    _say(f"  max abs err {err:.2e}")
    gc.close()


def test_layers_have_their_own_codebooks(gpu, oracle):
    """One context per layer in a single allocation (Section 3: codebooks are per layer): every layer matches an oracle
    cache of its own data, appends to one layer leave the others untouched, and the codebooks differ between layers
    whose value distributions differ."""
    _say("three layers in one arena, different data and error bounds per call order")
    B, H, Hq, S = 1, 2, 4, 200
    layers = gpu.KVCompLayers(3, B, H, Hq, 320, 1e-2, 2e-2, buffer_tokens=128)
    assert len(layers) == 3
    data, ocs = [], []
    for i in range(3):
        Kx, Vx = W.make_kv(B, H, S, 70 + i)
        if i == 1:   # a layer with a narrow bell inside each unit's range: a different histogram, hence codebook
            Kx = (Kx.astype(np.float32) ** 3 / 64).astype(np.float16)
            Vx = (Vx.astype(np.float32) ** 3 / 64).astype(np.float16)
        data.append((Kx, Vx))
        oc = oracle.OracleCache(B, H, Hq, 320, 1e-2, 2e-2, buffer_tokens=128)
        oc.build_codebook(Kx, Vx)
        oc.compress_blocks(Kx, Vx)
        ocs.append(oc)
    for i in (2, 0, 1):   # any order
        layers[i].build_codebook(_dev(data[i][0]), _dev(data[i][1]))
        layers[i].compress_blocks(_dev(data[i][0]), _dev(data[i][1]))
    kn, vn = W.make_new_tokens(B, H, 70, 70)
    for t in range(70):   # layer 1 grows by 70 tokens (one more block), the others stay
        ocs[1].append_token(kn[t], vn[t])
        layers[1].append_token(_dev(kn[t]), _dev(vn[t]))
    q = W.make_queries(B, Hq, 1, 70)[0]
    for i in range(3):
        _assert_same_cache(ocs[i], layers[i])
        for w in (K, V):
            ln, cd = layers[i].codebook(w)
            np.testing.assert_array_equal(ln, ocs[i].len[w])
            np.testing.assert_array_equal(cd, ocs[i].code[w])
        _attn_close(layers[i].attn_decode(_dev(q), SCALE).cpu().numpy(), ocs[i].attn_decode(q, SCALE))
    assert not np.array_equal(layers[0].codebook(K)[0], layers[1].codebook(K)[0])
    tot = layers.stats()
    assert tot["stored_bytes"] == sum(oc.stats()["stored_bytes"] for oc in ocs)
    assert abs(tot["compression_ratio"] - sum(oc.stats()["raw_bytes"] for oc in ocs) / tot["stored_bytes"]) < 1e-12
    layers.close()


def test_error_paths(gpu):
    import torch
    _say("error paths (all detected on the host or by the kernels' own checks)")
    B, H, S = 1, 2, 128
    Kx, Vx = W.make_kv(B, H, S, 26)
    gc = gpu.KVCompCache(B, H, H, S, 1e-2, 1e-2)
    dK, dV = _dev(Kx), _dev(Vx)
    with pytest.raises(gpu.KvcompError) as e:
        gc.compress_blocks(dK, dV)
    assert e.value.status == gpu.ERR_STATE
    with pytest.raises(gpu.KvcompError) as e:
        gc.attn_decode(_dev(W.make_queries(B, H, 1, 26)[0]), SCALE)
    assert e.value.status == gpu.ERR_STATE
    with pytest.raises(gpu.KvcompError) as e:
        gc.build_codebook(dK[:, :32].contiguous(), dV[:, :32].contiguous())
    assert e.value.status == gpu.ERR_INVALID_ARG
    bad = Kx.copy()
    bad[0, 5, 1, 7] = np.inf
    with pytest.raises(gpu.KvcompError) as e:
        gc.build_codebook(_dev(bad), dV)
    assert e.value.status == gpu.ERR_NONFINITE
    gc.build_codebook(dK, dV)
    big = torch.zeros((B, S + 64, H, 128), dtype=torch.float16, device="cuda:0")
    with pytest.raises(gpu.KvcompError) as e:
        gc.compress_blocks(big, big)
    assert e.value.status == gpu.ERR_CAPACITY
    gc.compress_blocks(dK, dV)
    with pytest.raises(gpu.KvcompError) as e:
        gc.compress_blocks(dK, dV)
    assert e.value.status == gpu.ERR_STATE
    with pytest.raises(gpu.KvcompError) as e:
        gc.append_token(dK[:, 0].contiguous(), dV[:, 0].contiguous())
    assert e.value.status == gpu.ERR_CAPACITY
    with pytest.raises(gpu.KvcompError) as e:   # new codebooks under existing records would invalidate them
        gc.build_codebook(dK, dV)
    assert e.value.status == gpu.ERR_STATE
    gc.reset(keep_codebook=False)
    gc.build_codebook(dK, dV)
    with pytest.raises(gpu.KvcompError):
        gpu.KVCompCache(1, 2, 6, 128, 1e-2, 1e-2)
    gc.close()


def test_nonfinite_token_is_reported_after_its_flush(gpu):
    """An Inf in an appended token: the appends never synchronise, so the flag that the flush's size pass sets is
    reported by the next synchronising call (statistics, decompression), once, and the cache stays usable."""
    _say("Inf in an appended token, reported at the next synchronising call")
    B, H, S = 1, 2, 100
    Kx, Vx = W.make_kv(B, H, S, 36)
    gc = gpu.KVCompCache(B, H, H, 256, 1e-2, 1e-2)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    gc.compress_blocks(_dev(Kx), _dev(Vx))
    kn, vn = W.make_new_tokens(B, H, 40, 36)
    kn[5, 0, 1, 17] = np.inf
    for t in range(27):           # 100 = one block + 36 buffered: the 28th append completes the second block
        gc.append_token(_dev(kn[t]), _dev(vn[t]))
    assert gc.stats()["n_blocks"] == 1     # still buffered: nothing has looked at the token yet
    gc.append_token(_dev(kn[27]), _dev(vn[27]))
    with pytest.raises(gpu.KvcompError) as e:
        gc.stats()
    assert e.value.status == gpu.ERR_NONFINITE
    assert gc.stats()["n_blocks"] == 2     # reported once; the cache goes on
    vn[30, 0, 0, 3] = np.nan
    for t in range(28, 40):
        gc.append_token(_dev(kn[t]), _dev(vn[t]))
    gc.stats()                             # the NaN is still in the fp16 buffer
    for t in range(52):
        gc.append_token(_dev(kn[t % 20 + 6]), _dev(vn[t % 20 + 6]))   # rows without Inf/NaN; flushes the NaN's block
    with pytest.raises(gpu.KvcompError) as e:
        gc.decompress(V, 256)
    assert e.value.status == gpu.ERR_NONFINITE
    gc.close()


def test_flush_replayed_past_the_arena_is_refused(gpu):
    """The interface forbids replaying a captured flush without the eager calls in between: every replay advances the
    arena tail on the device.  The placement kernel bounds it: once the records would run past the arena it writes
    nothing, the next synchronising call reports KVCOMP_ERR_CAPACITY, and after a reset the context works again."""
    import torch
    _say("captured flush replayed until the arena is full")
    B, H, S = 1, 1, 64
    Kx, Vx = W.make_kv(B, H, 128, 37)
    gc = gpu.KVCompCache(B, H, H, 128, 1e-2, 1e-2)
    dK, dV = _dev(Kx), _dev(Vx)
    gc.build_codebook(dK, dV)
    gc.compress_blocks(dK[:, :S].contiguous(), dV[:, :S].contiguous())
    kn, vn = W.make_new_tokens(B, H, 64, 37)
    dkn, dvn = _dev(kn), _dev(vn)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for t in range(64):
            gc.append_token(dkn[t], dvn[t])      # the 64th append compresses the block
    # the arena holds two blocks at the worst case of 12 bits per symbol (about 52 KiB); a replay adds about 12 KiB
    for _ in range(12):
        graph.replay()
    torch.cuda.synchronize()
    with pytest.raises(gpu.KvcompError) as e:
        gc.stats()
    assert e.value.status == gpu.ERR_CAPACITY
    gc.reset(keep_codebook=True)
    gc.compress_blocks(dK, dV)
    assert gc.stats()["n_blocks"] == 2
    gc.close()


@pytest.mark.parametrize("B,H", [(1, 1), (25, 16)])
def test_blocks_that_found_no_room_have_empty_entries(gpu, B, H):
    """The same with few records (placed by the last workgroup) and with many (placed by launches): until the fault is reported,
    no block that was refused has an entry that a reader would follow, and no later one is admitted."""
    import torch
    _say(f"entries of refused blocks, {B} x {H} heads")
    Kx, Vx = W.make_kv(B, H, 128, 38)
    gc = gpu.KVCompCache(B, H, H, 192, 1e-2, 1e-2)
    dK, dV = _dev(Kx), _dev(Vx)
    gc.build_codebook(dK, dV)
    gc.compress_blocks(dK[:, :64].contiguous(), dV[:, :64].contiguous())
    kn, vn = W.make_new_tokens(B, H, 64, 38)
    dkn, dvn, zero = _dev(kn), _dev(vn), torch.zeros((B, H, 128), dtype=torch.float16, device="cuda:0")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for t in range(64):
            gc.append_token(dkn[t], dvn[t])
    for _ in range(16):
        graph.replay()
    torch.cuda.synchronize()
    for which, b, h in ((K, 0, 0), (V, 0, 0), (V, B - 1, H - 1)):
        assert gc.block_entry(which, b, h, 1) == (0, 0)
    for t in range(64):       # smaller records, which would fit
        gc.append_token(zero, zero)
    for which, b, h in ((K, 0, 0), (V, 0, 0), (V, B - 1, H - 1)):
        assert gc.block_entry(which, b, h, 2) == (0, 0)
    with pytest.raises(gpu.KvcompError) as e:
        gc.stats()
    assert e.value.status == gpu.ERR_CAPACITY
    gc.close()


@pytest.mark.parametrize("B,H,Hq,S", [(1, 2, 2, 1000), (2, 2, 8, 300), (1, 1, 8, 64), (1, 4, 8, 4100)])
def test_fp16_baseline_attention(gpu, oracle, B, H, Hq, S):
    """The uncompressed comparison kernel (Section 4.3) against the oracle's attention on the raw fp16 values
    (K' = K, V' = V), to the same bar as the fused kernel; and against an oracle cache whose buffer holds the whole
    sequence, so that nothing is quantized and the oracle's own decode-attention call is the reference."""
    _say(f"fp16 baseline attention B={B} H={H} Hq={Hq} S={S}")
    Kx, Vx = W.make_kv(B, H, S, 27)
    q = W.make_queries(B, Hq, 1, 27)[0]
    G = Hq // H
    ref = np.zeros((B, Hq, 128))
    for b in range(B):
        for hq in range(Hq):
            ref[b, hq] = oracle.attention_head(Kx[b, :, hq // G], Vx[b, :, hq // G], q[b, hq], SCALE)
    if S < 4096:   # the largest buffer the oracle cache takes is 4096 tokens
        window = (S + 64) // 64 * 64
        oc = oracle.OracleCache(B, H, Hq, window, 1e-2, 1e-2, buffer_tokens=window)
        oc.build_codebook(Kx[:, :64] if S >= 64 else np.zeros((B, 64, H, 128), np.float16), Vx[:, :64] if S >= 64
                          else np.zeros((B, 64, H, 128), np.float16))
        oc.compress_blocks(Kx, Vx)
        assert oc.n_blocks == 0 and oc.n_res == S
        np.testing.assert_allclose(oc.attn_decode(q, SCALE), ref, rtol=0, atol=1e-12)
    base = gpu.BaselineFp16Attention(B, H, Hq)
    for n_splits in (0, 1, 5):
        out = base(_dev(Kx), _dev(Vx), _dev(q), SCALE, n_splits=n_splits).cpu().numpy()
        _attn_close(out, ref)


@pytest.mark.parametrize("G", [4, 8])
@pytest.mark.parametrize("S", [1, 15, 17, 63, 65, 257, 700])
def test_fp16_attention_of_large_groups_at_tile_edges(gpu, G, S):
    """Groups of 4 and 8 on the uncompressed cache: sequence lengths around the 16-, 32- and 64-token pieces of a tile, and
    scores that grow along the sequence, so that the softmax reference has to follow (by far more than its slack of 8)
    with sums already made.  Against float64 on the CPU; numerators and sums have fp32's
    resolution: 1e-5 of the largest output."""
    import torch
    B, H = 2, 2
    rng = np.random.default_rng(S * 10 + G)
    Kx = rng.standard_normal((B, S, H, 128)).astype(np.float16)
    Vx = rng.standard_normal((B, S, H, 128)).astype(np.float16)
    q = rng.standard_normal((B, H * G, 128)).astype(np.float16)
    for ramp in (0.0, 60.0):
        Kr = (Kx + (ramp * np.linspace(0, 1, S)[None, :, None, None] * q[:, None, ::G, :] / 128)).astype(np.float16)
        for n_splits in (0, 3):
            out = gpu.BaselineFp16Attention(B, H, H * G)(_dev(Kr), _dev(Vx), _dev(q), 1.0, n_splits=n_splits).cpu().numpy()
            k64, v64, q64 = (torch.from_numpy(x.astype(np.float64)) for x in (Kr, Vx, q))
            for b in range(B):
                for g in range(H * G):
                    p = torch.softmax(k64[b, :, g // G] @ q64[b, g], 0)
                    ref = (p @ v64[b, :, g // G]).numpy()
                    assert np.abs(out[b, g] - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max()), (ramp, n_splits, b, g)


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_fp16_attention_of_small_numerators(gpu, G):
    """Tokens whose numerators are far below the reference count with the resolution of fp32: the reference's tokens have V = 0,
    the others a score 4, 14, 18 or 22 lower (numerators down to 2^-32) and a V of their own channel.  The scores are exact;
    exp is off by half an ulp of the argument times log2 e (22 * 1.44 * 2^-24 = 1.9e-6) and an ulp of its own, the sums over
    140 equal numerators by less than 140 * 2^-24: 1e-5 of every value.  Two fp16 parts would leave 1.5e-5 at 14, 1e-3 at 18."""
    B, H, S = 1, 2, 140
    depth = {5: 4.0, 21: 14.0, 70: 18.0, 139: 22.0}   # token -> how far below; in both halves and the last tile
    Kx, Vx = (np.zeros((B, S, H, 128), np.float16) for _ in range(2))
    q = np.zeros((B, H * G, 128), np.float16)
    q[:, :, 11] = 1.0
    norm = float(S - len(depth)) + sum(np.exp(-d) for d in depth.values())
    ref = np.zeros(128)
    for i, (t, d) in enumerate(depth.items()):
        Kx[:, t, :, 11], Vx[:, t, :, 30 * i + 1] = -d, 32768.0
        ref[30 * i + 1] = 32768.0 * np.exp(-d) / norm
    out = gpu.BaselineFp16Attention(B, H, H * G)(_dev(Kx), _dev(Vx), _dev(q), 1.0).cpu().numpy()
    assert (np.abs(out - ref) <= 1e-5 * ref).all(), out[0, 0][ref > 0] / ref[ref > 0]


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("S", [17, 300, 700])
def test_fp16_attention_with_infinities_in_v(gpu, G, S):
    """An Inf in V, which the uncompressed attention takes as it is: every head of the group gets Inf with its sign in that
    channel, NaN where Infs of both signs meet or V holds a NaN, and the other channels do not notice.  The tokens are in the
    first and last tile of a split, at the softmax reference and (ramp) far below the final one."""
    import torch
    B, H = 1, 2
    rng = np.random.default_rng(S + G)
    Kx = rng.standard_normal((B, S, H, 128)).astype(np.float16)
    Vx = rng.standard_normal((B, S, H, 128)).astype(np.float16)
    q = rng.standard_normal((B, H * G, 128)).astype(np.float16)
    Vx[0, 0, :, 3], Vx[0, S - 1, :, 9], Vx[0, S // 2, 1, 127] = np.inf, -np.inf, np.inf
    Vx[0, S // 3, :, 40], Vx[0, S - 2, :, 40], Vx[0, S // 2, :, 64] = np.inf, -np.inf, np.nan
    for ramp in (0.0, 30.0):
        Kr = (Kx + (ramp * np.linspace(0, 1, S)[None, :, None, None] * q[:, None, ::G, :] / 128)).astype(np.float16)
        k64, v64, q64 = (torch.from_numpy(x.astype(np.float64)) for x in (Kr, Vx, q))
        ref = np.stack([(torch.softmax(k64[0, :, g // G] @ q64[0, g] / 8, 0) @ v64[0, :, g // G]).numpy() for g in range(H * G)])
        assert np.isposinf(ref[:, 3]).all() and np.isneginf(ref[:, 9]).all() and np.isnan(ref[:, [40, 64]]).all()
        for n_splits in (0, 1, 3):
            out = gpu.BaselineFp16Attention(B, H, H * G)(_dev(Kr), _dev(Vx), _dev(q), 0.125, n_splits=n_splits)
            np.testing.assert_allclose(out.cpu().numpy()[0], ref, rtol=0, atol=1e-5, err_msg=f"{ramp} {n_splits}")


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("n_splits,dead", [(2, [1]), (4, [0, 2]), (20, list(range(3, 19)))])
def test_fp16_attention_of_splits_that_score_minus_infinity(gpu, G, n_splits, dead):
    """Splits whose tokens all have score -Inf (K holds -Inf where every query is positive) take no part in the merge."""
    import torch
    B, H, S = 1, 2, 256 * n_splits
    rng = np.random.default_rng(n_splits + G)
    Kx, Vx = (rng.standard_normal((B, S, H, 128)).astype(np.float16) for _ in range(2))
    q = rng.standard_normal((B, H * G, 128)).astype(np.float16)
    q[..., 17] = 1.0
    live = np.ones(S, bool)
    for s in dead:
        Kx[0, 256 * s:256 * (s + 1), :, 17] = -np.inf
        live[256 * s:256 * (s + 1)] = False
    out = gpu.BaselineFp16Attention(B, H, H * G)(_dev(Kx), _dev(Vx), _dev(q), 0.125, n_splits=n_splits).cpu().numpy()
    k64, v64, q64 = (torch.from_numpy(x.astype(np.float64)) for x in (Kx[:, live], Vx[:, live], q))
    for g in range(H * G):
        ref = (torch.softmax(k64[0, :, g // G] @ q64[0, g] / 8, 0) @ v64[0, :, g // G]).numpy()
        assert np.abs(out[0, g] - ref).max() <= 1e-5, g


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("n_splits,first,last", [(1, 0, 64), (1, 64, 128), (1, 192, 256), (1, 256, 500), (2, 0, 64), (2, 256, 512),
                                                 (20, 256 * 3, 256 * 19), (20, 256 * 19, 256 * 20)])
def test_fp16_attention_of_tiles_that_score_minus_infinity_or_nan(gpu, G, n_splits, first, last):
    """Tiles of 64 tokens and splits of 256, a wave's first and later ones: tokens with score -Inf take no part, and NaN scores make
    the output NaN."""
    B, H, S = 1, 2, 256 * n_splits + (300 if n_splits == 1 else 0)
    rng = np.random.default_rng(n_splits + G + first)
    Kx, Vx = (rng.standard_normal((B, S, H, 128)).astype(np.float16) for _ in range(2))
    q = rng.standard_normal((B, H * G, 128)).astype(np.float16)
    q[..., 17] = 1.0
    live = np.ones(S, bool)
    live[first:last] = False
    k64, v64, q64 = (x.astype(np.float64) for x in (Kx[0, live], Vx[0, live], q[0]))
    attn = gpu.BaselineFp16Attention(B, H, H * G)
    Kx[:, ~live, :, 17] = -np.inf
    out = attn(_dev(Kx), _dev(Vx), _dev(q), 0.125, n_splits=n_splits).cpu().numpy()
    for g in range(H * G):
        s = k64[:, g // G] @ q64[g] / 8
        p = np.exp(s - s.max())
        assert np.abs(out[0, g] - p @ v64[:, g // G] / p.sum()).max() <= 1e-5, g
    Kx[:, ~live, :, 17] = np.nan
    assert np.isnan(attn(_dev(Kx), _dev(Vx), _dev(q), 0.125, n_splits=n_splits).cpu().numpy()).all()


def test_config1_full_size_sampled(gpu, oracle):
    """The benchmark workload (32 heads x 4096 tokens) in the launch configuration bench.py times."""
    w = W.CONFIGS["c1"]
    _say("config 1 full size: records sampled, attention on every head")
    Kx, Vx, oc, gc = _both(gpu, oracle, w.batch, w.n_kv_heads, w.n_q_heads, w.seq, w.seq, w.seq, w.rel_eb, w.rel_eb, w.seed,
                           limit=W.CODE_LEN_LIMIT[w.rel_eb])
    _assert_same_cache(oc, gc, sample=200)
    qs = W.make_queries(w.batch, w.n_q_heads, 2, w.seed)
    for i in range(2):
        err = _attn_close(gc.attn_decode(_dev(qs[i]), SCALE).cpu().numpy(), oc.attn_decode(qs[i], SCALE))
        _say(f"  step {i}: max abs err {err:.3e}")
    _say(f"  stats {gc.stats()}")
    gc.close()


@pytest.mark.parametrize("max_len,rel,Hq", [(6, 1e-2, 4), (7, 1e-2, 4), (7, 5e-3, 4), (8, 5e-3, 4), (10, 1e-2, 4),
                                            (12, 1e-2, 4), (6, 1e-2, 2), (5, 2e-2, 2), (5, 2e-2, 4), (6, 1e-2, 8),
                                            (6, 1e-2, 16), (8, 5e-3, 8), (10, 1e-2, 8), (12, 1e-2, 16), (8, 5e-3, 16),
                                            (10, 5e-3, 16)])
def test_code_length_limits_select_every_decoder_variant(gpu, oracle, max_len, rel, Hq):
    """Shorter maximum code words: more symbols per decode window (5, 4, 3, 3, 2 for limits up to 6, 7, 8, 10, 12;
    for every size of query-head group)."""
    _say(f"max_code_len={max_len} rel={rel} Hq={Hq}")
    B, H, S = 1, 2, 330
    Kx, Vx = W.make_kv(B, H, S, 31)
    oc = oracle.OracleCache(B, H, Hq, S + 64, rel, rel, max_code_len=max_len)
    oc.build_codebook(Kx, Vx)
    oc.compress_blocks(Kx, Vx)
    gc = gpu.KVCompCache(B, H, Hq, S + 64, rel, rel, max_code_len=max_len)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    gc.compress_blocks(_dev(Kx), _dev(Vx))
    for which in (K, V):
        ln_g, cd_g = gc.codebook(which)
        np.testing.assert_array_equal(ln_g, oc.len[which])
        np.testing.assert_array_equal(cd_g, oc.code[which])
        assert int(ln_g.max()) <= max_len
    _assert_same_cache(oc, gc)
    q = W.make_queries(B, Hq, 1, 31)[0]
    _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), oc.attn_decode(q, SCALE))
    gc.close()


@pytest.mark.parametrize("G", [1, 4, 8])
def test_long_code_words_and_length_limit(gpu, oracle, G):
    """A geometric code histogram at prefill drives the code words to the 12-bit limit (count halving on both sides);
    the later blocks then use every level, so records are large (above the 8 KiB that the first stage of the record
    staging moves) and the two-symbols-per-window decoder runs, for one query head per KV head and for groups."""
    _say(f"geometric prefill histogram -> 12-bit code words, {G} query heads per KV head")
    B, H, S = 1, 2, 256
    rng = np.random.default_rng(32)
    Kx, Vx = W.make_kv(B, H, S, 32)
    geo = np.minimum(rng.geometric(0.5, size=(B, 64, H, 128)) - 1, 50)   # code k with probability 2^-(k+1)
    kp = geo.astype(np.float16)
    kp[:, 0], kp[:, 1] = 0, 50          # every K unit (channel over the block's tokens) spans [0, 50] -> code == value
    vp = geo.astype(np.float16)
    vp[..., 0], vp[..., 1] = 0, 50      # every V unit (token over the channels) spans [0, 50]
    Kx[:, :64], Vx[:, :64] = kp, vp
    oc = oracle.OracleCache(B, H, G * H, S, 1e-2, 1e-2)
    oc.build_codebook(Kx[:, :64], Vx[:, :64])
    assert oc.halvings[K] > 0 and int(oc.len[K].max()) == 12 and int(oc.len[V].max()) == 12
    oc.compress_blocks(Kx, Vx)
    gc = gpu.KVCompCache(B, H, G * H, S, 1e-2, 1e-2)
    gc.build_codebook(_dev(Kx[:, :64]), _dev(Vx[:, :64]))
    gc.compress_blocks(_dev(Kx), _dev(Vx))
    for which in (K, V):
        ln_g, cd_g = gc.codebook(which)
        np.testing.assert_array_equal(ln_g, oc.len[which])
        np.testing.assert_array_equal(cd_g, oc.code[which])
    _assert_same_cache(oc, gc)
    q = W.make_queries(B, G * H, 1, 32)[0]
    _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), oc.attn_decode(q, SCALE))
    _say(f"  largest record {gc.stats()['max_record_bytes']} B, CR {gc.stats()['compression_ratio']:.3f}")
    gc.close()


@pytest.mark.parametrize("H,Hq", [(2, 2), (1, 4), (1, 8)])
@pytest.mark.parametrize("k_scale,q_scale,v_scale", [(256.0, 1.0 / 256.0, 64.0), (1.0 / 64.0, 64.0, 1.0 / 32.0)])
def test_attention_with_large_and_small_magnitudes(gpu, oracle, H, Hq, k_scale, q_scale, v_scale):
    """K, q and V scaled by powers of two: the scores do not change, the folded weights (q step, p step) move by
    several binades (the query-group path keeps them as scaled fp16 pairs)."""
    _say(f"scaled inputs H={H} Hq={Hq} k x{k_scale} q x{q_scale} v x{v_scale}")
    B, S = 1, 777
    Kx, Vx = W.make_kv(B, H, S, 41)
    Kx = (Kx.astype(np.float32) * k_scale).astype(np.float16)
    Vx = (Vx.astype(np.float32) * v_scale).astype(np.float16)
    q = (W.make_queries(B, Hq, 1, 41)[0].astype(np.float32) * q_scale).astype(np.float16)
    assert np.isfinite(Kx.astype(np.float32)).all() and np.isfinite(Vx.astype(np.float32)).all()
    oc = oracle.OracleCache(B, H, Hq, 1024, 1e-2, 1e-2, 0, 7)
    oc.build_codebook(Kx, Vx)
    oc.compress_blocks(Kx, Vx)
    gc = gpu.KVCompCache(B, H, Hq, 1024, 1e-2, 1e-2, max_code_len=7)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    gc.compress_blocks(_dev(Kx), _dev(Vx))
    _assert_same_cache(oc, gc)
    err = _attn_close(gc.attn_decode(_dev(q), SCALE).cpu().numpy(), oc.attn_decode(q, SCALE))
    _say(f"  max abs err {err:.3e}")
    gc.close()


@pytest.mark.parametrize("H,Hq,max_len", [(2, 2, 12), (1, 4, 9), (1, 8, 7)])
def test_block_quant_k(gpu, oracle, H, Hq, max_len):
    """K with one quantization range per 2D block (BlockQuant, Section 4.2): codes, range, codebook, records (their
    header holds one {min,max} pair), attention, and the append path with a flush."""
    _say(f"BlockQuant K: H={H} Hq={Hq} max code word {max_len}")
    B, S, rel = 2, 200, 1e-2
    Kx, Vx = W.make_kv(B, H, S, 51)
    Kx[1, 64:128, 0, :] = np.float16(-2.5)  # a constant K block
    oc = oracle.OracleCache(B, H, Hq, 320, rel, rel, 1, max_len)
    gc = gpu.KVCompCache(B, H, Hq, 320, rel, rel, k_mode=1, max_code_len=max_len)
    oc.build_codebook(Kx, Vx)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    codes_o, mm_o = oracle.tensor_quantize(K, Kx, rel, k_mode=1)
    codes_g, mm_g = gc.debug_codes(K, _dev(Kx))
    assert mm_g.shape == mm_o.shape == (B * H * (S // 64), 1, 2)
    np.testing.assert_array_equal(mm_g, mm_o)
    np.testing.assert_array_equal(codes_g, codes_o)
    for which in (K, V):
        ln_g, cd_g = gc.codebook(which)
        np.testing.assert_array_equal(ln_g, oc.len[which])
        np.testing.assert_array_equal(cd_g, oc.code[which])
    oc.compress_blocks(Kx, Vx)
    gc.compress_blocks(_dev(Kx), _dev(Vx))
    _assert_same_cache(oc, gc)
    kn, vn = W.make_new_tokens(B, H, 70, 51)
    qs = W.make_queries(B, Hq, 70, 51)
    for t in range(70):
        oc.append_token(kn[t], vn[t])
        gc.append_token(_dev(kn[t]), _dev(vn[t]))
        if t in (0, 55, 56, 69):  # the flush happens at t = 55
            err = _attn_close(gc.attn_decode(_dev(qs[t]), SCALE).cpu().numpy(), oc.attn_decode(qs[t], SCALE))
            _say(f"  step {t}: max abs err {err:.3e}")
    _assert_same_cache(oc, gc)
    st = gc.stats()
    _say(f"  CR {st['compression_ratio']:.3f}, K bits/symbol {st['payload_bits_k'] / (B * H * oc.n_blocks * 8192.0):.2f}")
    gc.close()


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("limit", [6, 7, 8, 10, 12])
def test_streams_of_short_and_of_very_unequal_slices(gpu, oracle, G, limit):
    """Codes with probability 2^-(k+1) in every block: the shortest code words of every table width, so that a chain's 32
    symbols end inside the first 64-bit unit or two of its stream, next to slices with every long code word; whole rows and
    columns of code 0, whose slices are as short as a slice can be, at both ends of the records too."""
    _say(f"short and unequal slices, code words of up to {limit} bits, {G} query heads per KV head")
    B, H, S = 1, 2, 64 * 9
    rng = np.random.default_rng(41 + limit)
    Kx, Vx = W.make_kv(B, H, S, 41)
    for X, unit_axis in ((Kx, "token"), (Vx, "channel")):
        geo = np.minimum(rng.geometric(0.5, size=X.shape) - 1, 50).astype(np.float16)
        long_rows = rng.random((B, S, 1, 128)) < (0.1 if limit <= 8 else 0.01)   # rare enough for the longest code words
        geo = np.where(long_rows, rng.integers(0, 51, X.shape), np.minimum(geo, 12)).astype(np.float16)
        geo[:, 60:64] = 0               # the last tokens (K: the last slices) of the first block
        geo[..., 120:] = 0              # the last channels (V: the last slices) of every block
        if unit_axis == "token":        # every K unit (channel over a block's tokens) spans [0, 50] -> code == value
            geo[:, 0::64], geo[:, 1::64] = 0, 50
        else:                           # every V unit (token over the channels) too
            geo[..., 0], geo[..., 1] = 0, 50
        X[...] = geo
    oc = oracle.OracleCache(B, H, G * H, S + 64, 1e-2, 1e-2, 0, limit)
    gc = gpu.KVCompCache(B, H, G * H, S + 64, 1e-2, 1e-2, max_code_len=limit)
    oc.build_codebook(Kx, Vx)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    assert all(int(oc.len[w][:51].min()) <= 3 and int(oc.len[w].max()) == limit for w in (K, V))
    for j in (3, 6):                # two blocks of any code: records longer than a small staging area
        for X in (Kx, Vx):
            X[:, 64 * j:64 * (j + 1)] = rng.integers(0, 51, (B, 64, H, 128))
        Kx[:, 64 * j], Kx[:, 64 * j + 1] = 0, 50
        Vx[:, 64 * j:64 * (j + 1), :, 0], Vx[:, 64 * j:64 * (j + 1), :, 1] = 0, 50
    oc.compress_blocks(Kx, Vx)
    gc.compress_blocks(_dev(Kx), _dev(Vx))
    sizes = [[gc.block_entry(w, 0, 1, j)[1] * 16 for j in range(9)] for w in (K, V)]
    assert all(z[j] > 4608 for z in sizes for j in (3, 6))
    assert limit == 6 or all(min(z) < 4608 - 32 for z in sizes)    # and records that fit it beside them
    for which in (K, V):
        got = gc.decompress(which, S).cpu().numpy()
        np.testing.assert_array_equal(got.view(np.uint16), oc.decompress(which).view(np.uint16))
    q = W.make_queries(B, G * H, 1, 41)[0]
    want = oc.attn_decode(q, 1e-3)
    _attn_close(gc.attn_decode(_dev(q), 1e-3).cpu().numpy(), want)
    for waves in (0, 1, 3):                        # a wave for each pair, nine and three pairs one after the other
        for stage_bytes in (0, 4608):              # records staged whatever their length, and long ones from global memory
            gc.set_tuning(n_splits=1, waves=waves, stage_bytes=stage_bytes)
            _attn_close(gc.attn_decode(_dev(q), 1e-3).cpu().numpy(), want)
    gc.close()


@pytest.mark.parametrize("B,H,S,k_mode,max_len", [(2, 2, 200, 0, 7), (1, 3, 333, 1, 10), (1, 1, 64, 0, 12)])
def test_stand_alone_decompression(gpu, oracle, B, H, S, k_mode, max_len):
    """The decompressed cache (blocks reconstructed in fp16, then the buffered tokens) is bit-identical to the
    oracle's, and the fp16 attention kernel on it (the multi-kernel pipeline) agrees with the oracle's attention up
    to the fp16 rounding of the reconstructed values."""
    _say(f"decompress B={B} H={H} S={S} k_mode={k_mode} max code word {max_len}")
    Kx, Vx = W.make_kv(B, H, S, 61)
    oc = oracle.OracleCache(B, H, H, S + 64, 1e-2, 2e-2, k_mode, max_len)
    gc = gpu.KVCompCache(B, H, H, S + 64, 1e-2, 2e-2, k_mode=k_mode, max_code_len=max_len)
    oc.build_codebook(Kx, Vx)
    oc.compress_blocks(Kx, Vx)
    gc.build_codebook(_dev(Kx), _dev(Vx))
    gc.compress_blocks(_dev(Kx), _dev(Vx))
    kn, vn = W.make_new_tokens(B, H, 5, 61)
    for t in range(5):
        oc.append_token(kn[t], vn[t])
        gc.append_token(_dev(kn[t]), _dev(vn[t]))
    tokens = S + 5
    dec = {}
    for which in (K, V):
        ref = oc.decompress(which)
        got = gc.decompress(which, tokens)
        assert tuple(got.shape) == ref.shape == (B, tokens, H, 128)
        np.testing.assert_array_equal(got.cpu().numpy().view(np.uint16), ref.view(np.uint16))
        walked = gc.decompress(which, tokens, tree_walk=True)   # the bit-serial tree walk gives the same bits
        np.testing.assert_array_equal(walked.cpu().numpy().view(np.uint16), ref.view(np.uint16))
        dec[which] = got
    with pytest.raises(gpu.KvcompError) as e:
        gc.decompress(K, tokens - 1)
    assert e.value.status == gpu.ERR_CAPACITY
    q = W.make_queries(B, H, 1, 61)[0]
    out = gpu.BaselineFp16Attention(B, H, H)(dec[K], dec[V], _dev(q), SCALE).cpu().numpy()
    ref = np.asarray(oc.attn_decode(q, SCALE))
    assert np.abs(out - ref).max() <= 2e-3 * max(1.0, np.abs(ref).max())   # values rounded to fp16: 2^-11 relative each
    gc.close()


def _staging(oc):
    """the staging area that the largest record of the cache asks for"""
    largest = max((16 * int(oc.size16[w][:, :oc.n_blocks].max()) for w in (K, V)), default=0) if oc.n_blocks else 0
    return (largest + 16 + 255) // 256 * 256


def _rare_tokens(B, H, n, seed):
    """tokens whose codes lie at both ends: long code words of a codebook that was built on normal samples"""
    rng = np.random.default_rng(seed)
    shape = (n, B, H, 128)
    return [(rng.choice([-1.0, 1.0], shape) * rng.uniform(0.9, 1.0, shape)).astype(np.float16) for _ in range(2)]


@pytest.mark.parametrize("look", [False, True])
@pytest.mark.parametrize("B,H,S,rel,limit", [(1, 3, 192, 2e-3, 8), (1, 1, 320, 2e-3, 12), (3, 1, 130, 1e-2, 6),
                                             (1, 5, 64, 5e-3, 10), (1, 2, 63, 1e-2, 12)])
def test_decompression_widths_and_partial_workgroups(gpu, oracle, B, H, S, rel, limit, look):
    """Every table width, more than 128 levels (codes beyond int8), block counts that leave waves of the last workgroup
    idle or that are none, and a flush between two decompressions that makes a record outgrow the staging area of before, with
    a statistics call, which reads the control words, in between (look) and without.  Bit for bit against the oracle."""
    Kx, Vx, oc, gc = _both(gpu, oracle, B, H, H, max(S, 64), S, S + 64, rel, rel, seed=71, limit=limit)
    kn, vn = _rare_tokens(B, H, 64, 72)
    staging = _staging(oc)
    for step in range(2):
        for which in (K, V):
            got = gc.decompress(which, oc.n_blocks * 64 + oc.n_res).cpu().numpy()
            np.testing.assert_array_equal(got.view(np.uint16), oc.decompress(which).view(np.uint16))
        if step == 0:
            for t in range(64):
                oc.append_token(kn[t], vn[t])
                gc.append_token(_dev(kn[t]), _dev(vn[t]))
            assert _staging(oc) > staging or limit == 8   # 251 levels in 8 bits: no code word is much longer than another
            if look:
                gc.stats()
    gc.close()


def test_decompression_after_replays_of_a_captured_flush(gpu, oracle):
    """A flush inside a graph enlarges a record whenever the graph is replayed, and the host does not see it: decompression
    looks at the control words every time from then on.  Replays start from the state of the capture and are followed by an
    eager refill, as the interface asks."""
    import torch
    _say("decompression around replays of a captured flush")
    B, H = 1, 2
    Kx, Vx, oc, gc = _both(gpu, oracle, B, H, H, 64, 64, 192, 5e-3, 5e-3, seed=78, limit=10)
    kn, vn = _rare_tokens(B, H, 64, 79)
    dK, dV, dkn, dvn = _dev(Kx), _dev(Vx), _dev(kn), _dev(vn)
    before = [oc.decompress(w).view(np.uint16).copy() for w in (K, V)]
    staging = _staging(oc)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for t in range(64):
            gc.append_token(dkn[t], dvn[t])
    for t in range(64):
        oc.append_token(kn[t], vn[t])
    assert _staging(oc) > staging
    for _ in range(3):
        gc.reset()
        gc.compress_blocks(dK, dV)
        graph.replay()
        for w in (K, V):    # the host's view: the first block
            assert np.array_equal(gc.decompress(w, 64).cpu().numpy().view(np.uint16), before[w])
        gc.reset()
        gc.compress_blocks(dK, dV)
        for t in range(64):
            gc.append_token(dkn[t], dvn[t])
        for w in (K, V):
            np.testing.assert_array_equal(gc.decompress(w, 128).cpu().numpy().view(np.uint16), oc.decompress(w).view(np.uint16))
    gc.close()


def test_decompression_after_a_flush_that_another_stream_did_not_wait_for(gpu, oracle):
    """The control words are read on one stream while the flush that enlarges a record still waits on another: the
    decompression behind the flush must look again."""
    import torch
    _say("statistics on a stream of their own while a flush waits")
    B, H = 1, 2
    Kx, Vx, oc, gc = _both(gpu, oracle, B, H, H, 64, 64, 192, 2e-3, 2e-3, seed=75, limit=12)
    kn, vn = W.make_new_tokens(B, H, 64, 76)
    kn, vn = (kn * 50).astype(np.float16), (vn ** 3).astype(np.float16)  # rare codes: longer records
    dkn, dvn = _dev(kn), _dev(vn)
    dK, dV = _dev(Kx), _dev(Vx)
    largest = gc.stats()["max_record_bytes"]
    for attempt in range(8):                   # two streams may share a hardware queue, and then nothing overtakes
        gc.reset()
        gc.compress_blocks(dK, dV)
        torch.cuda.synchronize()
        behind, aside = torch.cuda.Stream(), torch.cuda.Stream()
        with torch.cuda.stream(behind):
            torch.cuda._sleep(20_000_000)      # some ten milliseconds
            for t in range(64):
                gc.append_token(dkn[t], dvn[t])
        with torch.cuda.stream(aside):
            overtook = gc.stats()["max_record_bytes"] == largest
        with torch.cuda.stream(behind):
            got = [gc.decompress(w, 128).cpu().numpy() for w in (K, V)]
        assert gc.stats()["max_record_bytes"] > largest
        if overtook:
            break
    else:
        pytest.skip("no two streams that overtake each other")
    for t in range(64):
        oc.append_token(kn[t], vn[t])
    for w in (K, V):
        np.testing.assert_array_equal(got[w].view(np.uint16), oc.decompress(w).view(np.uint16))
    gc.close()


@pytest.mark.parametrize("size16", [600, 0x10000000, 0xffffffff])
@pytest.mark.parametrize("tree_walk", [False, True])
def test_refused_block_is_reported_by_the_next_decompression(gpu, oracle, size16, tree_walk):
    """A Block Offsets Array entry whose size exceeds every staging area (one written over here; the kernel's own check refuses
    it, also where 16 * size wraps): the block comes out as NaN, the others as they are, and the next decompression, of
    whichever tensor, reports it once."""
    import torch
    _say(f"damaged block entry, size {size16:#x}")
    B, H, S = 2, 3, 200
    _, _, oc, gc = _both(gpu, oracle, B, H, H, S, S, 256, 1e-2, 1e-2, 77)
    off, size = gc.block_entry(K, 1, 2, 1)
    table = gc.arena[: gc.arena.numel() // 8 * 8].view(torch.int64)
    at = torch.nonzero(table == off + (size << 32)).flatten().tolist()
    assert len(at) == 1
    words = gc.arena[8 * at[0]:8 * at[0] + 8].view(torch.int32)
    words[1] = size16 - (1 << 32 if size16 >> 31 else 0)
    assert gc.block_entry(K, 1, 2, 1) == (off, size16)
    want = oc.decompress(K).view(np.uint16).copy()
    got = gc.decompress(K, S, tree_walk=tree_walk).cpu().numpy()
    assert np.isnan(got[1, 64:128, 2]).all()
    got[1, 64:128, 2] = want.view(np.float16)[1, 64:128, 2]
    np.testing.assert_array_equal(got.view(np.uint16), want)
    with pytest.raises(gpu.KvcompError) as e:
        gc.decompress(V, S, tree_walk=tree_walk)
    assert e.value.status == gpu.ERR_STATE
    words[1] = size
    for w in (K, V):
        got = gc.decompress(w, S, tree_walk=tree_walk).cpu().numpy()
        np.testing.assert_array_equal(got.view(np.uint16), oc.decompress(w).view(np.uint16))
    gc.close()


def test_decompression_of_blocks_is_not_captured(gpu, oracle):
    """A graph would freeze the staging area and the block count, so decompressing blocks under capture is refused; the capture
    itself goes on, and decompressing buffered tokens alone can be captured."""
    import torch
    _say("decompression under stream capture")
    _, _, oc, gc = _both(gpu, oracle, 1, 2, 2, 130, 130, 256, 1e-2, 1e-2, 73)
    Kx, Vx, _, few = _both(gpu, oracle, 1, 2, 2, 64, 20, 256, 1e-2, 1e-2, 74)
    out, tail = (torch.zeros((1, n, 2, 128), dtype=torch.float16, device="cuda:0") for n in (130, 20))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for tree_walk in (False, True):
            with pytest.raises(gpu.KvcompError) as e:
                gc.decompress(K, 130, out=out, tree_walk=tree_walk)
            assert e.value.status == gpu.ERR_HIP
        few.decompress(V, 20, out=tail)
    for _ in range(3):
        tail.zero_()
        graph.replay()
        assert np.array_equal(tail.cpu().numpy().view(np.uint16), Vx[:, :20].view(np.uint16))
    assert torch.count_nonzero(out) == 0
    got = gc.decompress(K, 130, out=out).cpu().numpy()
    np.testing.assert_array_equal(got.view(np.uint16), oc.decompress(K).view(np.uint16))
    gc.close()
    few.close()


@pytest.mark.parametrize("name,rel", [("c2", 1e-2), ("c2", 5e-3), ("c2", 2e-2), ("c3", 1e-2), ("c4", 1e-2)])
def test_large_configs_full_size_sampled(gpu, oracle, name, rel):
    """The long-context (with its error-bound sweep), grouped-query and 70B-shaped workloads at their full prompt
    size, in the launch configuration bench.py times (automatic splits, the code word limit of workloads.CODE_LEN_LIMIT).  The oracle quantizes
    the whole tensors (the codebooks depend on all of it); records are compared on a sample of blocks and the
    attention output on five (batch, kv head) pairs -- the two ends and three from the middle of the range, so that
    every part of the kernel's workgroup numbering is covered -- which the oracle recomputes from its own compressed
    copy of those heads."""
    w = W.CONFIGS[name]
    assert rel in W.C2_REL_EB_SWEEP and (name == "c2" or rel == w.rel_eb)
    B, H, Hq, S = w.batch, w.n_kv_heads, w.n_q_heads, w.seq
    G = Hq // H
    limit = W.CODE_LEN_LIMIT[rel]
    _say(f"{name} full size: B={B} H={H} Hq={Hq} S={S} rel_eb={rel} code words <= {limit} bits")
    Kx, Vx = W.make_kv(B, H, S, w.seed)
    gc = gpu.KVCompCache(B, H, Hq, S + 64, rel, rel, max_code_len=limit)
    dK, dV = _dev(Kx), _dev(Vx)
    gc.build_codebook(dK, dV)
    gc.compress_blocks(dK, dV)
    # the same prompt through the one-pass entry point that bench.py times (sizes from block histograms, placement in
    # several chunks, K written before V is sized): must give the same cache
    gp = gpu.KVCompCache(B, H, Hq, S + 64, rel, rel, max_code_len=limit)
    gp.prefill(dK, dV)
    del dK, dV
    st_c, st_p = gc.stats(), gp.stats()
    for key in ("n_blocks", "n_res", "record_bytes_k", "record_bytes_v", "payload_bits_k", "payload_bits_v", "stored_bytes"):
        assert st_c[key] == st_p[key], key
    _say("  gpu compressed; oracle quantizes")
    NB = S // 64
    book, codes, mms = {}, {}, {}
    for which, X in ((K, Kx), (V, Vx)):
        codes[which], mms[which] = oracle.tensor_quantize(which, X, rel)
        hist = oracle.histogram(codes[which])
        np.testing.assert_array_equal(gc.histogram(which).astype(np.uint64), hist)
        ln, cd, _ = oracle.build_codebook(hist, oracle.n_sym(rel), limit)
        ln_g, cd_g = gc.codebook(which)
        np.testing.assert_array_equal(ln_g, ln)
        np.testing.assert_array_equal(cd_g, cd)
        book[which] = (ln, cd)
    # Placement at full size: the record size of EVERY block from the oracle's codes and code lengths (the sampled
    # records below pin this size against oracle.encode_block), offsets by a running sum in (tensor, batch, head,
    # block) order; the device's Block Offsets Array is compared on the sample and on the very last entry.
    hdr = {K: 4 * 128 + 2 * 128, V: 4 * 64 + 2 * 128}
    size16 = {}
    for which in (K, V):
        ln8 = book[which][0].astype(np.uint8)
        bits = ln8[codes[which].reshape(B * H * NB, -1)].sum(axis=1, dtype=np.int64)
        size16[which] = (hdr[which] + 4 * ((bits + 31) // 32) + 15) // 16
    off16 = np.concatenate([[0], np.cumsum(np.concatenate([size16[K], size16[V]]))])
    rng = np.random.default_rng(5)
    picks = [(int(rng.integers(2)), int(rng.integers(B)), int(rng.integers(H)), int(rng.integers(NB))) for _ in range(48)]
    picks += [(K, 0, 0, 0), (K, B - 1, H - 1, NB - 1), (V, 0, 0, 0), (V, B - 1, H - 1, NB - 1)]
    for which, b, h, j in picks:
        i = (b * H + h) * NB + j
        rec = oracle.encode_block(which, codes[which][i], mms[which][i], *book[which])
        assert (len(rec) + 15) // 16 == size16[which][i]
        want = (int(off16[which * B * H * NB + i]), int(size16[which][i]))
        assert gc.block_entry(which, b, h, j) == want, (which, b, h, j)
        assert gp.block_entry(which, b, h, j) == want, (which, b, h, j)
        for cache in (gc, gp):
            got = cache.get_block(which, b, h, j)
            assert len(got) == (len(rec) + 15) // 16 * 16
            np.testing.assert_array_equal(got[: len(rec)], rec)
            assert not got[len(rec):].any()
    gp.close()
    del codes, mms
    q = W.make_queries(B, Hq, 1, w.seed)[0]
    out = gc.attn_decode(_dev(q), SCALE).cpu().numpy()
    sampled = {}
    BH = B * H
    pairs = sorted({0, BH - 1, BH // 2, BH // 3 + 1, (5 * BH) // 8 + 2})
    for b, h in ((i // H, i % H) for i in pairs):
        oc = oracle.OracleCache(1, 1, G, S + 64 + w.append_steps, rel, rel, 0, limit)
        oc.len, oc.code = [book[K][0], book[V][0]], [book[K][1], book[V][1]]
        oc.compress_blocks(np.ascontiguousarray(Kx[b:b + 1, :, h:h + 1]), np.ascontiguousarray(Vx[b:b + 1, :, h:h + 1]))
        ref = oc.attn_decode(np.ascontiguousarray(q[b:b + 1, h * G:(h + 1) * G]), SCALE)
        err = _attn_close(out[b:b + 1, h * G:(h + 1) * G], ref)
        # well inside the 1e-3 bar: the kernels' own error is a few 1e-5 at most (integer weights of 22 bits, fp32
        # accumulation); a tenfold loss of weight resolution would still pass the bar on these inputs and is caught here
        assert err <= 2e-4 * max(1.0, float(np.abs(np.asarray(ref)).max())), err
        _say(f"  (b={b}, h={h}): attention max abs err {err:.3e}")
        sampled[(b, h)] = oc
    gc.close()
    if not w.append_steps:
        return
    # the streaming phase at full size: every decode step appends one token per sequence (a full buffer is compressed
    # with the prompt's codebooks) and attends; the sampled heads are followed by oracle caches of their own
    T = w.append_steps
    _say(f"  streaming: {T} decode steps")
    gc = gpu.KVCompCache(B, H, Hq, S + T, rel, rel, max_code_len=limit)
    dK, dV = _dev(Kx), _dev(Vx)
    gc.build_codebook(dK, dV)
    gc.compress_blocks(dK, dV)
    del dK, dV
    kn, vn = W.make_new_tokens(B, H, T, w.seed)
    qs = W.make_queries(B, Hq, T, w.seed)
    dkn, dvn, dq = _dev(kn), _dev(vn), _dev(qs)
    check = {0, 62, 63, 64, 255, 256, T - 1}
    outs = {}
    for t in range(T):
        o = gc.append_attn_decode(dkn[t], dvn[t], dq[t], SCALE)
        if t in check:
            outs[t] = o.cpu().numpy()
    st = gc.stats()
    assert st["n_blocks"] == (S + T) // 64 and st["n_res"] == (S + T) % 64
    for (b, h), oc in sampled.items():
        worst = 0.0
        for t in range(T):
            oc.append_token(kn[t][b:b + 1, h:h + 1], vn[t][b:b + 1, h:h + 1])
            if t in check:
                ref = oc.attn_decode(np.ascontiguousarray(qs[t][b:b + 1, h * G:(h + 1) * G]), SCALE)
                worst = max(worst, _attn_close(outs[t][b:b + 1, h * G:(h + 1) * G], ref))
                assert worst <= 2e-4 * max(1.0, float(np.abs(np.asarray(ref)).max())), worst
        for which in (K, V):
            for j in range(NB, oc.n_blocks):   # the blocks compressed while streaming
                np.testing.assert_array_equal(gc.get_block(which, b, h, j), oc.get_block(which, 0, 0, j))
        _say(f"  (b={b}, h={h}): {oc.n_blocks - NB} streamed blocks bit-exact, attention max abs err {worst:.3e}")
    gc.close()
