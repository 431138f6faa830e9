"""Autoregressive decode against a key/value cache, on the GPU through the C ABI.

What decode computes has a plain definition: with a causal mask, position t of the full
forward over a sequence depends on positions <= t only, so the output of a decode step at
position t must equal row t of the oracle's causal forward over the whole sequence.  The
oracle is used as it stands (no decode-specific code in it)."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from oracle import stack_oracle as O  # noqa: E402
from paper_2410_08791_amd import binding as sp  # noqa: E402
from paper_2410_08791_amd import synth  # noqa: E402
from tests.gpu_util import DEV, dev_f32, dev_u16, host_u16, bf16_vals, max_rel, ptr, rand_bf16, stack_errs, stream_ptr  # noqa: E402

TOL = 2e-2


def both(got, ref, x):
    """Error against max |ref| and against what the stack added to its input; both <= TOL."""
    d = ref.shape[-1]
    e = stack_errs(got.reshape(-1, d), ref.reshape(-1, d), x.reshape(-1, d))
    return max(e["out"], e["contrib"])


@pytest.mark.parametrize("B,n,max_len,Hq,Hkv,hd", [
    (2, 1, 8, 4, 4, 64), (3, 77, 128, 4, 2, 64), (2, 600, 1024, 8, 2, 128), (1, 1024, 1024, 2, 1, 128),
    (1, 4099, 4104, 2, 2, 64),
])
def test_append_and_single_query_attention(B, n, max_len, Hq, Hkv, hd):
    """Cache n positions with spk_kv_append (in two chunks), then attend the last position's
    query: equals the last row of the oracle's causal attention over the n positions."""
    rng = np.random.default_rng(n * 7 + Hq)
    ld = (Hq + 2 * Hkv) * hd
    bits, vals = rand_bf16(rng, (B, n, ld))
    shape = O.StackShape("decoder", 1, Hq * hd, Hq, Hkv, hd, 64, True, 1e-5)
    q = vals[:, :, :Hq * hd].reshape(B * n, Hq * hd)
    k = vals[:, :, Hq * hd:(Hq + Hkv) * hd].reshape(B * n, Hkv * hd)
    v = vals[:, :, (Hq + Hkv) * hd:].reshape(B * n, Hkv * hd)
    ref = O.attention(q, k, v, B, n, shape).reshape(B, n, Hq * hd)[:, -1]

    kt = torch.zeros(B * Hkv * hd * max_len, dtype=torch.int16, device=DEV)
    vc = torch.zeros(B * Hkv * max_len * hd, dtype=torch.int16, device=DEV)
    cut = n // 3
    for lo, hi in [(0, cut), (cut, n)]:
        if hi > lo:
            chunk = dev_u16(np.ascontiguousarray(bits[:, lo:hi]).reshape(-1))
            assert sp.spk_kv_append(stream_ptr(), ptr(chunk), ptr(kt), ptr(vc), B, hi - lo, lo, Hq, Hkv, hd,
                                    max_len) == sp.SP_OK
    # cache contents, bit for bit
    kt_h = host_u16(kt).reshape(B, Hkv, hd, max_len)[..., :n]
    vc_h = host_u16(vc).reshape(B, Hkv, max_len, hd)[:, :, :n]
    kb = bits[:, :, Hq * hd:(Hq + Hkv) * hd].reshape(B, n, Hkv, hd)
    vb = bits[:, :, (Hq + Hkv) * hd:].reshape(B, n, Hkv, hd)
    assert np.array_equal(kt_h, kb.transpose(0, 2, 3, 1)) and np.array_equal(vc_h, vb.transpose(0, 2, 1, 3))

    last = dev_u16(np.ascontiguousarray(bits[:, -1]).reshape(-1))
    o = torch.zeros(B * Hq * hd, dtype=torch.int16, device=DEV)
    assert sp.spk_decode_attention(stream_ptr(), ptr(last), ptr(kt), ptr(vc), ptr(o), B, n, max_len, Hq, Hkv,
                                   hd) == sp.SP_OK
    torch.cuda.synchronize()
    got = bf16_vals(host_u16(o)).reshape(B, Hq * hd)
    err = max_rel(got, ref)
    print(f"decode attention B={B} n={n} Hq/Hkv={Hq}/{Hkv} hd={hd}: max rel err {err:.3e}")
    assert err <= 8e-3          # one bf16 rounding of the output


@pytest.mark.parametrize("B,n,max_len,Hq,Hkv,hd,lo,hi", [
    (*c, lo, hi) for c in ((1, 700, 704, 2, 1, 64), (2, 1500, 1504, 4, 4, 128), (1, 900, 904, 8, 1, 128))
    for lo, hi in ((0, 129), (300, 560), (0, 39), (1, 699))
] + [(1, 40, 48, 3, 1, 64, 0, 39), (1, 40, 48, 3, 1, 64, 5, 30)])
def test_decode_attention_infinite_keys_and_values(B, n, max_len, Hq, Hkv, hd, lo, hi):
    """Positions whose score is -inf (an infinite key element against a positive query element) have weight 0,
    also where they are all that a wave holds; an infinite value of the last position reaches its own element
    of the output and no other."""
    rng = np.random.default_rng(n + lo)
    q = np.abs(rng.standard_normal((B, Hq, hd))) * 0.5
    k, v = rng.standard_normal((B, Hkv, n, hd)), rng.standard_normal((B, Hkv, n, hd))
    rnd = lambda a: synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(a.astype(np.float32))).astype(np.float64)  # noqa: E731
    q, k, v = rnd(q), rnd(k), rnd(v)
    s = np.einsum("bgrd,bgnd->bgrn", q.reshape(B, Hkv, Hq // Hkv, hd), k) / np.sqrt(hd)
    s[..., lo:hi] = -np.inf
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    ref = np.einsum("bgrn,bgnd->bgrd", p, v).reshape(B, Hq, hd)
    k[:, :, lo:hi, 5] = -np.inf
    v[:, :, n - 1, 9] = np.inf
    kc, vc = np.full((B, Hkv, hd, max_len), np.nan), np.full((B, Hkv, max_len, hd), np.nan)
    kc[..., :n], vc[:, :, :n] = k.transpose(0, 1, 3, 2), v
    bits = lambda a: dev_u16(synth.f32_to_bf16_bits(a.astype(np.float32)).reshape(-1))  # noqa: E731
    qd = bits(np.concatenate([q.reshape(B, -1), np.zeros((B, 2 * Hkv * hd))], axis=1))
    kd, vd = bits(kc), bits(vc)
    o = torch.zeros(B * Hq * hd, dtype=torch.int16, device=DEV)
    assert sp.spk_decode_attention(stream_ptr(), ptr(qd), ptr(kd), ptr(vd), ptr(o), B, n, max_len, Hq, Hkv, hd) == sp.SP_OK
    torch.cuda.synchronize()
    got = bf16_vals(host_u16(o)).reshape(B, Hq, hd)
    assert np.all(got[..., 9] == np.inf)
    keep = np.arange(hd) != 9
    assert max_rel(got[..., keep], ref[..., keep]) <= 8e-3          # one bf16 rounding of the output


def single_query_ref(q, k, v):
    """Float64 attention of one query per sequence: q [B, Hq, hd], k and v [B, Hkv, n, hd]."""
    B, Hq, hd = q.shape
    Hkv = k.shape[1]
    s = np.matmul(q.reshape(B, Hkv, Hq // Hkv, hd), k.transpose(0, 1, 3, 2)) / np.sqrt(hd)
    p = np.exp(s - s.max(-1, keepdims=True))
    return np.matmul(p / p.sum(-1, keepdims=True), v).reshape(B, Hq, hd)


@pytest.mark.parametrize("B,Hq,Hkv,n,hd", [
    (B, Hq, Hkv, n, hd)
    for B, Hq, Hkv in ((2, 5, 1), (20, 16, 8), (70, 16, 8), (34, 16, 4), (131, 16, 4), (33, 24, 8))
    for n in (1, 127, 129, 384, 385, 1021) for hd in (64, 128)
    if B * Hkv * n * hd <= 1 << 25          # beyond, the float64 reference takes seconds
])
def test_decode_attention_heads_and_waves(B, Hq, Hkv, n, hd):
    """One, two and four query heads per work-group (groups of five, two, four, three) with two, four and eight
    waves, around the context lengths where their number changes."""
    rng = np.random.default_rng(B + n + hd)
    max_len = (n + 7) // 8 * 8
    qb, q = rand_bf16(rng, (B, (Hq + 2 * Hkv), hd))
    kb, k = rand_bf16(rng, (B, Hkv, n, hd))
    vb, v = rand_bf16(rng, (B, Hkv, n, hd))
    kc, vc = np.full((B, Hkv, hd, max_len), 0x7FC1, np.uint16), np.full((B, Hkv, max_len, hd), 0x7FC1, np.uint16)
    kc[..., :n], vc[:, :, :n] = kb.transpose(0, 1, 3, 2), vb
    qd, kd, vd = dev_u16(qb.reshape(-1)), dev_u16(kc.reshape(-1)), dev_u16(vc.reshape(-1))
    o = torch.full(((B + 1) * Hq * hd,), 7, dtype=torch.int16, device=DEV)
    assert sp.spk_decode_attention(stream_ptr(), ptr(qd), ptr(kd), ptr(vd), ptr(o), B, n, max_len, Hq, Hkv, hd) == sp.SP_OK
    torch.cuda.synchronize()
    out = host_u16(o).reshape(B + 1, Hq, hd)
    assert np.all(out[B] == 7)                                      # the row behind o
    assert max_rel(bf16_vals(out[:B]), single_query_ref(q[:, :Hq], k, v)) <= 8e-3      # one bf16 rounding of the output


@pytest.mark.parametrize("shift", [1, 4])
def test_decode_attention_takes_queries_at_any_element(shift):
    """The fused activation may start at any bf16 element: only the cache is read by 16 bytes."""
    rng = np.random.default_rng(shift)
    B, Hq, Hkv, n, hd = 2, 4, 2, 96, 64
    qb, q = rand_bf16(rng, (B, Hq + 2 * Hkv, hd))
    kb, k = rand_bf16(rng, (B, Hkv, n, hd))
    vb, v = rand_bf16(rng, (B, Hkv, n, hd))
    qd = dev_u16(np.concatenate([np.zeros(shift, np.uint16), qb.reshape(-1)]))[shift:]
    assert qd.data_ptr() % 16
    kd, vd = dev_u16(kb.transpose(0, 1, 3, 2)), dev_u16(vb)
    o = torch.zeros(B * Hq * hd, dtype=torch.int16, device=DEV)
    assert sp.spk_decode_attention(stream_ptr(), ptr(qd), ptr(kd), ptr(vd), ptr(o), B, n, n, Hq, Hkv, hd) == sp.SP_OK
    torch.cuda.synchronize()
    got = bf16_vals(host_u16(o)).reshape(B, Hq, hd)
    assert max_rel(got, single_query_ref(q[:, :Hq], k, v)) <= 8e-3      # one bf16 rounding of the output


def attention_only_layer(Hq, Hkv, hd, B):
    """A decoder layer whose q, k and v are the leading elements of the normed input, whose output projection is the
    identity and whose MLP is zero: y - x is the attention output itself."""
    w = synth.Workload("attn_only", "decoder", 1, Hq * hd, Hq, Hkv, hd, 128, True, B, 1)
    desc = sp.make_desc(w)
    blob = torch.zeros(sp.sp_layer_blob_bytes(C.byref(desc)), dtype=torch.uint8, pin_memory=True)
    v = sp.blob_views(desc, blob.numpy())
    d, one = Hq * hd, synth.f32_to_bf16_bits(np.ones(1, np.float32))[0]
    v["g1"][:] = one
    v["g2"][:] = one
    wqkv = v["wqkv"].reshape(-1, d)
    for r0, n in ((0, d), (d, Hkv * hd), (d + Hkv * hd, Hkv * hd)):
        wqkv[np.arange(r0, r0 + n), np.arange(n)] = one
    v["wo"].reshape(d, d)[np.arange(d), np.arange(d)] = one
    return w, desc, blob


@pytest.mark.parametrize("B,Hq,Hkv,hd,pos,max_len", [
    (1, 1, 1, 64, 4608, 4616),       # fifteen splits: two batches of rows in the combination
    (1, 4, 1, 128, 8191, 8192),      # sixteen, one group of four
    (1, 2, 1, 64, 32767, 32768),     # sixty-four, the longest cache
    (16, 16, 8, 64, 4100, 4104),     # four: the number of work-groups sets the limit
    (2, 64, 8, 64, 8300, 8304),      # groups of eight as two blocks of four, four waves
    (8, 64, 8, 64, 4100, 4104),      # the same, two waves
    (1, 32, 32, 64, 8300, 8304),     # one head per work-group, four waves
    (2, 32, 16, 64, 8300, 8304),     # two heads, four waves
    (3, 6, 2, 128, 1024, 1032),      # four splits, groups of three
    (2, 8, 8, 64, 1023, 1024),       # one split
])
def test_decode_step_over_a_long_cache(B, Hq, Hkv, hd, pos, max_len):
    """The attention of a decode step against float64, over a cache of random keys and values, and the cache
    afterwards: position pos holds the new key and value, every other bit is what it was."""
    rng = np.random.default_rng(pos + Hq)
    w, desc, blob = attention_only_layer(Hq, Hkv, hd, B)
    d = w.d_model
    x = (rng.standard_normal((B, d)) * 0.7).astype(np.float32)
    a = bf16_vals(synth.f32_to_bf16_bits((x / np.sqrt(np.mean(x.astype(np.float64) ** 2, -1, keepdims=True) + w.norm_eps)).astype(np.float32)))
    kb, k = rand_bf16(rng, (B, Hkv, max_len, hd))
    vb, v = rand_bf16(rng, (B, Hkv, max_len, hd))
    cache_bits = np.concatenate([np.ascontiguousarray(kb.transpose(0, 1, 3, 2)).reshape(-1), vb.reshape(-1)])
    assert cache_bits.size * 2 == sp.sp_kv_cache_bytes(C.byref(desc), B, max_len)
    xd = dev_f32(x)
    out = []
    slot = (blob.numel() + 4095) // 4096 * 4096
    for budget in (None, sp.sp_workspace_bytes(C.byref(desc), 0) + slot):
        cache = dev_u16(cache_bits)
        eng = sp.Engine(desc, [blob], 1, 1, budget_bytes=budget)
        yd = torch.empty_like(xd)
        eng.decode(xd, yd, cache, B, pos, max_len)
        eng.sync()
        out.append((yd.cpu().numpy(), host_u16(cache), eng.stats().plan.arena_bytes_used))
        eng.destroy()
    # a budget without room for the splits' partial results: the same bits
    assert out[0][2] - out[1][2] == sp.sp_decode_scratch_bytes(C.byref(desc)) > 0
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    got = out[0][0].astype(np.float64) - x
    k[:, :, pos], v[:, :, pos] = a[:, :Hkv * hd].reshape(B, Hkv, hd), a[:, :Hkv * hd].reshape(B, Hkv, hd)
    ref = single_query_ref(a.reshape(B, Hq, hd), k[:, :, :pos + 1], v[:, :, :pos + 1]).reshape(B, d)
    assert max_rel(got, ref) <= 8e-3          # one bf16 rounding of the output
    after = out[0][1]
    kc, vc = after[:after.size // 2].reshape(B, Hkv, hd, max_len), after[after.size // 2:].reshape(B, Hkv, max_len, hd)
    assert np.array_equal(bf16_vals(kc[..., pos]), k[:, :, pos]) and np.array_equal(bf16_vals(vc[:, :, pos]), v[:, :, pos])
    kc[..., pos], vc[:, :, pos] = kb[:, :, pos], vb[:, :, pos]
    assert np.array_equal(after, cache_bits)


@pytest.mark.parametrize("B,Hq,Hkv,hd,pos,max_len", [
    (1, 4, 1, 64, 4096, 4104),       # sixteen splits of 256 positions, two waves
    (1, 4, 1, 128, 4097, 4104),      # the first that take four waves, the last split short
    (1, 2, 1, 64, 8193, 8200),       # seventeen: the seventeenth row of partial results is a batch of its own
    (2, 32, 8, 64, 8300, 8304),      # groups of four in one block, eight waves
    (6, 12, 6, 128, 1100, 1104),     # the fewest work-groups but 121 that keep eight waves, one head each
    (3, 8, 2, 128, 1281, 1288),      # six splits, the last of one position
    (11, 12, 3, 128, 1024, 1032),    # two heads, eight waves
    (11, 24, 3, 64, 1024, 1032),     # four heads, eight waves
    (2, 32, 8, 64, 8191, 8192),      # two heads of four, four waves: sixteen splits, a cache's readers on one XCD
    (2, 56, 7, 64, 1918, 1920),      # two heads of eight, two waves
    (13, 40, 10, 64, 1024, 1032),    # four heads, four waves
    (12, 24, 3, 64, 5058, 5064),     # four heads, more than two rounds
    (2, 44, 44, 64, 1574, 1576),     # no fifth split of four waves
])
def test_decode_step_edges_of_the_splits(B, Hq, Hkv, hd, pos, max_len):
    test_decode_step_over_a_long_cache(B, Hq, Hkv, hd, pos, max_len)


def test_decode_kernel_argument_errors():
    t = torch.zeros(1 << 16, dtype=torch.int16, device=DEV)
    s = stream_ptr()
    assert sp.spk_decode_attention(s, ptr(t), ptr(t), ptr(t), ptr(t), 1, 4, 8, 4, 4, 80) == sp.SP_ERR_INVALID_ARG
    assert sp.spk_decode_attention(s, ptr(t), ptr(t), ptr(t), ptr(t), 1, 9, 8, 4, 4, 64) == sp.SP_ERR_INVALID_ARG
    assert sp.spk_decode_attention(s, ptr(t), ptr(t), ptr(t), ptr(t), 1, 4, 7, 4, 4, 64) == sp.SP_ERR_INVALID_ARG
    assert sp.spk_decode_attention(s, ptr(t), ptr(t), ptr(t), ptr(t), 1, 4, 8, 4, 3, 64) == sp.SP_ERR_INVALID_ARG
    assert sp.spk_kv_append(s, ptr(t), ptr(t), ptr(t), 1, 4, 6, 4, 4, 64, 8) == sp.SP_ERR_INVALID_ARG
    assert sp.spk_kv_append(s, None, ptr(t), ptr(t), 1, 4, 0, 4, 4, 64, 8) == sp.SP_ERR_INVALID_ARG
    torch.cuda.synchronize()


class Gen:
    """A small causal decoder stack, its oracle output over S positions, and a runner that
    prefills S0 positions and decodes the rest one by one."""

    def __init__(self, w):
        self.w = w
        self.desc = sp.make_desc(w)
        self.blobs, self.views = sp.pinned_blobs(w, self.desc)
        self.x = synth.make_input(w)                                   # [B, S, d]
        sh = O.StackShape(w.arch, w.n_layers, w.d_model, w.n_q_heads, w.n_kv_heads, w.head_dim, w.d_ffn,
                          w.causal, w.norm_eps)
        self.ref = O.stack_forward(self.x, self.views, w.batch, w.seq, sh, dtype=np.float64).reshape(
            w.batch, w.seq, w.d_model)

    def run(self, k, p, s0, max_len, flags=0, pinned=0, budget_layers=None):
        w = self.w
        B, S, d = w.batch, w.seq, w.d_model
        eng = sp.Engine(self.desc, self.blobs, k, p, flags=flags, pinned=pinned, budget_layers=budget_layers)
        cache = torch.empty(sp.sp_kv_cache_bytes(C.byref(self.desc), B, max_len), dtype=torch.uint8, device=DEV)
        cache.fill_(0xFF)                                              # NaN patterns: stale reads would show
        out = np.full((B, S, d), np.nan, dtype=np.float32)
        if s0:
            xd = dev_f32(np.ascontiguousarray(self.x[:, :s0]))
            yd = torch.empty_like(xd)
            eng.prefill(xd, yd, cache, B, s0, max_len)
            eng.sync()
            out[:, :s0] = yd.cpu().numpy()
        for t in range(s0, S):
            xd = dev_f32(np.ascontiguousarray(self.x[:, t]))
            yd = torch.empty_like(xd)
            eng.decode(xd, yd, cache, B, t, max_len)
            eng.sync()
            out[:, t] = yd.cpu().numpy()
        st = eng.stats()
        assert eng.destroy() == sp.SP_OK
        return out, st


@pytest.fixture(scope="module")
def gen():
    # grouped-query heads, 5 layers, 2 sequences of 40 positions
    return Gen(synth.Workload("gen_small", "decoder", 5, 256, 4, 2, 64, 512, True, 2, 40))


def test_decode_matches_the_causal_forward_of_the_oracle(gen):
    out, st = gen.run(1, 1, s0=24, max_len=48)
    assert np.all(np.isfinite(out))
    err_prefill = both(out[:, :24], gen.ref[:, :24], gen.x[:, :24])
    err_decode = both(out[:, 24:], gen.ref[:, 24:], gen.x[:, 24:])
    print(f"gen_small: prefill 24 positions max rel err {err_prefill:.3e}; 16 decode steps {err_decode:.3e}")
    assert err_prefill <= TOL and err_decode <= TOL
    # every decode step streams the whole stack once: 5 copies per call with 2 slots
    assert st.calls == 1 + 16 and st.last_h2d_copies == 5


def test_decode_from_an_empty_cache_and_bits_across_windows(gen):
    base, _ = gen.run(8, 8, s0=0, max_len=40)                          # resident, no prefill
    assert both(base, gen.ref, gen.x) <= TOL
    for k, p, pinned, flags in [(1, 1, 0, 0), (2, 1, 0, sp.SP_FLAG_WRAP_PREFETCH), (1, 1, 2, sp.SP_FLAG_POISON),
                                (1, 2, 0, sp.SP_FLAG_NO_OVERLAP)]:
        out, st = gen.run(k, p, s0=0, max_len=40, flags=flags, pinned=pinned)
        assert np.array_equal(out.view(np.uint32), base.view(np.uint32)), (k, p, pinned, flags)
        assert not st.plan.fully_resident


def test_decode_head_dim_128_and_prefill_equals_forward():
    w = synth.Workload("gen_hd128", "decoder", 2, 512, 4, 4, 128, 1024, True, 3, 21)
    g = Gen(w)
    out, _ = g.run(1, 1, s0=20, max_len=24)
    assert both(out, g.ref, g.x) <= TOL
    # prefill runs the same kernels as sp_forward: same bits
    eng = sp.Engine(g.desc, g.blobs, 1, 1)
    xd = dev_f32(g.x)
    yd = torch.empty_like(xd)
    eng.forward(xd, yd, w.batch, w.seq)
    eng.sync()
    cache = torch.empty(sp.sp_kv_cache_bytes(C.byref(g.desc), w.batch, 24), dtype=torch.uint8, device=DEV)
    y2 = torch.empty_like(xd)
    eng.prefill(xd, y2, cache, w.batch, w.seq, 24)
    eng.sync()
    assert torch.equal(yd, y2)
    eng.destroy()


def test_decode_argument_errors(gen):
    w = gen.w
    eng = sp.Engine(gen.desc, gen.blobs, 1, 1)
    x = torch.zeros(w.batch, w.d_model, device=DEV)
    cache = torch.zeros(sp.sp_kv_cache_bytes(C.byref(gen.desc), w.batch, 16), dtype=torch.uint8, device=DEV)
    for pos, max_len in [(16, 16), (-1, 16), (0, 12), (0, 1 << 20)]:
        with pytest.raises(sp.SuperpipeError) as ex:
            eng.decode(x, x, cache, w.batch, pos, max_len)
        assert ex.value.code == sp.SP_ERR_SHAPE
    with pytest.raises(sp.SuperpipeError):
        eng.prefill(torch.zeros(w.batch, 17, w.d_model, device=DEV), torch.zeros(w.batch, 17, w.d_model, device=DEV),
                    cache, w.batch, 17, 16)
    eng.destroy()
    assert sp.sp_kv_cache_bytes(C.byref(gen.desc), w.batch, 12) == 0
    assert sp.sp_kv_cache_bytes(C.byref(gen.desc), w.batch, 16) == 5 * 2 * w.batch * 2 * 64 * 16 * 2
    # encoder stacks have no causal mask: no cache
    we = synth.WORKLOADS["vith"].with_(n_layers=1, batch=1)
    de = sp.make_desc(we)
    be, _ = sp.pinned_blobs(we, de)
    ee = sp.Engine(de, be, 1, 1)
    xe = torch.zeros(1, we.d_model, device=DEV)
    with pytest.raises(sp.SuperpipeError) as ex:
        ee.decode(xe, xe, cache, 1, 0, 16)
    assert ex.value.code == sp.SP_ERR_STATE
    ee.destroy()


@pytest.mark.parametrize("B,S,s0,Hq,Hkv,hd", [
    (1, 1030, 1021, 4, 1, 128),     # one split, four at 1024 cached positions, five from 1025 on; one group of four
    (2, 1540, 1534, 6, 2, 64),      # six splits, seven from 1537 cached positions on; a group of three
    (1, 1090, 1087, 16, 1, 64),     # a group of sixteen: two head blocks read the cache, one stores
    (1, 515, 509, 8, 1, 128),       # one split, a group of eight
    (2, 10, 0, 2, 2, 128),          # the first positions: waves without any
])
def test_decode_splits_and_groups(B, S, s0, Hq, Hkv, hd):
    """Decode attention around the sizes where the positions are split, for every number of query heads
    per work-group, against the oracle's causal forward."""
    g = Gen(synth.Workload("gen_split", "decoder", 1, Hq * hd, Hq, Hkv, hd, 128, True, B, S))
    out, _ = g.run(1, 1, s0=s0, max_len=(S + 7) // 8 * 8)
    assert both(out[:, s0:], g.ref[:, s0:], g.x[:, s0:]) <= TOL
