"""GPU: row blocks on the block kernels at the row counts and widths where their launches change."""
import ctypes as C

import numpy as np
import pytest

import paper_2407_19947_amd as pkg
import synth_inputs as si

pytestmark = pytest.mark.gpu


# widths with a ragged last k chunk (1280, 2816), features that end inside a 256- and a 128-feature work-group
@pytest.mark.parametrize("d,heads,f", [(256, 2, 256), (1280, 10, 2816), (2048, 32, 1024)])
@pytest.mark.parametrize("rows", [17, 33, 64, 65, 127, 129, 256, 1024, 1025, 2048, 2049])
def test_block_rows_against_decode_kernels(d, heads, f, rows, monkeypatch):
    """A prompt of one forward and the smallest block (33 rows), edges of the 64- and 128-row tiles, the largest block whose k range is summed in pieces and
    the smallest that is not, a full block and one row more: the stair logits behind a prompt ingested in blocks against
    those behind the same prompt ingested by the decode kernels (same inputs, another order of additions: 1e-5 of the
    logits' size measured; keys and values are rounded to half in both, so single roundings can fall differently)."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=2, d_model=d, n_heads=heads, d_ffn=f, vocab=528),
                           draft=dict(kind="prefix", n_layers=1), P=rows + 1, G=1)
    target, draft = si.make_pair(w)
    prompt = si.make_prompt(w)
    got = {}
    for mode in ("block", "rows"):
        if mode == "rows":
            monkeypatch.setenv("STAIRS_NO_BLOCK_PREFILL", "1")
        with pkg.Stairs(target, None, k_max=0, max_seq=rows + 16) as s:
            s.prefill(prompt)
            got[mode] = s.verify(0, logits=True)[2].astype(np.float64)
    rms = np.sqrt(np.mean(got["rows"] ** 2))
    assert np.max(np.abs(got["block"] - got["rows"])) < 2e-3 * rms


@pytest.mark.parametrize("lens", [[18, 33, 34, 49, 300, 18], [17, 200, 5, 1025, 1026, 65, 1300], [700, 700, 700, 129]])
def test_prompts_of_a_batch_share_blocks(lens):
    """Prompts that share a block (17 .. 1024 rows: the smallest, ends on and beside multiples of 16 rows, more than one block's
    worth), too short, and too long to share one: every sequence's tokens are those of the sequence generated alone, before the
    reservation (there prompts of up to 32 rows take the decode kernels)."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=2, d_model=512, n_heads=4, d_ffn=768, vocab=1040),
                           draft=dict(kind="prefix", n_layers=1), P=2, G=1)
    target, draft = si.make_pair(w)
    rng = np.random.default_rng(len(lens))
    prompts = [rng.integers(0, 1040, P).astype(np.int32) for P in lens]
    with pkg.Stairs(target, draft, k_max=2, max_seq=max(lens) + 32) as s:
        alone = [s.generate(p, 12, 2)[0].copy() for p in prompts]
        s.reserve_batch(len(lens))
        toks, _ = s.generate_batch(prompts, 12, 2)
    for b, want in enumerate(alone):
        assert np.array_equal(toks[b], want), lens[b]


@pytest.mark.parametrize("f", [8192, 11008])
def test_more_than_four_pieces(f):
    """k = 8192 is summed in 8 pieces, 11008 in 10 of unequal length: prompts whose down projection spreads them over
    work-groups alone (40 rows) and keeps them in registers in the block they share (1900 rows) give the same tokens."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=2, d_model=512, n_heads=4, d_ffn=f, vocab=1040),
                           draft=dict(kind="prefix", n_layers=1), P=2, G=1)
    target, draft = si.make_pair(w)
    rng = np.random.default_rng(f)
    prompts = [rng.integers(0, 1040, P).astype(np.int32) for P in (41, 1000, 18, 500, 35, 300)]
    with pkg.Stairs(target, draft, k_max=2, max_seq=1040) as s:
        s.reserve_batch(len(prompts))
        alone = np.stack([s.generate(p, 12, 2)[0].copy() for p in prompts])
        toks, _ = s.generate_batch(prompts, 12, 2)
    assert np.array_equal(toks, alone)


@pytest.mark.parametrize("rows", [16, 17, 24, 31, 32])
def test_prompts_of_one_forward_take_the_decode_kernels(rows, monkeypatch):
    """A prompt that one forward of the decode kernels holds goes through those (they are faster there): the stair logits
    behind it are the bits of the context that has no block kernels for prompts."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=2, d_model=512, n_heads=4, d_ffn=768, vocab=1040),
                           draft=dict(kind="prefix", n_layers=1), P=rows + 1, G=1)
    target, _ = si.make_pair(w)
    prompt = si.make_prompt(w)
    got = []
    for off in (None, "1"):
        if off:
            monkeypatch.setenv("STAIRS_NO_BLOCK_PREFILL", off)
        with pkg.Stairs(target, None, k_max=0, max_seq=rows + 16) as s:
            s.prefill(prompt)
            got.append(s.verify(0, logits=True)[2].copy())
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("B,k", [(8, 2), (22, 2)])
def test_short_prompts_of_a_batch(B, k):
    """Prompts of 17 rows and more share blocks, in forwards of 24 rows (decode kernels) and of 66 (block kernels).  A
    sequence's tokens depend neither on its neighbours nor on their order; they are those of the sequence alone on the
    reserved context, where it takes the same kernels."""
    w = si.scaled_workload("cfg2_125m", target=dict(n_layers=2, d_model=512, n_heads=4, d_ffn=768, vocab=1040),
                           draft=dict(kind="prefix", n_layers=1), P=2, G=1)
    target, draft = si.make_pair(w)
    rng = np.random.default_rng(22)
    prompts = [rng.integers(0, 1040, P).astype(np.int32) for P in ([17, 18, 19, 25, 32, 33, 34, 60] * 3)[:B]]
    with pkg.Stairs(target, draft, k_max=k, max_seq=96) as s:
        s.reserve_batch(B)
        alone = np.stack([s.generate(p, 12, k)[0].copy() for p in prompts])
        first, _ = s.generate_batch(prompts, 12, k)
        turned, _ = s.generate_batch(prompts[::-1], 12, k)
    assert np.array_equal(first, turned[::-1])
    assert np.array_equal(first, alone)


class _BlkGemm(C.Structure):
    """struct BlkGemm of csrc/stairs_kernels.h"""
    _fields_ = [("W", C.c_void_p), ("NTILES", C.c_int), ("tile_first", C.c_int), ("K", C.c_int), ("XF", C.c_void_p),
                ("RT", C.c_int), ("R", C.c_int), ("kind", C.c_int), ("out", C.c_void_p), ("ldo", C.c_int),
                ("ssq", C.c_void_p), ("ssq_n", C.c_int), ("eps", C.c_float), ("frag_out", C.c_void_p), ("gain", C.c_void_p),
                ("ssq_out", C.c_void_p), ("rows", C.c_void_p), ("cs", C.c_void_p), ("Kc", C.c_void_p), ("Vc", C.c_void_p),
                ("slot_stride", C.c_size_t), ("cap", C.c_int), ("hd", C.c_int), ("da", C.c_int), ("pieces", C.c_int)]


def _cxx(name, restype, *argtypes):
    """a host function of the library's C++ side, by its mangled name"""
    f = getattr(pkg.lib(), name)
    f.restype, f.argtypes = restype, argtypes
    return f


@pytest.mark.parametrize("R", [1, 63, 64, 65, 200, 1025])
@pytest.mark.parametrize("K,pieces", [(256, 1), (768, 3), (1280, 4), (2048, 4), (11008, 10)])
def test_small_block_gemm_shape_has_the_bits_of_the_large_one(K, pieces, R):
    """The 128 x 64 shape, whose ring holds four k-steps, against 256 x 64: pieces of 8 k-steps, the shortest there are (256, 768,
    2048 in 8), of 10 (1280) and of unequal length (11008), one piece beyond 1024 rows, rows around its tile."""
    import torch
    assert _cxx("_ZN6stairs17configure_kernelsEv", C.c_int)() == 0
    launch = _cxx("_ZN6stairs18launch_blk_gemm_asEibRKNS_7BlkGemmEP12ihipStream_tPfm", C.c_int, C.c_int, C.c_bool,
                  C.POINTER(_BlkGemm), C.c_void_p, C.c_void_p, C.c_size_t)
    NT, RT = 19, (R + 127) // 128 * 8
    g = torch.Generator().manual_seed(K + R)
    W = (torch.randn(NT * 16 * K, generator=g) * 0.1).to(torch.bfloat16).cuda()
    X = torch.randn(K // 32 * RT * 1024, generator=g).to(torch.bfloat16).cuda()
    for P in ((1,) if R > 1024 else {pieces, min(8, K // 256)}):
        part = torch.empty(P * ((R + 15) // 16 * 16) * NT * 16, device="cuda")
        outs = []
        for shape, split in ((1, False), (3, False), (3, True)):
            if split and P == 1:
                continue
            y = torch.full((R, NT * 16), float("nan"), device="cuda")
            p = _BlkGemm(W=W.data_ptr(), NTILES=NT, K=K, XF=X.data_ptr(), RT=RT, R=R, out=y.data_ptr(), ldo=NT * 16, pieces=P)
            torch.cuda.synchronize()
            assert launch(shape, split, C.byref(p), None, part.data_ptr(), part.numel()) == 0
            torch.cuda.synchronize()
            outs.append(y)
        assert torch.isfinite(outs[0]).all()
        for y in outs[1:]:
            assert torch.equal(y, outs[0]), P


@pytest.mark.parametrize("R", [17, 65, 129, 256])
@pytest.mark.parametrize("K,pieces", [(768, 3), (2048, 4), (8192, 8), (11008, 10)])
def test_block_gemm_forms_have_the_same_bits(K, pieces, R):
    """One product by both tile shapes, its k pieces added up in registers and through memory: the same bits, and those of
    a 64-bit product but for the roundings of K single-precision additions (operands carry bf16 high + low parts).  Widths:
    pieces of unequal length (11008), a last k chunk of half the length (768, 11008), an odd number of weight tiles, rows
    on both sides of the 64- and 128-row tiles."""
    import torch
    assert _cxx("_ZN6stairs17configure_kernelsEv", C.c_int)() == 0
    assert _cxx("_ZN6stairs10blk_piecesEi", C.c_int, C.c_int)(K) == pieces
    launch = _cxx("_ZN6stairs18launch_blk_gemm_asEibRKNS_7BlkGemmEP12ihipStream_tPfm", C.c_int, C.c_int, C.c_bool,
                  C.POINTER(_BlkGemm), C.c_void_p, C.c_void_p, C.c_size_t)
    NT, RT, ks = 33, (R + 127) // 128 * 8, K // 32
    g = torch.Generator().manual_seed(K + R)
    w = torch.randn(NT * 16, K, generator=g).to(torch.bfloat16)
    x = torch.randn(RT * 16, K, generator=g)
    hi = x.to(torch.bfloat16)
    lo = (x - hi.float()).to(torch.bfloat16)
    # operand tiles [chunk of 16 k-steps][tile][k-step][lane r + 16 g][8], the last chunk as long as is left
    t = w.view(NT, 16, ks, 4, 8).permute(0, 2, 3, 1, 4)                      # [tile][k-step][g][r][8]
    W = torch.cat([t[:, c:c + 16].reshape(-1) for c in range(0, ks, 16)]).cuda()
    # fragments [k-step][column tile][high, low][lane][8]
    X = torch.stack([v.view(RT, 16, ks, 4, 8).permute(2, 0, 3, 1, 4) for v in (hi, lo)], 2).reshape(-1).cuda()
    part = torch.empty(pieces * ((R + 15) // 16 * 16) * NT * 16, device="cuda")
    outs = []
    for shape in (0, 1):
        for split in (False, True):
            y = torch.full((R, NT * 16), float("nan"), device="cuda")
            p = _BlkGemm(W=W.data_ptr(), NTILES=NT, K=K, XF=X.data_ptr(), RT=RT, R=R, out=y.data_ptr(), ldo=NT * 16, pieces=pieces)
            torch.cuda.synchronize()
            assert launch(shape, split, C.byref(p), None, part.data_ptr(), part.numel()) == 0
            torch.cuda.synchronize()
            outs.append(y.cpu())
    for y in outs[1:]:
        assert torch.equal(y, outs[0])
    xs = hi.double()[:R] + lo.double()[:R]
    want, size = xs @ w.double().t(), xs.abs() @ w.double().abs().t()
    assert ((outs[0].double() - want).abs() <= 2 * K * 2.0 ** -24 * size).all()


PLAIN, RESID, SWIGLU, QKV, RELU = range(5)             # kinds of a block projection


@pytest.mark.parametrize("R", [23, 40, 240, 250])
@pytest.mark.parametrize("kind", [PLAIN, RESID, SWIGLU, QKV, RELU])
def test_every_result_of_a_block_gemm_has_the_same_bits_in_every_form(kind, R):
    """What each kind leaves (values, fragments, sums of squares, caches), with the rows normalised where a kind is ever used
    so: by the three tile shapes, the pieces added up in registers and by the second kernel.  264 tiles: the second kernel takes
    two by two tiles from 250 rows on (16 column tiles) and one by two or two by one below (15 and fewer, odd numbers too); rows
    that end inside a column tile."""
    import torch
    assert _cxx("_ZN6stairs17configure_kernelsEv", C.c_int)() == 0
    launch = _cxx("_ZN6stairs18launch_blk_gemm_asEibRKNS_7BlkGemmEP12ihipStream_tPfm", C.c_int, C.c_int, C.c_bool,
                  C.POINTER(_BlkGemm), C.c_void_p, C.c_void_p, C.c_size_t)
    NT, K, pieces, hd, slots, cap = 264, 768, 3, 128, 3, 256
    N, RT, da = NT * 16, (R + 127) // 128 * 8, NT * 16 // 3
    assert (NT * ((R + 15) // 16) >= 4096) == (R == 250)
    g = torch.Generator().manual_seed(100 * kind + R)
    rand = lambda *s: torch.randn(*s, generator=g)
    W = (rand(N * K) * 0.05).to(torch.bfloat16).cuda()
    X = rand(K // 32 * RT * 1024).to(torch.bfloat16).cuda()
    ssq = (rand(R, K // 32) ** 2 * 32).cuda() if kind != RESID else None
    x0, gain = rand(R, N).cuda(), (1 + 0.3 * rand(N)).cuda()
    cs = rand(R, 64, 2).cuda()
    # rows of three sequences and padding rows, which leave no keys and values
    slot = torch.arange(R) * slots // R
    pos = torch.arange(R) - (slot * R + slots - 1) // slots
    pos[5::9] = -1
    at = torch.stack([slot, pos], 1).int().contiguous().cuda()
    part = torch.empty(pieces * ((R + 15) // 16 * 16) * N, device="cuda")
    results = []
    for shape, split in ((1, False), (0, False), (3, False), (0, True), (1, True), (3, True)):
        out = x0.clone() if kind == RESID else torch.full((R, N), float("nan"), device="cuda")
        frag = torch.zeros(N // 32 * RT * 1024, dtype=torch.bfloat16, device="cuda")
        ss = torch.zeros(R, N // 32, device="cuda")
        Kc, Vc = (torch.zeros(slots * cap * da, dtype=torch.float16, device="cuda") for _ in range(2))
        p = _BlkGemm(W=W.data_ptr(), NTILES=NT, K=K, XF=X.data_ptr(), RT=RT, R=R, kind=kind, out=out.data_ptr(), ldo=N,
                     ssq=ssq.data_ptr() if ssq is not None else None, ssq_n=K // 32, eps=1e-5, frag_out=frag.data_ptr(), gain=gain.data_ptr(),
                     ssq_out=ss.data_ptr(), rows=at.data_ptr(), cs=cs.data_ptr(), Kc=Kc.data_ptr(), Vc=Vc.data_ptr(),
                     slot_stride=cap * da, cap=cap, hd=hd, da=da, pieces=pieces)
        torch.cuda.synchronize()
        assert launch(shape, split, C.byref(p), None, part.data_ptr(), part.numel()) == 0
        torch.cuda.synchronize()
        results.append([t.view(torch.int16) for t in (out, frag, ss, Kc, Vc)])
    for n, (name, first) in enumerate(zip(("out", "frag", "ssq", "K", "V"), results[0])):
        for r in results[1:]:
            assert torch.equal(r[n], first), name
    written = {PLAIN: (0,), RESID: (0, 1, 2), SWIGLU: (1,), QKV: (0, 3, 4), RELU: (1,)}[kind]
    for n in written:
        assert torch.count_nonzero(results[0][n]) > 0


class _PosRef(C.Structure):
    _fields_ = [("base", C.c_void_p), ("offset", C.c_int), ("rps", C.c_int)]


class _RowNorm(C.Structure):
    _fields_ = [("gain", C.c_void_p), ("ssq_part", C.c_void_p), ("ssq_n", C.c_int), ("eps", C.c_float)]


class _GemmEpi(C.Structure):
    """struct GemmEpi of csrc/stairs_kernels.h"""
    _fields_ = [("counters", C.c_void_p), ("out", C.c_void_p), ("ssq_out", C.c_void_p), ("rope_cs", C.c_void_p), ("pos", _PosRef),
                ("Kc", C.c_void_p), ("Vc", C.c_void_p), ("Kc32", C.c_void_p), ("Vc32", C.c_void_p), ("cap", C.c_int), ("H", C.c_int),
                ("hd", C.c_int), ("kv_slot_stride", C.c_size_t), ("frag_out", C.c_void_p), ("frag_gain", C.c_void_p), ("act", C.c_int),
                ("stream_weights", C.c_int)]


R_QKV, R_WO, R_GATEUP, R_DOWN, R_HEAD = range(5)       # roles of a decode projection


# tiles that end inside a work-group's eight; k of half a chunk, ends on half a chunk and on a whole one, odd and even numbers of
# chunks, more than 8 pairs; one launch (split False) and two.  None: the fragment-reading kernel, with one and with two tiles
# a wave
@pytest.mark.parametrize("role,tiles,K,hd,split", [
    (R_QKV, 48, 256, 64, False), (R_QKV, 264, 2304, 128, True), (R_QKV, 1872, 1536, 128, False), (R_QKV, 1872, 2304, 64, False),
    (R_GATEUP, 268, 768, 64, False), (R_GATEUP, 268, 2304, 64, True), (R_GATEUP, 1860, 1280, 64, False),
    (R_HEAD, 522, 1024, 64, False), (R_HEAD, 19, 8448, 64, True), (R_HEAD, 1860, 2304, 64, False),
    (R_WO, 522, 768, 64, False), (R_WO, 98, 4096, 64, True), (R_WO, 1860, 1280, 64, False),
    (R_DOWN, 20, 8448, 64, True), (R_DOWN, 20, 7936, 64, True), (R_DOWN, 1860, 2304, 64, False),
    (R_QKV, 240, 1280, 128, None), (R_GATEUP, 448, 1280, 64, None), (R_HEAD, 341, 1280, 64, None), (R_DOWN, 47, 2304, 64, None)])
def test_projections_of_17_to_64_rows_have_the_bits_of_one_row(role, tiles, K, hd, split):
    """The projections that go to the kernel that shares the fragments through LDS, and some at those row counts that do not: all
    they leave (values, sums of squares, the next projection's fragments, keys and values of several sequences, one of them not
    active) against the same projection of each row alone, which takes another kernel."""
    import torch
    assert _cxx("_ZN6stairs17configure_kernelsEv", C.c_int)() == 0
    takes = _cxx("_ZN6stairs12shared_takesEiiii", C.c_bool, *[C.c_int] * 4)
    splits = _cxx("_ZN6stairs13shared_splitsEiii", C.c_bool, *[C.c_int] * 3)
    gemm = _cxx("_ZN6stairs11launch_gemmEiiPKviiPKfiiNS_7RowNormEPfRKNS_7GemmEpiEP12ihipStream_tPK15HIP_vector_typeIjLj4EE", None,
                C.c_int, C.c_int, C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_int, C.c_int, _RowNorm, C.c_void_p,
                C.POINTER(_GemmEpi), C.c_void_p, C.c_void_p)
    to_frag = _cxx("_ZN6stairs17launch_split_fragEPKfiiiS1_P15HIP_vector_typeIjLj4EEP12ihipStream_t", None,
                   C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_void_p, C.c_void_p, C.c_void_p)
    frag_u4 = lambda k: (4 << 20) // 16 + (k + 31) // 32 * 256 + (k // 512 + 1) * 272         # frag_alloc_bytes
    N, cap = tiles * 16, 32
    resid = role in (R_WO, R_DOWN)
    d, width = N // 3, N // 2 if role == R_GATEUP else N // 3 if role == R_QKV else N
    g = torch.Generator().manual_seed(role + tiles + K)
    rand = lambda *s: torch.randn(*s, generator=g)
    W = (rand(N * K) * 0.05).to(torch.bfloat16).cuda()
    chunks = (K + 511) // 512
    partial = torch.empty((chunks + 1) * 32 * N, device="cuda")
    counters = torch.zeros(2048, dtype=torch.int32, device="cuda")
    for M, rps in ((33, 3), (47, 47), (48, 4), (64, 8)) + (((17, 17), (32, 2)) if resid and K > 15 * 512 else ()):
        if split is None and M == 64 and not resid:
            continue                                   # (shared there)
        assert takes(role, M, tiles, K) == (split is not None) and (split is None or splits(M, tiles, K) == split)
        X, gain, next_gain = rand(M, K).cuda(), (1 + 0.3 * rand(K)).cuda(), (1 + 0.3 * rand(N)).cuda()
        ssq, x0 = (rand(M, K // 16) ** 2 * 16).cuda(), rand(M, width).cuda()
        cs = rand(M, 64, 2).cuda()
        slots = M // rps
        state = torch.tensor([[int(torch.randint(0, max(1, cap - rps), (1,), generator=g)), 0, 0, int(s != 1)] for s in range(slots)],
                             dtype=torch.int32)
        cap_m = cap if rps <= cap else 64
        dstate = state.cuda()
        xf = torch.zeros(frag_u4(K) * 8, dtype=torch.bfloat16, device="cuda")
        to_frag(X.data_ptr(), K, M, K, None if resid else gain.data_ptr(), xf.data_ptr(), None)

        def fresh():
            out = x0.clone() if resid else torch.full((M, width), float("nan"), device="cuda")
            ss = torch.zeros(M, tiles, device="cuda")
            frag = torch.zeros(frag_u4(width) * 8, dtype=torch.bfloat16, device="cuda")
            Kc, Vc = (torch.zeros(slots * cap_m * d if role == R_QKV else 8, dtype=torch.float16, device="cuda") for _ in range(2))
            return out, ss, frag, Kc, Vc

        def launch(out, ss, frag, Kc, Vc, first, n):   # rows first .. first + n - 1: all of them or one
            one = n == 1
            s = first // rps if one else 0
            where = state[s].clone()
            where[0] += first % rps if one else 0
            base = where.cuda() if one else dstate
            e = _GemmEpi(counters=counters.data_ptr(), out=out.data_ptr() + first * width * 4, ssq_out=ss.data_ptr() + first * tiles * 4,
                         rope_cs=cs.data_ptr() + first * 512, pos=_PosRef(base.data_ptr(), 0, 1 if one else rps),
                         Kc=Kc.data_ptr() + (s * cap_m * d * 2 if role == R_QKV else 0), Vc=Vc.data_ptr() + (s * cap_m * d * 2 if role == R_QKV else 0),
                         cap=cap_m, H=d // hd, hd=hd, kv_slot_stride=cap_m * d, frag_out=None if one or role == R_QKV else frag.data_ptr(),
                         frag_gain=None if role == R_GATEUP else next_gain.data_ptr(), act=int(role == R_HEAD and M == 48),
                         stream_weights=int(M in (17, 33)))
            nrm = _RowNorm() if resid else _RowNorm(gain.data_ptr(), ssq.data_ptr() + first * (K // 16) * 4, K // 16, 1e-5)
            gemm(role, 1, W.data_ptr(), N, K, X.data_ptr() + first * K * 4, K, n, nrm, partial.data_ptr(), C.byref(e), None,
                 None if one else xf.data_ptr())
            torch.cuda.synchronize()

        got, want = fresh(), fresh()
        torch.cuda.synchronize()
        launch(*got, 0, M)
        for r in range(M):
            launch(*want, r, 1)
        if role != R_QKV:
            to_frag(want[0].data_ptr(), width, M, width, None if role == R_GATEUP else next_gain.data_ptr(), want[2].data_ptr(), None)
            torch.cuda.synchronize()
        for name, a, b in zip(("out", "ssq", "frag", "K", "V"), got, want):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16)), (name, M)
        inactive = slice(rps, 2 * rps) if role == R_QKV and slots > 1 else slice(0, 0)
        kept = torch.ones(M, dtype=torch.bool)
        kept[inactive] = False
        assert torch.isfinite(got[0][kept.cuda()]).all() and torch.isnan(got[0][~kept.cuda()]).all()


@pytest.mark.parametrize("M", [1, 4, 7])
def test_unembedding_writes_its_output_alone(M):
    """A caller's structure may name its caches for every role: an unembedding touches none of them."""
    import torch
    assert _cxx("_ZN6stairs17configure_kernelsEv", C.c_int)() == 0
    gemm = _cxx("_ZN6stairs11launch_gemmEiiPKviiPKfiiNS_7RowNormEPfRKNS_7GemmEpiEP12ihipStream_tPK15HIP_vector_typeIjLj4EE", None,
                C.c_int, C.c_int, C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_int, C.c_int, _RowNorm, C.c_void_p,
                C.POINTER(_GemmEpi), C.c_void_p, C.c_void_p)
    N, K = 4096, 512
    assert _cxx("_ZN6stairs13rows_path_ldsEiiii", C.c_size_t, *[C.c_int] * 4)(R_HEAD, M, N, K) > 0
    W, X = torch.ones(N * K, dtype=torch.bfloat16, device="cuda"), torch.ones(M, K, device="cuda")
    out, partial = torch.zeros(M, N, device="cuda"), torch.zeros(2 * M * N, device="cuda")
    counters = torch.zeros(4096, dtype=torch.int32, device="cuda")
    caches = [torch.full((M * N,), 7.0, device="cuda") for _ in range(4)]
    e = _GemmEpi(counters=counters.data_ptr(), out=out.data_ptr(), hd=64,
                 **{n: t.data_ptr() for n, t in zip(("Kc", "Vc", "Kc32", "Vc32"), caches)})
    torch.cuda.synchronize()
    gemm(R_HEAD, 1, W.data_ptr(), N, K, X.data_ptr(), K, M, _RowNorm(), partial.data_ptr(), C.byref(e), None, None)
    torch.cuda.synchronize()
    assert (out == K).all() and all((t == 7).all() for t in caches)
