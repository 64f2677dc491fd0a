"""The attention of a row block by itself against 64-bit arithmetic: segments of several sequences in one work-group, padding
rows, lengths around the 16-, 32- and 64-key steps, a cache that ends on half a step, the encoder's fixed key set and bias."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2407_19947_amd as pkg

pytestmark = pytest.mark.gpu

LAUNCH = "_ZN6stairs22launch_attention_flashEPKfPKvS3_iiimPK15HIP_vector_typeIiLj2EEiPS4_IjLj4EEP12ihipStream_tRKNS_8AttnModeE"


class AttnMode(C.Structure):
    _fields_ = [("scale", C.c_float), ("bias", C.c_void_p), ("bias_ld", C.c_int), ("bias_zero", C.c_int), ("kv_fixed", C.c_int),
                ("frag_out", C.c_void_p), ("frag_rt", C.c_int)]


def key_tiles(k):                                      # [slots, H, cap, hd] -> operand tiles
    s, h, cap, hd = k.shape
    return k.view(s, h, cap // 16, 16, hd // 32, 4, 8).permute(0, 1, 2, 4, 5, 3, 6).contiguous()


def value_tiles(v):
    s, h, cap, hd = v.shape
    return v.view(s, h, cap // 32, 2, 4, 4, hd // 16, 16).permute(0, 1, 2, 6, 4, 7, 3, 5).contiguous()


class Case:
    """segs: (slot, first position, rows) one after the other, each from a multiple of 16 rows on"""

    def __init__(self, H, hd, cap, slots, segs, kv_fixed=0, bias=False, seed=0, scale=1.0):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        self.H, self.hd, self.cap, self.slots, self.segs, self.kv_fixed, self.d = H, hd, cap, slots, segs, kv_fixed, H * hd
        rows = []
        for s, (slot, pos0, n) in enumerate(segs):
            rows += [(slot, pos0 + i) for i in range(n)]
            if s + 1 < len(segs):
                rows += [(slot, -1)] * (-n % 16)
        self.R = len(rows)
        self.rows = torch.tensor(rows, dtype=torch.int32, device="cuda")
        self.q = torch.randn(self.R, self.d, device="cuda", generator=g) * scale
        self.k = torch.randn(slots, H, cap, hd, device="cuda", generator=g).half()
        self.v = torch.randn(slots, H, cap, hd, device="cuda", generator=g).half()
        self.bias = torch.randn(H, 2 * cap - 1, device="cuda", generator=g) if bias else None
        self.mode = AttnMode(1.0 if bias else 0.0, self.bias.data_ptr() if bias else None, 2 * cap - 1, cap - 1, kv_fixed, None, 0)
        self.kt, self.vt = key_tiles(self.k), value_tiles(self.v)
        self.RT = (self.R + 127) // 128 * 8
        self.frag = torch.zeros(self.d // 32 * self.RT * 2 * 512, dtype=torch.bfloat16, device="cuda")

    def launch(self, library):
        fn = getattr(library, LAUNCH)
        fn.restype = None
        fn(C.c_void_p(self.q.data_ptr()), C.c_void_p(self.kt.data_ptr()), C.c_void_p(self.vt.data_ptr()), self.cap, self.d, self.H,
           C.c_size_t(self.H * self.cap * self.hd), C.c_void_p(self.rows.data_ptr()), self.R, C.c_void_p(self.frag.data_ptr()),
           C.c_void_p(torch.cuda.current_stream().cuda_stream), C.byref(self.mode))

    def result(self):
        f = self.frag.view(self.d // 32, self.RT, 2, 4, 16, 8).double().sum(2)
        return f.permute(1, 3, 0, 2, 4).reshape(self.RT * 16, self.d)[:self.R]

    def exact(self):
        out = torch.zeros(self.R, self.d, dtype=torch.float64, device="cuda")
        r0 = 0
        scale = 1.0 if self.bias is not None else self.hd ** -0.5
        for slot, pos0, n in self.segs:
            q = self.q[r0:r0 + n].double().view(n, self.H, self.hd)
            pos = torch.arange(pos0, pos0 + n, device="cuda")
            L = self.kv_fixed or pos0 + n
            keys = torch.arange(L, device="cuda")
            for h in range(self.H):
                s = q[:, h] @ self.k[slot, h, :L].double().t().contiguous() * scale
                if self.bias is not None:
                    s += self.bias[h].double()[keys[None, :] - pos[:, None] + self.cap - 1]
                if not self.kv_fixed:
                    s.masked_fill_(keys[None, :] > pos[:, None], -np.inf)
                out[r0:r0 + n, h * self.hd:(h + 1) * self.hd] = torch.softmax(s, -1) @ self.v[slot, h, :L].double()
            r0 += (n + 15) // 16 * 16
        return out


ODD = [(0, 0, 1), (1, 0, 15), (2, 0, 16), (3, 0, 17), (4, 0, 33), (5, 0, 63), (6, 0, 64), (7, 0, 65), (0, 40, 24)]


@pytest.mark.parametrize("H,hd,cap,slots,segs,kv_fixed,bias", [
    (4, 64, 96, 8, ODD, 0, False),                    # one tile a wave; 96: the last 64 keys are half past the cache
    (4, 128, 96, 8, ODD, 0, False),
    (4, 128, 352, 1, [(0, 0, 341)], 0, False),
    (4, 64, 4160, 2, [(1, 4000, 130)], 0, False),
    (64, 64, 96, 8, ODD * 4, 0, False),               # two tiles a wave (enough work-groups for two per CU)
    (64, 128, 96, 8, ODD * 4, 0, False),
    (64, 128, 1056, 1, [(0, 0, 1041)], 0, False),
    (4, 64, 224, 1, [(0, 0, 211)], 211, True),        # encoder: every row sees every key
    (64, 128, 1024, 1, [(0, 0, 1000)], 1000, True),
])
def test_against_64_bits(H, hd, cap, slots, segs, kv_fixed, bias):
    """Keys, values and probabilities as half high + low, 32-bit sums: about 1e-6 of the result's size, and the result's own
    split into bf16 high + low (2^-17 a value); 2e-5 in the 2-norm leaves a factor of four.  Padding rows are zeros."""
    c = Case(H, hd, cap, slots, segs, kv_fixed, bias, seed=H + hd, scale=0.3 if bias else 1.0)
    c.launch(pkg.lib())
    torch.cuda.synchronize()
    got, want = c.result(), c.exact()
    assert torch.isfinite(got).all()
    assert (got - want).norm() / want.norm() < 2e-5
    assert (got[c.rows[:, 1] < 0] == 0).all()


@pytest.mark.parametrize("hd", [64, 128])
def test_rows_do_not_depend_on_what_they_share_a_block_with(hd):
    """A sequence alone (one tile a wave) and among others (two tiles a wave): the same bits."""
    H, cap = 64, 160
    many = Case(H, hd, cap, 8, [(s, 0, 40 + 13 * s) for s in range(8)] * 2, seed=3)
    many.launch(pkg.lib())
    r0 = sum((40 + 13 * s + 15) // 16 * 16 for s in range(5))
    one = Case(H, hd, cap, 8, [(5, 0, 105)], seed=3)
    one.k, one.v, one.kt, one.vt = many.k, many.v, many.kt, many.vt
    one.q = many.q[r0:r0 + 105].contiguous()
    one.launch(pkg.lib())
    torch.cuda.synchronize()
    assert torch.equal(one.result(), many.result()[r0:r0 + 105])


@pytest.mark.parametrize("hd,scale", [(64, 1.0), (128, 1.0), (64, 0.0)])
def test_queries_up_to_the_largest_half(hd, scale):
    """A scaled query of 65000 is a half (the decode kernels' range, whatever the softmax's base).  One such dimension against keys
    of 1e-4 .. 2e-4 adds 8 .. 16 to a score; what its low part leaves out, 2^-22 of that, is within the tolerance above."""
    c = Case(4, hd, 160, 1, [(0, 0, 150)], seed=hd)
    c.mode.scale = scale
    head_scale = scale or hd ** -0.5
    big = torch.zeros(4, hd, dtype=torch.bool, device="cuda")
    big[:, 5] = True
    c.q[:, big.view(-1)] = c.q[:, big.view(-1)].sign() * (65000.0 / head_scale)
    c.q[:, ~big.view(-1)] *= hd ** -0.5 / head_scale
    c.k[..., 5] = c.k[..., 5].sign() * (1 + c.k[..., 5].abs().clamp(max=1)) * 2.0 ** -13
    c.kt = key_tiles(c.k)
    c.launch(pkg.lib())
    torch.cuda.synchronize()
    c.q = c.q * (head_scale / hd ** -0.5)              # (exact() scales by hd^-0.5)
    got, want = c.result(), c.exact()
    assert torch.isfinite(got).all()
    assert (got - want).norm() / want.norm() < 2e-5


@pytest.mark.parametrize("hd", [64, 128])
def test_biases_of_the_lowest_value(hd):
    """The lowest float as a bias hides a key from the rows that see another one; rows whose keys all have it see them equally."""
    cap, n = 224, 211
    c = Case(4, hd, cap, 1, [(0, 0, n)], n, True, seed=hd)
    c.q.zero_()
    c.bias.fill_(0)
    c.bias[0].fill_(torch.finfo(torch.float32).min)    # head 0: every key; the others: those behind the row
    c.bias[1:, cap:] = torch.finfo(torch.float32).min
    c.launch(pkg.lib())
    torch.cuda.synchronize()
    got, want = c.result(), c.exact()
    assert torch.isfinite(got).all()
    assert (got - want).norm() / want.norm() < 2e-5
