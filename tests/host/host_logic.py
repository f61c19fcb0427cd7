"""Checks of the library's host logic (launch limits, launch counts, memory held) on the HIP runtime of
fake_hip.cpp, which books allocations and launches and computes nothing.  Run by tests/test_host_logic.py
as a program of its own, one check per process:  host_logic.py <fake runtime> <library> <check>."""
import ctypes
import sys

VP, I64 = ctypes.c_void_p, ctypes.c_int64


class BgdParams(ctypes.Structure):
    _fields_ = [("steps", ctypes.c_int32), ("lr", ctypes.c_float), ("beta1", ctypes.c_float), ("beta2", ctypes.c_float),
                ("eps", ctypes.c_float), ("tok_chunk", I64), ("form", ctypes.c_int32), ("loss_clip", ctypes.c_float),
                ("batch", I64), ("resid_increment", ctypes.c_int32)]


class QParams(ctypes.Structure):
    _fields_ = [("bits", ctypes.c_int32), ("group", ctypes.c_int32), ("block", ctypes.c_int32), ("grid", ctypes.c_int32),
                ("damp", ctypes.c_float), ("sym", ctypes.c_int32)]


class LayerDesc(ctypes.Structure):
    _fields_ = [("m", I64), ("n", I64), ("T", I64), ("W0", VP), ("X", VP), ("Xhat", VP), ("s", VP), ("M", VP), ("P", VP),
                ("window_offset", ctypes.c_int32), ("window_total", ctypes.c_int32), ("q", QParams), ("bgd", BgdParams),
                ("s_groups", VP), ("n_groups", ctypes.c_int32)]


class LayerOut(ctypes.Structure):
    _fields_ = [("codes", VP), ("scales", VP), ("zeros", VP), ("W_hat", VP), ("H", VP), ("U", VP), ("dead", VP),
                ("loss_trace", VP), ("loss_final", ctypes.c_double), ("ms_total", ctypes.c_double)]


def buf(k):
    """A device address of the caller's; nothing reads it."""
    return VP((1 << 36) + (k << 34))


class Library:
    def __init__(self, fake, lib):
        self.fake = ctypes.CDLL(fake, mode=ctypes.RTLD_GLOBAL)  # first: the library's HIP calls bind to it
        for f in ("fake_held", "fake_peak", "fake_launches", "fake_bad_launches", "fake_copies", "fake_mallocs"):
            getattr(self.fake, f).restype = I64
        self.fake.fake_set_limit.argtypes = [I64]
        self.fake.fake_set_host_value.argtypes = [ctypes.c_double]
        self.c = ctypes.CDLL(lib)
        self.c.realq_last_error.restype = ctypes.c_char_p
        self.c.realq_last_error.argtypes = [VP]
        self.c.realq_ctx_destroy.argtypes = [VP]
        self.ctx = VP()
        assert self.c.realq_ctx_create(ctypes.byref(self.ctx), None) == 0

    def call(self, name, *args):
        """A call of the ABI on this context; ints go as int64, floats as float."""
        conv = {int: I64, float: ctypes.c_float}
        rc = getattr(self.c, name)(self.ctx, *[conv.get(type(a), lambda x: x)(a) for a in args])
        return rc, "" if rc == 0 else self.c.realq_last_error(self.ctx).decode()

    def ok(self, name, *args):
        rc, msg = self.call(name, *args)
        assert rc == 0, (name, rc, msg)
        assert self.fake.fake_bad_launches() == 0

    def state(self, m, n, T, s=buf(4), M=None, P=None, same=False, **params):
        b = BgdParams()
        self.c.realq_bgd_params_default(ctypes.byref(b))
        b.steps = 2
        for k, v in params.items():
            setattr(b, k, v)
        st = VP()
        self.ok("realq_bgd_state_create", ctypes.byref(st), buf(1), buf(2), buf(2) if same else buf(3), s, M, P, m, n, T,
                ctypes.byref(b))
        return st

    def layer(self, m, n, T, s=False, M=False, P=False, **params):
        """(code, message) of realq_quantize_layer."""
        d, o = LayerDesc(), LayerOut()
        self.c.realq_qparams_default(ctypes.byref(d.q))
        self.c.realq_bgd_params_default(ctypes.byref(d.bgd))
        for k, v in params.items():
            setattr(d.bgd, k, v)
        d.m, d.n, d.T = m, n, T
        d.W0, d.X, d.Xhat = buf(1).value, buf(2).value, buf(3).value
        d.s, d.M, d.P = (buf(4 + i).value if on else None for i, on in enumerate((s, M, P)))
        d.window_total = -(-n // 128) if P else 0
        o.codes = o.scales = o.zeros = o.W_hat = o.loss_trace = buf(7).value
        return self.call("realq_quantize_layer", ctypes.byref(d), ctypes.byref(o))

    def fresh(self):
        """A new context, the old one's memory given back."""
        self.c.realq_ctx_destroy(self.ctx)
        assert self.held() == 0
        assert self.c.realq_ctx_create(ctypes.byref(self.ctx), None) == 0

    def held(self):
        return self.fake.fake_held()

    def launches(self):
        return self.fake.fake_launches(b"") + self.fake.fake_copies()


def whole_lines(L):
    """Activations whose rows are whole 128-byte lines are read where they are: the state holds the
    arrays it needs and no copy of them."""
    for m, n, T in ((1024, 4096, 262144), (64, 1024, 65536), (512, 8192, 131072)):
        h0 = L.held()
        st = L.state(m, n, T, steps=1)
        Tp = T + 128
        arrays = m * Tp * 4 + 2 * m * n * 4 + 2 * m * n * 2 + n * Tp * 2 + m * 2 * Tp * 2
        workspaces = 2 * (256 << 20)  # the difference of the two inputs, a chunk at a time
        assert L.held() - h0 <= arrays + workspaces + (1 << 20), (m, n, T, L.held() - h0, arrays)
        L.c.realq_bgd_state_destroy(st)


def many_tokens(L):
    """Rows that need a padded copy, 2^24 of them: no launch past the grid limit."""
    T = 1 << 24
    for n in (133, 136):
        st = L.state(64, n, T)
        L.ok("realq_bgd_lock_block", st, 0, 128)
        L.ok("realq_bgd_loss", st, buf(5), buf(6))
        L.c.realq_bgd_state_destroy(st)
    L.ok("realq_handoff", buf(1), None, buf(2), T, 133, 64, buf(3))


def short_chunks(L):
    """Batches and token chunks that are not multiples of 8: the state's arrays grow by a sixteenth at most
    over the aligned case's, besides a copy of the inputs in the places' order, and its set-up and lock
    take as many launches as that case's, the two copies' and those of one more piece of the base (3)."""
    m, n, T = 1024, 4096, 262144
    for clip in (0.0, 0.95):
        for case in (dict(batch=9), dict(batch=100), dict(batch=1001), dict(batch=1), dict(tok_chunk=4),
                     dict(tok_chunk=1003), dict(batch=65535, tok_chunk=33)):
            got = []
            for params in ({k: (v + 7) // 8 * 8 for k, v in case.items()}, case):
                h0 = L.held()
                L.fake.fake_reset()
                st = L.state(m, n, T, loss_clip=clip, **params)
                made = L.launches()
                L.fake.fake_reset()
                L.ok("realq_bgd_lock_block", st, 0, 128)
                got.append((L.held() - h0, made, L.launches()))
                L.c.realq_bgd_state_destroy(st)
            (h_al, made_al, lock_al), (h, made, lock) = got
            assert h <= 1.07 * (h_al + 2 * T * n), (case, h, h_al)
            assert made <= made_al + 5 and lock == lock_al == 1, (case, got)


def slice_memory(L):
    """Products summed in float64 hold at most 3 GiB of slices whatever their size, give them back
    when other memory runs out, and take no new memory after a call with more tokens."""
    staging = 4 * (257 << 20)  # the four bf16 copies of a token chunk
    for n, T in ((4096, 131072), (14336, 65536), (28672, 32768)):
        h0 = L.held()
        L.ok("realq_hessian_accum", buf(1), buf(2), T, n, buf(3))
        assert L.held() - h0 <= staging + (3 << 30) + (1 << 26), (n, L.held() - h0)
    full = L.held()
    L.fake.fake_set_limit(full)  # nothing left: the state's arrays replace the slices
    st = L.state(1024, 1024, 65536)
    L.c.realq_bgd_state_destroy(st)
    L.ok("realq_hessian_accum", buf(1), buf(2), 65536, 14336, buf(3))  # in what is left, or into H itself
    L.fake.fake_set_limit(L.held())
    L.ok("realq_hessian_accum", buf(1), buf(2), 65536, 14336, buf(3))
    L.fake.fake_set_limit(-1)
    for n in (256, 1024, 3000):
        for s in (None, buf(2)):
            L.ok("realq_hessian_accum", buf(1), s, 40000, n, buf(3))
            L.fake.fake_reset()
            for T in range(1, 40000, 211):
                L.ok("realq_hessian_accum", buf(1), s, T, n, buf(3))
            assert L.fake.fake_mallocs() == 0, (n, s)


def little_room(L):
    """Calls succeed in the memory that they cannot do without (measured as the least before padded
    copies of the activations and product slices existed, and 2% for padded rows), and in any larger
    amount: what is optional leaves room for what is not."""
    cases = [(5588, dict(m=1024, n=4096, T=262144, steps=8, lr=1e-5)),
             (6356, dict(m=1024, n=4096, T=262144, steps=8, lr=1e-5, s=True)),
             (1158, dict(m=1000, n=1352, T=30001, steps=4, M=True, P=True)),
             (2782, dict(m=4096, n=1353, T=30001, steps=4, M=True, s=True)),
             (3672, dict(m=512, n=4097, T=200001, steps=2)), (3609, dict(m=512, n=4097, T=200001, steps=0)),
             (3237, dict(m=512, n=4096, T=200000, steps=2, batch=1001)),
             (3989, dict(m=512, n=4097, T=200000, steps=2, batch=100, s=True)),
             (9644, dict(m=512, n=14336, T=65536, steps=2, s=True)),
             (1301, dict(m=512, n=2048, T=65536, steps=2, loss_clip=0.95, batch=1003))]
    for mb, case in cases:
        for room in [int(mb * 1.02) + 64 * k for k in range(120)]:
            L.fresh()
            L.fake.fake_set_limit(room << 20)
            rc, msg = L.layer(**case)
            assert rc == 0, (case, room, mb, msg)
        rc, msg = L.layer(**case)  # once more on the buffers held
        assert rc == 0, (case, msg)
    for mb in range(272, 1200, 16):
        L.fresh()
        L.fake.fake_set_limit(mb << 20)
        L.ok("realq_handoff", buf(1), buf(2), buf(3), 65536, 4097, 1000, buf(5))


def under_capture(L):
    """While the stream records a graph, calls no larger than earlier ones allocate nothing, also where
    they take another route or more slices than the larger call did."""
    i32 = ctypes.c_int
    calls = [("realq_hessian_accum", lambda T, n: (buf(1), None, T, n, buf(3))),
             ("realq_hessian_accum", lambda T, n: (buf(1), buf(2), T, n, buf(3))),
             ("realq_fisher_accum", lambda T, n: (buf(1), T, n, buf(3))),
             ("realq_pullback_metric", lambda T, n: (buf(1), None, T, n, i32(0), buf(3))),
             ("realq_pullback_metric", lambda T, n: (buf(1), buf(2), T, n, i32(1), buf(3))),
             ("realq_handoff", lambda T, n: (buf(1), buf(2), buf(3), T, n, 1000, buf(5)))]
    sizes = [(T, n) for T in (8192, 5000, 4096, 1025, 300, 17) for n in (8192, 4096, 2048, 1001, 512, 133, 16)]
    for name, args in calls:
        for T0, n0 in ((8192, 8192), (4096, 2048), (1025, 1001)):
            L.fresh()
            L.ok(name, *args(T0, n0))
            L.fake.fake_reset()
            L.fake.fake_set_capturing(1)
            for T, n in sizes:
                if T <= T0 and n <= n0:
                    L.ok(name, *args(T, n))
                    assert L.fake.fake_mallocs() == 0, (name, T0, n0, T, n)
            L.fake.fake_set_capturing(0)


if __name__ == "__main__":
    globals()[sys.argv[3]](Library(sys.argv[1], sys.argv[2]))
    print("passed")
