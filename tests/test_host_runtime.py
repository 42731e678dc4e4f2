"""The host runtime's behaviour around failures and limits, against a HIP
runtime made of host memory (fake_hip.cpp): no GPU needed."""
import fake_hip


def test_failed_source_staging_leaves_the_handle_usable():
    """A combined solve whose staging of source parameters cannot be
    allocated reports that, and the handle's other solves go on as before;
    so does the combined one once there is memory again."""
    fake_hip.run('''
h = problem((9, 10, 11), 4, G=3)
assert solve(h)[0] == dsn.DSN_OK
fake.fake_host_limit(10000)
assert solve(h, n_src=200, combine=True)[0] == dsn.DSN_ERR_OUT_OF_MEMORY
assert solve(h)[0] == dsn.DSN_OK, dsn.last_error()
assert solve(h, n_src=3, combine=True)[0] == dsn.DSN_OK, dsn.last_error()
fake.fake_host_limit(1 << 40)
assert solve(h, n_src=200, combine=True)[0] == dsn.DSN_OK, dsn.last_error()
h.close()
''')


def test_capturing_stream_is_refused_untouched():
    """A solve on a stream that is being captured is refused before anything
    is recorded, and the handle's later solves still clear the face words of
    the sweep before when its shape has changed: here the single-pencil words
    and then a tile's."""
    fake_hip.run('''
stream = 0x1000
for entry in ("solve", "noalloc", "adjoint", "batch", "fused"):
    h = problem((9, 20, 18), 4, G=2, fixup=1)
    h.set_sweep_shape(1, 16)
    assert solve(h, stream=stream)[0] == dsn.DSN_OK
    h.set_sweep_shape(1, 16, 0, 2)
    events()
    fake.fake_capture(stream, 1)
    src = SourceSpec(position=(-2.3, 0.7, 0.9), spectrum=np.ones(2))
    s, keep = dsn._source_struct(src, 2)
    o, keep2 = dsn._opts(2, 1e-5, 100, [2, 2], False, stream, batch_mode=int(entry == "fused"))
    buf = np.zeros(8)
    ptr = buf.ctypes.data_as(C.c_void_p)
    if entry == "solve":
        st = solve(h, stream=stream)[0]
        assert solve(h, stream=stream, iters=None)[0] == dsn.DSN_ERR_DEVICE
    elif entry == "noalloc":
        st = dsn.lib().dsn_solve_noalloc(h.handle, C.byref(s), C.byref(o), ptr, None, None)
    elif entry == "adjoint":
        J = C.c_double()
        st = dsn.lib().dsn_solve_adjoint(h.handle, C.byref(s), ptr, C.byref(o), C.byref(J), ptr, None, None)
    else:
        st = dsn.lib().dsn_solve_batch((C.c_void_p * 1)(h.handle.value), 1, (C.POINTER(dsn.Source) * 1)(C.pointer(s)),
                                       np.ones(1, np.int32).ctypes.data_as(dsn._ip), C.byref(o),
                                       (C.c_void_p * 1)(buf.ctypes.data), None)
    assert st == dsn.DSN_ERR_DEVICE, (entry, st)
    log = events()
    assert not [e for e in log if "captured" in e], (entry, log)
    fake.fake_capture(stream, 0)
    assert solve(h, stream=stream)[0] == dsn.DSN_OK
    log = events()
    sweep = min(i for i, e in enumerate(log) if "k_sweep_tile" in e)
    assert "fill" in log[:sweep], (entry, log)
    h.close()
''')


def test_tile_shape_beyond_its_face_offsets_runs_as_pencils():
    """A tile's z faces are addressed with 32-bit offsets over a row of
    pencils, of which the upper half means no face.  In FP64 a row of 32767
    pencils of 512 voxels just fits; one pencil more, and a handle pinned to
    a tile shape sweeps by pencils of as many directions."""
    fake_hip.run('''
from types import SimpleNamespace
def kernels(NJ):
    n = (512, 8 * NJ, 1)
    h = dsn.Problem(SimpleNamespace(nx=n[0], ny=n[1], nz=n[2], dx=1.0, dy=1.0, dz=1.0, density=None, fixup=0,
                    material=np.zeros(n[0] * n[1], np.uint8), sigma_t=np.ones((1, 1)), sigma_s=np.zeros((1, 1, 1, 1)),
                    sn_order=2, legendre_order=0), "fp64")
    h.set_sweep_shape(1, 64, 0, 2)
    events()
    st, info = solve(h)
    assert st == dsn.DSN_OK, dsn.last_error()
    h.close()
    return info.sweep_relay, ["k_sweep_tile" in e for e in events() if "k_sweep" in e]
assert kernels(32767) == (2, [True, True])
assert kernels(32768) == (0, [False, False])
''')


# default shapes by mesh, order, precision, fixup and sources, where one kind
# of item was measured at least a tenth faster: time of a solve on pencils over
# that on tiles
FASTER_ON = [
    ("pencils", (24, 8, 16), 16, "fp32", 1, 40, 0.62),
    ("pencils", (24, 24, 24), 16, "fp32", 1, 12, 0.74),
    ("pencils", (24, 40, 40), 16, "fp32", 1, 4, 0.77),
    ("pencils", (64, 24, 24), 8, "fp32", 1, 40, 0.85),
    ("pencils", (24, 24, 24), 16, "fp64", 1, 4, 0.80),
    ("pencils", (24, 8, 16), 8, "fp64", 1, 40, 0.73),
    ("pencils", (24, 8, 40), 8, "fp64", 0, 40, 0.85),
    ("pencils", (24, 8, 8), 10, "fp32", 0, 64, 0.0),  # a single pencil: nothing to hand over
    ("tiles", (24, 72, 72), 8, "fp32", 1, 1, 1.46),
    ("tiles", (8, 24, 24), 8, "fp32", 1, 40, 1.26),
    ("tiles", (24, 32, 32), 8, "fp32", 0, 40, 1.31),
    ("tiles", (24, 48, 48), 16, "fp32", 1, 1, 1.21),
    ("tiles", (64, 64, 64), 8, "fp32", 1, 1, 1.45),
    ("tiles", (24, 48, 48), 8, "fp64", 1, 1, 1.40),
    ("tiles", (24, 72, 72), 8, "fp64", 0, 1, 1.35),
]


def test_default_shape_is_the_faster_kind():
    out = fake_hip.run('''
for kind, n, sn, precision, fixup, n_src, gain in %r:
    h = problem(n, sn, precision, fixup=fixup)
    st, info = solve(h, n_src=n_src)
    assert st == dsn.DSN_OK, dsn.last_error()
    if ("tiles" if info.sweep_relay else "pencils") != kind:
        print(kind, n, sn, precision, fixup, n_src, gain)
    h.close()
''' % (FASTER_ON,))
    assert out == "", out
