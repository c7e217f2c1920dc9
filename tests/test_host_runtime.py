"""The library's host side where the GPU calls are answered by hip_host.cpp: what it allocates, which
kernels it launches in which shapes, and what it does when memory runs out."""
from host_runtime import host_runtime  # noqa: F401  (a fixture)


def test_full_device_keeps_gate_lists_and_fused_blocks_running(host_runtime):
    """A circuit, a noisy density matrix and fused blocks need no memory beyond the state's: where the
    parameter buffer cannot be allocated (device or pinned), gates run one by one and blocks on their tiles,
    call after call, and the buffer is used once there is room."""
    host_runtime("""
def is_window(): return any("k_window" in l[0] for l in launches())
dims = (3, 2, 4, 3, 2, 3, 2, 3)
c = Q.qd_circuit_create(dims)
for q in (0, 3, 5, 7, 2): Q.qd_circuit_add(c, Q.QD_GATE_F, q)
s, rho = Q.qd_state_init(dims, Q.QD_C128, 0), Q.qd_density_init((2, 3, 2), Q.QD_C128, 0)
big = (3,) * 14
g = type("G", (), dict(kind="U", targets=(0, 1, 2), controls=(), cvals=(), a=0, U=np.eye(27)))
f = Q.qd_fuse(big, [g], 27, 0)
t = Q.qd_state_init(big, Q.QD_C64, 0)
chan = ("chan", (1,), Q.qd_channel_kraus(Q.QD_CHANNEL_DEPHASING, 3, 0.1))
for kind in (DEVICE, PINNED):
    hip.host_limit(kind, hip.host_held(kind) + (1 << 20))
    for _ in range(2):
        hip.host_reset()
        Q.qd_circuit_apply(s, c)
        Q.qd_density_apply_ops(rho, [chan, ("chan", (0,), Q.qd_channel_kraus(Q.QD_CHANNEL_DEPHASING, 2, 0.1)), chan])
        Q.qd_state_sync(s)
        assert len(launches()) >= 5 and not is_window(), launches()
        hip.host_reset()
        Q.qd_apply_fused(t, f, Q.QD_MODE_FP32_MFMA)
        Q.qd_state_sync(t)
        assert [l[0] for l in launches() if "k_fused" in l[0]], launches()
    hip.host_limit(kind, -1)
hip.host_reset()
Q.qd_circuit_apply(s, c)
assert is_window() and len(launches()) == 1, launches()
hip.host_reset()
Q.qd_apply_fused(t, f, Q.QD_MODE_FP32_MFMA)
assert "k_dense_mfma" in launches()[0][0], launches()
for h in (s, rho, t): Q.qd_state_free(h)
Q.qd_fused_free(f)
""")


def test_parameter_buffers_pass_from_state_to_state(host_runtime):
    """A program that makes a state for each circuit does not allocate a parameter buffer for each: freed
    states leave theirs, a bounded number of them, to the next ones, from any thread; an allocation that
    finds no room gets the memory back."""
    host_runtime("""
import threading
RING = 8 << 20
dims = (3, 2, 4, 3, 2, 3, 2, 3)
c = Q.qd_circuit_create(dims)
for q in (0, 3, 5, 7, 2): Q.qd_circuit_add(c, Q.QD_GATE_F, q)
def one():
    s = Q.qd_state_init(dims, Q.QD_C128, 0)
    Q.qd_circuit_apply(s, c)
    return s
for _ in range(20): Q.qd_state_free(one())
assert hip.host_made(PINNED) == 1 and hip.host_made(DEVICE) == 21, (hip.host_made(PINNED), hip.host_made(DEVICE))
many = [one() for _ in range(30)]
assert hip.host_held(PINNED) == 30 * RING           # one each while they live
for s in many: Q.qd_state_free(s)
assert hip.host_held(PINNED) <= 4 * RING and hip.host_held(DEVICE) <= 4 * RING
def work():
    for _ in range(200): Q.qd_state_free(one())
ts = [threading.Thread(target=work) for _ in range(8)]
for t in ts: t.start()
for t in ts: t.join()
assert hip.host_held(PINNED) <= 4 * RING and hip.host_held(DEVICE) <= 4 * RING
assert hip.host_held(DEVICE) > 0
hip.host_limit(DEVICE, hip.host_held(DEVICE) + (1 << 20))
s = Q.qd_state_init((2,) * 20, Q.QD_C128, 0)          # 16 MB: fits without the spare buffers only
hip.host_limit(DEVICE, -1)
Q.qd_state_free(s)
assert hip.host_held(DEVICE) == 0 and hip.host_held(PINNED) == 0
s = one()                                             # a buffer that a graph has recorded is not passed on
hip.host_capture(1)
Q.qd_apply_gate_ex(s, (1, 3, 5), (), (), np.linalg.qr(np.random.default_rng(1).standard_normal((18, 18)))[0], 1)
hip.host_capture(0)
Q.qd_state_free(s)
assert hip.host_held(DEVICE) == 0 and hip.host_held(PINNED) == 0
""")


def test_tiles_of_small_registers_spread_over_the_card(host_runtime):
    """The LDS tile kernel leaves a small register enough tiles for the card (192 of 256 compute units, or
    tiles of 256 amplitudes), whatever the radix by which tiles grow; a large one keeps tiles of about 9 KB."""
    host_runtime("""
def tiles(dims, prec, t):
    s = Q.qd_state_init(dims, prec, 0)
    hip.host_reset()
    U = Q.qd_gate_matrix(Q.QD_GATE_F, dims[t], 0)
    Q.qd_apply_gate(s, (t,), (), (), U)
    Q.qd_state_free(s)
    (name, grid, block, lds), = launches()
    assert "k_slices_tiled" in name
    amp = 16 if prec == Q.QD_C128 else 8
    assert grid * lds == np.prod(dims) * amp
    return grid, lds // amp
for prec in (Q.QD_C128, Q.QD_C64):
    for dims in ((8,) * 5, (4,) * 7, (7,) * 5, (9,) * 4, (5,) * 6, (2,) * 14, (3,) * 9, (2, 3) * 5):
        n, size = tiles(dims, prec, len(dims) - 1)
        assert n * max(dims) >= 192 or size < 256 * max(dims), (dims, prec, n, size)
assert tiles((8,) * 5, Q.QD_C64, 4) == (64, 512)
assert tiles((2,) * 20, Q.QD_C128, 19) == (1024, 1024) and tiles((2,) * 20, Q.QD_C64, 19) == (512, 2048)
assert tiles((3,) * 13, Q.QD_C128, 12) == (2187, 729)
""")


def test_direct_launch_shapes_by_touched_bytes(host_runtime):
    """Untuned complex128 gates of d_T <= 4 take small workgroups where their passes go to HBM, and the
    default ones where the caches hold what they touch."""
    host_runtime("""
def shape(dims, t, c=()):
    s = Q.qd_state_init(dims, Q.QD_C128, 0)
    hip.host_reset()
    dT = int(np.prod([dims[q] for q in t]))
    U = np.linalg.qr(np.random.default_rng(1).standard_normal((dT, dT)))[0].astype(complex)
    Q.qd_apply_gate(s, t, c, [dims[q] - 1 for q in c], U)
    Q.qd_state_free(s)
    (name, grid, block, lds), = launches()
    assert "k_slices_direct" in name
    return block
two = lambda n: (2,) * n
assert shape(two(20), (0,)) == 256 and shape(two(21), (0,)) == 64          # 16 MB, 32 MB
assert shape(two(21), (0,), (17,)) == 256 and shape(two(22), (0,), (18,)) == 64
assert shape(two(21), (0, 1)) == 256 and shape(two(22), (0, 1)) == 64      # d_T = 4: 32 MB, 64 MB
assert shape(two(21), (11, 12)) == 128 and shape(two(20), (11,)) == 256    # strides 512 and 256
assert shape((3,) + two(20), (0,)) == 256 and shape((3,) + two(21), (0,)) == 64   # 50 and 100 MB
""")


def test_explicit_direct_settings_hold(host_runtime):
    """A workgroup size or a number of slices per thread that the caller has set is what gates run with, also
    where it is the default's; 0 gives the shapes of untuned gates back."""
    host_runtime("""
s = Q.qd_state_init((2,) * 24, Q.QD_C128, 0)
U = Q.qd_gate_matrix(Q.QD_GATE_F, 2, 0)
def shape():
    hip.host_reset()
    Q.qd_apply_gate(s, (0,), (), (), U)
    (name, grid, block, lds), = launches()
    return block, (1 << 23) // (grid * block)
assert shape() == (64, 1)
for param, value, want in ((Q.QD_TUNE_DIRECT_BLOCK, 256, (256, 2)), (Q.QD_TUNE_DIRECT_SPT, 2, (256, 2)),
                           (Q.QD_TUNE_DIRECT_BLOCK, 128, (128, 2)), (Q.QD_TUNE_DIRECT_SPT, 4, (256, 4))):
    Q.qd_tune_set(param, value)
    assert shape() == want, (param, value, shape())
    Q.qd_tune_set(param, 0)
    assert shape() == (64, 1)
Q.qd_tune_set(Q.QD_TUNE_DIRECT_BLOCK, 256)
Q.qd_tune_set(Q.QD_TUNE_DIRECT_SPT, 0)
assert shape() == (256, 2)
Q.qd_tune_set(Q.QD_TUNE_DIRECT_BLOCK, 0)
Q.qd_state_free(s)
""")


def test_tile_elems_choose_the_tile(host_runtime, tmp_path):
    """QD_TUNE_TILE_ELEMS and tuned entries say how large a tile grows; untuned tiles stop at 9 KB whatever
    the budget. The autotuner times no launch twice under two names."""
    host_runtime(f"""
path = {str(tmp_path / "tune.json")!r}
def tile(dims, prec):
    s = Q.qd_state_init(dims, prec, 0)
    hip.host_reset()
    Q.qd_apply_gate(s, (len(dims) - 1,), (), (), Q.qd_gate_matrix(Q.QD_GATE_F, dims[-1], 0))
    (name, grid, block, lds), = launches()
    assert "k_slices_tiled" in name
    Q.qd_state_free(s)
    return lds // (16 if prec == Q.QD_C128 else 8)
""" + """
for prec, untuned in ((Q.QD_C128, 1024), (Q.QD_C64, 2048)):
    dims, full = (2,) * 22, 2048 if prec == Q.QD_C128 else 4096       # 256 threads of 8 or 16 amplitudes
    assert tile(dims, prec) == untuned
    for elems in (256, 512, 1024, 2048, 4096):
        Q.qd_tune_set(Q.QD_TUNE_TILE_ELEMS, elems)
        assert tile(dims, prec) == min(elems * full // 2048, full), (prec, elems)
    assert tile((3,) * 13, prec) == (729 if prec == Q.QD_C128 else 2187)
    Q.qd_tune_set(Q.QD_TUNE_TILE_ELEMS, 0)
    assert tile(dims, prec) == untuned
    for elems in (512, 2048):
        with open(path, "w") as f:
            f.write("[\\n{\\"prec\\": %d, \\"bucket\\": 0, \\"tiled\\": 1, \\"block\\": 256, \\"spt\\": 1, \\"tile_elems\\": %d}\\n]\\n"
                    % (prec, elems))
        Q.qd_tune_load(path)
        assert tile(dims, prec) == min(elems * full // 2048, full), (prec, elems)
    Q.qd_tune_set(Q.QD_TUNE_TILE_ELEMS, 0)                             # discards the table
    s = Q.qd_state_init(dims, prec, 0)
    hip.host_reset()
    Q.qd_autotune(s, None)
    Q.qd_state_free(s)
    runs = [[]]                                                        # the tiled candidates of each stride class
    for name, *shape in launches():
        if "k_slices_tiled" not in name: runs.append([])
        else: runs[-1].append(tuple(shape))
    runs = [r for r in runs if r]
    assert runs and all(len(r) == 11 * len(set(r)) for r in runs), [(len(r), len(set(r))) for r in runs]    # 11 launches time one
    Q.qd_tune_set(Q.QD_TUNE_RUN_MIN, 0)
""")


def test_density_operations_hold_a_bounded_list(host_runtime):
    """A superoperator on d_T = 32 takes 16.8 MB: sixty in one call need the memory of a few. Small
    operations still share passes."""
    host_runtime("""
import resource
rho = Q.qd_density_init((32, 2), Q.QD_C64, 0)
K = np.eye(32, dtype=complex)
chan = ("chan", (0,), [K])
Q.qd_density_apply_ops(rho, [chan, chan])
before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
hip.host_reset()
Q.qd_density_apply_ops(rho, [chan] * 60)
grown = (resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before) * 1024
assert grown < 200e6, grown
assert len(launches()) == 60
Q.qd_state_free(rho)
rho = Q.qd_density_init((3, 2, 3, 2), Q.QD_C128, 0)
dep = lambda q, d: ("chan", (q,), Q.qd_channel_kraus(Q.QD_CHANNEL_DEPOLARIZING, d, 0.1))
hip.host_reset()
Q.qd_density_apply_ops(rho, [dep(q, (3, 2, 3, 2)[q]) for q in (0, 1, 2, 3, 0, 2)])
(name, *_), = launches()
assert "k_window" in name
Q.qd_state_free(rho)
""")


def test_fusing_stages_through_a_bounded_pinned_buffer(host_runtime):
    """Two thousand blocks of 81 x 81 (0.2 GB) pass through some 9 MB of pinned memory, and a call that finds
    no room for a later group leaves nothing behind; a small circuit still waits for the GPU once."""
    host_runtime("""
dims = (3,) * 12
U = np.linalg.qr(np.random.default_rng(1).standard_normal((81, 81)))[0].astype(complex)
def gate(t): return type("G", (), dict(kind="U", targets=t, controls=(), cvals=(), a=0, U=U))
ga = Q.GateArray([gate((0, 1, 2, 3 + i % 2)) for i in range(2000)], lambda i: dims)
f = Q.qd_fuse(dims, ga, 81, 0)
assert Q.qd_fused_count(f) == 2000
assert hip.host_peak(PINNED) < 10 << 20, hip.host_peak(PINNED)
assert hip.host_held(PINNED) == 0
whole = hip.host_held(DEVICE)
Q.qd_fused_free(f)
assert hip.host_held(DEVICE) == 0
hip.host_limit(DEVICE, whole // 2)
try:
    Q.qd_fuse(dims, ga, 81, 0)
    raise AssertionError("half of the memory was enough")
except Q.QDError as e:
    assert e.code == Q.QD_ENOMEM
hip.host_limit(DEVICE, -1)
assert hip.host_held(DEVICE) == 0 and hip.host_held(PINNED) == 0
hip.host_reset()
V = Q.qd_gate_matrix(Q.QD_GATE_F, 3, 0)
small = [type("G", (), dict(kind="U", targets=(q,), controls=(), cvals=(), a=0, U=V)) for q in range(12)]
f = Q.qd_fuse(dims, small, 9, 0)
assert Q.qd_fused_count(f) == 6 and hip.host_waits() <= 2
Q.qd_fused_free(f)
""")


def test_trips_are_counted_beside_passes(host_runtime):
    """qd_state_gate_launches counts the passes a list stands for, qd_state_gate_trips the launches made."""
    host_runtime("""
dims = (3, 2, 4, 3, 2, 3, 2, 3)
c = Q.qd_circuit_create(dims)
for q in (0, 3, 5, 7, 2): Q.qd_circuit_add(c, Q.QD_GATE_F, q)
s = Q.qd_state_init(dims, Q.QD_C128, 0)
hip.host_reset()
Q.qd_circuit_apply(s, c)
assert (Q.qd_state_gate_launches(s), Q.qd_state_gate_trips(s), len(launches())) == (5, 1, 1)
hip.host_capture(1)
Q.qd_circuit_apply(s, c)                                  # recorded one by one
hip.host_capture(0)
Q.qd_apply_gate(s, (0,), (), (), Q.qd_gate_matrix(Q.QD_GATE_F, 3, 0))
assert (Q.qd_state_gate_launches(s), Q.qd_state_gate_trips(s), len(launches())) == (11, 7, 7)
Q.qd_state_free(s)
""")


def test_streaming_where_runs_end_inside_sectors(host_runtime):
    """Direct complex128 gates whose planes begin inside 64-byte sectors: plain accesses up to strides of 512
    on states up to 2 GB, of 64 above, streaming ones beyond."""
    host_runtime("""
def streams(d, n, stride, prec=Q.QD_C128):
    dims = (d,) * n
    s = Q.qd_state_init(dims, prec, 0)
    hip.host_reset()
    t = n - 1 - round(np.log(stride) / np.log(d))
    Q.qd_apply_gate(s, (t,), (), (), Q.qd_gate_matrix(Q.QD_GATE_F, d, 0))
    Q.qd_state_free(s)
    (name, *_), = launches()
    assert "k_slices_direct" in name
    return "Lb1E" in name
assert not streams(3, 16, 27) and not streams(3, 17, 243) and streams(3, 16, 729)
assert not streams(7, 10, 49) and streams(7, 10, 343) and streams(5, 12, 125)
assert not streams(5, 12, 625, Q.QD_C64)
""")


def test_capture_query_that_fails_is_no_launch_error(host_runtime):
    """Asked whether it is captured, the null stream answers with an error while another thread captures a
    stream of its own. Lists then run one by one and blocks on their tiles, and the answer is not reported
    as the error of a launch."""
    host_runtime("""
dims = (3, 2, 4, 3, 2, 3, 2, 3)
c = Q.qd_circuit_create(dims)
for q in (0, 3, 5, 7, 2): Q.qd_circuit_add(c, Q.QD_GATE_F, q)
s = Q.qd_state_init(dims, Q.QD_C128, 0)
big = (3,) * 14
g = type("G", (), dict(kind="U", targets=(0, 1, 2), controls=(), cvals=(), a=0, U=np.eye(27)))
f = Q.qd_fuse(big, [g], 27, 0)
t = Q.qd_state_init(big, Q.QD_C64, 0)
hip.host_reset()
hip.host_capture(-1)
Q.qd_circuit_apply(s, c)
Q.qd_apply_fused(t, f, Q.QD_MODE_FP32_MFMA)
Q.qd_apply_gate_ex(s, (1, 3, 5), (), (), np.linalg.qr(np.random.default_rng(1).standard_normal((18, 18)))[0], 1)
hip.host_capture(0)
names = [l[0] for l in launches()]
assert len(names) == 7 and not any("k_window" in n for n in names) and "k_fused" in names[5], names
Q.qd_state_sync(s)
""")
