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
