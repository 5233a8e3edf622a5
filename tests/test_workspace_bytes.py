"""What a plan's workspace holds per record: the record (48 bytes), its centre
(8), rectangle (8), tiles, depth bits, first slot and group offset (4 each),
and nothing beyond the groups' sums and the regions' alignment."""
import ctypes as C

from test_abi_cpu import L, _kf, _view  # noqa: F401 (L: a fixture)


def test_bytes_per_record(L):  # noqa: F811
    from paper_2506_02741_amd import _lib

    def need(n):
        ka, va, h = (_lib.vtgs_keyframe * 1)(_kf(n)), (_lib.vtgs_view * 1)(_view()), C.c_void_p()
        assert L.vtgs_plan_create(ka, 1, va, 1, C.byref(_lib.default_params()), 4096, C.byref(h)) == 0
        try:
            return L.vtgs_plan_workspace_bytes(h)
        finally:
            L.vtgs_plan_destroy(h)
    n = 1 << 20
    assert 80 * n <= need(2 * n) - need(n) <= 81 * n
