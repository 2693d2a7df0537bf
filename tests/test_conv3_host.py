"""Host checks of the network kernels' and the batch's entry points: what they take.  Without a GPU
an accepted call ends at its launch (KATS_EHIP); the buffers are never touched."""
from ctypes import c_int64, c_uint64, c_void_p

import pytest

torch = pytest.importorskip("torch")
K = pytest.importorskip("paper_2201_02309_amd")
from paper_2201_02309_amd import network as N  # noqa: E402

EINVAL, EHIP = -1, -6
PTR = c_void_p(1 << 20)

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="accepted calls would launch")


def _conv(shape, xs, ys):
    lib = K.load_library()
    a = ((c_int64 * 3)(*xs), (c_int64 * 3)(*ys), (c_int64 * 6)(*shape))
    st = {lib.katsevich_conv3(PTR, a[0], PTR, None, PTR, a[1], a[2], 0, None),
          lib.katsevich_conv3_grad(PTR, a[0], PTR, a[1], a[2], PTR, PTR, PTR,
                                   c_uint64(lib.katsevich_conv3_scratch_bytes()), None)}
    assert len(st) == 1
    return st.pop()


PLANE = 512 * 512


@pytest.mark.parametrize("cin,xc,ok", [
    (1, 300 * PLANE, True), (1, 1 << 62, True),              # one channel: its stride plays no part
    (16, 272 * PLANE, True), (16, (4096 - 1) * PLANE // 15, True), (16, 274 * PLANE, False),
    (2, (1 << 30) - PLANE, True), (2, (1 << 30) - PLANE + 1, False), (2, 1 << 62, False), (2, -1, False)])
def test_channel_strides(cin, xc, ok):
    want = EHIP if ok else EINVAL
    dense = (16 * PLANE, PLANE, 16 * PLANE)
    assert _conv((1, cin, 16, 10, 512, 512), (16 * xc if xc < 1 << 40 else xc, xc, PLANE), dense) == want
    assert _conv((1, 16, cin, 10, 512, 512), dense, (0, xc, PLANE)) == want


MANY = 1 << 24


@pytest.mark.parametrize("shape,ok", [
    ((1, 1, MANY - 1, 1, 1), True), ((1, 1, MANY, 1, 1), False), ((1 << 12, 1 << 6, 1 << 6, 1, 1), False),
    ((MANY // 3, 3, 1, 1, 1), True), ((MANY // 3 + 1, 3, 1, 1, 1), False)])
def test_launch_limits_of_planes(shape, ok):
    """A workgroup per plane: less than 2^24 of them, 2^32 threads."""
    lib = K.load_library()
    want = EHIP if ok else EINVAL
    s, n = (c_int64 * 3)(1, 1, 1), (c_int64 * 5)(*shape)
    assert lib.katsevich_stack3(PTR, s, PTR, n, None) == want
    assert (lib.katsevich_prelu_scratch_bytes(n) > 0) == ok
    assert lib.katsevich_prelu_grad(PTR, s, PTR, s, PTR, PTR, s, PTR, n, PTR, c_uint64(1 << 62), None) == want


# blocks of 8192 samples: 2 a plane, 2^12 a plane
@pytest.mark.parametrize("shape,ok", [((1, 1, MANY // 2 - 1, 1, 8193), True), ((1, 1, MANY // 2, 1, 8193), False),
                                      ((1, 1, (1 << 12) - 1, 1 << 13, 1 << 12), True),
                                      ((1, 1, 1 << 12, 1 << 13, 1 << 12), False)])
def test_launch_limits_of_prelu(shape, ok):
    lib = K.load_library()
    s, n = (c_int64 * 3)(1, 1, 1), (c_int64 * 5)(*shape)
    assert (lib.katsevich_prelu_scratch_bytes(n) > 0) == ok
    assert lib.katsevich_prelu_grad(PTR, s, PTR, s, PTR, PTR, s, PTR, n, PTR, c_uint64(1 << 62),
                                    None) == (EHIP if ok else EINVAL)


@pytest.mark.parametrize("shape,ok", [((1, 1, 1, 1, 8 * (MANY - 1), 1), True), ((1, 1, 1, 1, 8 * MANY, 1), False),
                                      ((65535, 1, 1, 1, 1, 1), True), ((65536, 1, 1, 1, 1, 1), False),
                                      ((1, 1, 1, 4 * 65535, 1, 1), True), ((1, 1, 1, 4 * 65535 + 1, 1, 1), False)])
def test_launch_limits_of_convolutions(shape, ok):
    assert _conv(shape, (1, 1, 1), (1, 1, 1)) == (EHIP if ok else EINVAL)


def test_batch_without_host_memory():
    """A batch whose host tables cannot be allocated is refused, not ended by an exception."""
    import subprocess
    import sys
    code = """
import ctypes, resource, sys
lib = ctypes.CDLL(sys.argv[1])
resource.setrlimit(resource.RLIMIT_AS, (16 << 30, 16 << 30))
p = (ctypes.c_void_p * 1)(1 << 20)
print(lib.katsevich_backproject_batch(p, p, p, (1 << 31) - 1, None))
"""
    r = subprocess.run([sys.executable, "-c", code, K.katsevich.LIB_PATH], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.split() == ["-7"], (r.returncode, r.stderr[-500:])


@pytest.mark.parametrize("call", [lambda x: K.katsevich.conv3(x, torch.zeros(1, 1, 3, 3, 3)),
                                  lambda x: K.katsevich.conv3_grad(x, x, (1, 1, 3, 3, 3)),
                                  lambda x: K.katsevich.stack3(x),
                                  lambda x: K.katsevich.prelu_grad(x, x, torch.zeros(1))])
def test_volumes_of_another_kind(call):
    """Host tensors, and types and ranks that the kernels do not read, are refused by the binding."""
    for x in (torch.zeros(1, 1, 2, 3, 4), torch.zeros(1, 1, 2, 3, 4, dtype=torch.float16), torch.zeros(1, 2, 3, 4)):
        with pytest.raises(K.KatsevichError) as e:
            call(x)
        assert e.value.status == EINVAL
