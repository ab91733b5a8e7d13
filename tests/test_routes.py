"""Which kernel form small and middle grids take (CPU): the shapes at which
more waves on a block's tiles, or one launch for the whole backward, measured
slower keep the plain forms, and those at which they gain do not."""
import pytest

from routes import CUS, _lib, backward, forward


# (D, blocks, L, causal, docs): the groups lose or gain nothing there
@pytest.mark.parametrize("D,n,L,causal,docs", [
    (64, 16, 64, 1, 0), (64, 256, 128, 1, 0), (64, 64, 160, 0, 0), (64, 512, 256, 1, 0),
    (64, 480, 300, 1, 0), (64, 480, 300, 1, 1), (64, 512, 512, 0, 0), (64, 768, 1536, 1, 0),
    (64, 1280, 2048, 1, 1), (64, 1280, 8192, 0, 0), (64, 1536, 8192, 1, 0),
    (128, 64, 64, 1, 0), (128, 256, 256, 1, 0), (128, 256, 256, 0, 0), (128, 320, 4096, 0, 0),
    (128, 504, 3000, 0, 0), (128, 640, 4096, 1, 0)])
def test_forward_keeps_one_group(D, n, L, causal, docs):
    assert _lib().fwd(D, n, L, causal, docs, CUS) == 1


@pytest.mark.parametrize("D,n,L,causal,docs,groups", [
    (64, 32, 256, 1, 0, 2), (64, 64, 2048, 1, 0, 4), (64, 512, 512, 1, 0, 2),
    (64, 512, 1024, 0, 0, 2), (64, 1024, 4096, 1, 0, 2), (64, 1280, 8192, 1, 1, 2),
    (128, 128, 300, 0, 0, 2), (128, 512, 4096, 1, 0, 2), (128, 640, 4096, 1, 1, 2)])
def test_forward_groups(D, n, L, causal, docs, groups):
    assert _lib().fwd(D, n, L, causal, docs, CUS) == groups


@pytest.mark.parametrize("D,n,L,causal,docs,groups", [
    (64, 128, 160, 1, 0, 1), (64, 480, 300, 1, 0, 1), (64, 512, 512, 0, 0, 1), (64, 504, 3000, 0, 0, 2),
    (64, 2040, 3000, 1, 0, 1), (128, 384, 4096, 0, 0, 1), (128, 768, 3000, 1, 1, 1),
    (64, 255, 300, 1, 0, 2), (64, 512, 8192, 1, 0, 4), (64, 1024, 4096, 1, 0, 2),
    (128, 512, 4096, 1, 0, 2), (128, 640, 4096, 1, 1, 2)])
def test_dq_groups(D, n, L, causal, docs, groups):
    assert _lib().dq(D, n, L, causal, docs, CUS) == groups


@pytest.mark.parametrize("n,L,causal,docs,groups", [
    (200, 128, 1, 0, 1), (512, 4096, 0, 0, 1), (648, 3000, 1, 0, 1), (768, 3000, 1, 1, 1), (512, 512, 1, 0, 1),
    (256, 512, 0, 0, 2), (512, 8192, 1, 0, 2), (640, 4096, 1, 1, 2)])
def test_dkdv_groups(n, L, causal, docs, groups):
    assert _lib().kv(n, L, causal, docs, CUS) == groups


@pytest.mark.parametrize("D,n,L,causal,rope,joint", [
    (64, 160, 160, 1, 0, 0), (64, 160, 256, 1, 0, 0), (128, 160, 64, 1, 0, 0),
    (128, 160, 512, 0, 0, 0), (128, 160, 512, 1, 0, 0), (128, 144, 300, 0, 0, 0),
    (128, 144, 300, 1, 0, 1), (128, 228, 1536, 0, 0, 0), (64, 16, 128, 1, 0, 0),
    (64, 128, 256, 1, 0, 1), (64, 16, 128, 1, 1, 1), (128, 128, 64, 1, 0, 1),
    (128, 160, 1024, 1, 0, 1), (64, 320, 4096, 0, 0, 1), (64, 321, 4096, 1, 0, 0)])
def test_joint_backward(D, n, L, causal, rope, joint):
    assert _lib().both(D, n, L, causal, rope, CUS) == joint


def test_routes_by_shape():
    assert forward(256, 256, 16, 64) == 1 and backward(256, 256, 16, 64) == "short"
    assert backward(4, 256, 4, 64) == "joint" and backward(4, 256, 128, 64) == "short"
    assert backward(8, 8192, 16, 128) == (1, 1)


def test_no_known_cu_count_means_the_plain_forms():
    for D in (64, 128):
        for L in (64, 300, 1024, 8192):
            for c in (0, 1):
                assert _lib().fwd(D, 8, L, c, 0, 0) == 1 and _lib().dq(D, 8, L, c, 0, 0) == 1
                assert _lib().kv(8, L, c, 1, 0) == 1 and not _lib().both(D, 8, L, c, 0, 0)
