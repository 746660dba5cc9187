"""Workspace sizes of the pose solves: a workspace kept for the largest problem a
program has serves all its smaller ones, and holds what the launches write."""
import pytest

from paper_2412_12392_amd import _lib


@pytest.fixture(scope="module")
def lib():
    return _lib.load()


# Both sides of the changes of launch shape (131,072 pixels; 1,536 workgroups an accumulation).
FRAMES = [(2, 2), (48, 64), (120, 160), (160, 224), (240, 320), (256, 512), (257, 511), (362, 362), (363, 363),
          (384, 512), (512, 512), (720, 960), (1449, 1449), (4096, 4096)]


def test_track_workspace_grows_with_the_frame(lib):
    frames = sorted(FRAMES, key=lambda f: f[0] * f[1])
    sizes = [lib.m3s_track_workspace_bytes(h, w) for h, w in frames]
    assert sizes == sorted(sizes), list(zip(frames, sizes))


@pytest.mark.parametrize("H,W", FRAMES)
def test_backend_workspace_grows_with_the_edges(lib, H, W):
    edges = list(range(1, 300)) + [383, 384, 385, 511, 512, 767, 768, 769, 1023, 1535, 1536, 1537, 4000, 65535]
    sizes = [lib.m3s_backend_workspace_bytes(8, H, W, e) for e in edges]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("E", [1, 2, 6, 15, 16, 63, 64, 65, 199, 384, 1535, 1536, 65535])
def test_backend_workspace_grows_with_the_frame(lib, E):
    frames = sorted(FRAMES, key=lambda f: f[0] * f[1])
    sizes = [lib.m3s_backend_workspace_bytes(8, h, w, E) for h, w in frames]
    assert sizes == sorted(sizes), list(zip(frames, sizes))
    assert [lib.m3s_backend_workspace_bytes(n, 48, 64, E) for n in range(2, 129)] == \
        sorted(lib.m3s_backend_workspace_bytes(n, 48, 64, E) for n in range(2, 129))


@pytest.mark.parametrize("N,H,W,E", [(32, 384, 512, 65), (8, 120, 160, 15), (96, 160, 224, 199), (4, 384, 512, 15),
                                     (4, 384, 512, 16), (2, 2, 2, 1), (128, 48, 64, 65535)])
def test_backend_workspace_holds_its_parts(lib, N, H, W, E):
    def blocks(matches):  # workgroups of 256 lanes an edge, at that many matches a lane
        return min(1024, -(-H * W // (256 * matches)))

    per_edge = blocks(8) if blocks(8) * E >= 1536 else blocks(4)
    n = 7 * (N - 1)
    parts = [per_edge * E * 32 * 4,          # a row of 32 floats a workgroup
             E * (12 * 4 + 40 * 8 + 56 * 8),  # relative pose, normal equations and blocks of an edge
             n * n * 8,                       # the matrix of the dense solve
             3 * E * 4]                       # the blocks every edge enters
    assert lib.m3s_backend_workspace_bytes(N, H, W, E) >= sum(parts)


@pytest.mark.parametrize("H,W", FRAMES)
def test_track_workspace_holds_its_parts(lib, H, W):
    n = H * W
    groups = min(2048, -(-n // 512) if n <= 131072 else -(-n // 1024))
    assert lib.m3s_track_workspace_bytes(H, W) >= 256 + 2 * groups * 32 * 4
