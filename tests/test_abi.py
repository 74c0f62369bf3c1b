"""Host-only checks of the C ABI: the library loads, exports every declared
symbol, and rejects bad arguments before touching any device."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    import paper_2510_21956_amd as la
    if not os.path.exists(la.library_path()):
        from paper_2510_21956_amd import build
        build.build_library()
    return la.load_library()


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "la.h")).read()
    return sorted(set(re.findall(r"LA_API[^;(]*?\b(la_[a-z_]+)\s*\(", text)))


def test_exports_match_header(lib):
    names = declared_symbols()
    import paper_2510_21956_amd as la
    assert names == sorted(la.EXPORTS)
    for n in names:
        assert hasattr(lib, n), n


def test_version_and_strings(lib):
    import paper_2510_21956_amd as la
    assert la.la_version() >= 100
    assert la.la_status_string(0) == "LA_OK"
    for code in range(1, 8):
        assert la.la_status_string(code).startswith("LA_ERR_")
    assert la.la_status_string(99) == "unknown la_status"


def test_workspace_bytes(lib):
    import paper_2510_21956_amd as la
    assert la.la_workspace_bytes(4, 16, 4096, 64, la.LA_F32, 1, 0) > 0
    assert la.la_workspace_bytes(4, 16, 4096, 64, la.LA_F32, 1, 1) > \
        la.la_workspace_bytes(4, 16, 4096, 64, la.LA_F32, 1, 0)
    assert la.la_workspace_bytes(4, 16, 4096, 48, la.LA_F32, 1, 0) == 0      # unsupported D
    assert la.la_workspace_bytes(4, 16, 4096, 256, la.LA_F32, 1, 1) > 0
    assert la.la_workspace_bytes(0, 16, 4096, 64, la.LA_F32, 1, 0) == 0      # bad shape
    assert la.la_workspace_bytes(1, 1, 1, 64, 7, 1, 0) == 0                  # bad dtype
    # size limits: B*H*N*D < 2^40 elements, B*H < 2^31 / 4096
    assert la.la_workspace_bytes(1, 1, 2 ** 31 - 1, 128, la.LA_F32, 1, 0) > 0
    assert la.la_workspace_bytes(64, 64, 2 ** 21, 128, la.LA_F32, 1, 0) == 0   # 2^40 elements
    assert la.la_workspace_bytes(1024, 1024, 64, 64, la.LA_F32, 1, 0) == 0     # too many slices
    # a backward pass that recomputes O and g needs room for them and for the forward pass
    assert la.la_workspace_bytes(4, 16, 4096, 64, la.LA_F32, 1, 2) >= \
        la.la_workspace_bytes(4, 16, 4096, 64, la.LA_F32, 1, 1) + \
        la.la_workspace_bytes(4, 16, 4096, 64, la.LA_F32, 1, 0) + 4 * 16 * 4096 * (64 * 4 + 4)
    # the test hook changes the plan, hence the sizes; 0, 0 restores the automatic plan
    auto = la.la_workspace_bytes(4, 16, 4096, 64, la.LA_F32, 1, 0)
    la.la_debug_override(64, 0)
    assert la.la_workspace_bytes(4, 16, 4096, 64, la.LA_F32, 1, 0) > auto
    la.la_debug_override(0, 1)
    assert la.la_saved_state_bytes(4, 16, 4096, 64, la.LA_F32, 1) == 0
    la.la_debug_override(0, 0)
    assert la.la_workspace_bytes(4, 16, 4096, 64, la.LA_F32, 1, 0) == auto
    # slices x segments must fit the launch grid
    la.la_debug_override(64, 0)
    assert la.la_workspace_bytes(1, 4096, 2 ** 26, 16, la.LA_F32, 1, 0) == 0
    la.la_debug_override(0, 0)
    # the hand-over buffer: present for the matrix-core head sizes, absent otherwise
    assert la.la_saved_state_bytes(4, 16, 4096, 64, la.LA_F32, 1) > 0
    assert la.la_saved_state_bytes(4, 16, 4096, 128, la.LA_BF16, 0) > 0
    assert la.la_saved_state_bytes(4, 16, 4096, 16, la.LA_F32, 1) == 0
    assert la.la_saved_state_bytes(4, 16, 4096, 48, la.LA_F32, 1) == 0


@pytest.mark.parametrize("B,H,N,e,causal,want", [
    (4, 16, 4096, 4, 1, "sums"), (1, 8, 8000, 2, 1, "sums"), (1, 1, 200000, 2, 0, "sums"), (6, 10, 1000, 2, 1, "sums"),
    (10, 17, 400, 2, 1, "unused"), (1, 65, 1000, 2, 1, "unused"), (10, 10, 1000, 4, 1, "unused"), (10, 50, 200, 4, 1, "unused"), (8, 1000, 40, 2, 1, "unused"),  # one segment with the mask
    (8, 1000, 40, 2, 0, "none"), (10, 50, 200, 4, 0, "none"), (8, 1000, 300, 4, 0, "sums")])
def test_hand_over_size_at_head_size_256(lib, B, H, N, e, causal, want):
    """Bounded by 96 MiB or one tensor, and no room for sums where none are handed over."""
    import paper_2510_21956_amd as la
    n = la.la_saved_state_bytes(B, H, N, 256, la.LA_F32 if e == 4 else la.LA_BF16, causal)
    assert n <= max(96 << 20, B * H * N * 256 * e)
    assert n == {"unused": 256, "none": 0}.get(want, n) and (want != "sums" or n >= 4 * B * H * 128 * 129 * 4)
    if want == "sums":  # no more than the segments of the sums kernel have: theirs are the workspace's first part
        slots = 4 * (128 * 128 + 2 * 128)
        shares = B * H * N * 4 * (1 if e == 4 else 1 + 2 * 128)
        ws = la.la_workspace_bytes(B, H, N, 256, la.LA_F32 if e == 4 else la.LA_BF16, causal, 0)
        nseg = (ws - shares) // (4 * slots * B * H)
        assert n <= 4 * B * H * nseg * 4 * (128 * 128 + 128) + 1024 * B * H


@pytest.mark.parametrize("D", [16, 32, 64, 128, 256])
def test_sizes_stay_below_the_documented_bound(lib, D):
    """include/la.h: what a buffer for every length up to N takes; sizes themselves may fall as N grows."""
    import paper_2510_21956_amd as la
    E = {16: 32, 256: 128}.get(D, D)
    for BH in (1, 3, 16, 60, 130, 156, 200, 700, 3100):
        M = 4 * max(BH, 128) if D == 256 else max(BH, {16: 3072, 32: 3072, 64: 1536, 128: 768}[D])
        for dt, causal in ((la.LA_F32, 0), (la.LA_F32, 1), (la.LA_BF16, 0), (la.LA_BF16, 1)):
            most = [0, 0, 0]
            for N in (1, 33, 300, 773, 1165, 3001, 10000, 65537):
                wide = D == 256 and dt == la.LA_BF16
                bound = (4 * M * E * (E + 2) + (BH * N * (1028 if wide else 4) if D == 256 else 0),
                         4 * M * E * (2 * E + 4) + (BH * (N + 1) * (3080 if wide else 8) if D == 256 else BH * N * 4),
                         4 * M * E * (E + 2) + (BH * 1024 if D == 256 else 0))
                size = (la.la_workspace_bytes(1, BH, N, D, dt, causal, 0),
                        la.la_workspace_bytes(1, BH, N, D, dt, causal, 1),
                        la.la_saved_state_bytes(1, BH, N, D, dt, causal))
                most = [max(x, y) for x, y in zip(most, size)]
                assert all(x <= y + 1024 for x, y in zip(most, bound)), (BH, N, dt, causal, most, bound)


@pytest.mark.parametrize("BH,N,D,e,causal,most", [
    (4, 500, 128, 4, 1, 64), (4, 500, 128, 2, 1, 32), (1, 256, 16, 4, 1, 8), (1, 30000, 64, 2, 1, 512),
    (60, 4000, 64, 4, 1, 512), (42, 9979, 128, 4, 1, 256), (190, 10000, 128, 2, 1, 768), (64, 100000, 64, 4, 0, 512),
    (12, 61, 16, 4, 0, 12), (5, 51, 64, 4, 0, 5), (10, 60, 32, 4, 1, 10), (28, 112, 64, 4, 1, 112), (37, 128, 32, 4, 0, 37)])
def test_cuts(lib, BH, N, D, e, causal, most):
    """Short sequences are cut into the shortest segments, unless that costs more kernels than it saves, and no cut leaves a few segments over what the compute
    units hold in whole rounds."""
    import paper_2510_21956_amd as la
    S = max(D, 32)
    slots = la.la_workspace_bytes(1, BH, N, D, la.LA_F32 if e == 4 else la.LA_BF16, causal, 0) // (4 * (S * S + 2 * S))
    assert 0.9 * most <= slots <= most


@pytest.mark.parametrize("BH,N,D,dt", [(120, 383, 256, 1), (4, 2000, 256, 0), (190, 4000, 128, 0), (252, 2000, 128, 1),
                                       (7000, 40, 16, 0), (20000, 40, 16, 0), (15, 2000, 256, 0), (8, 3600, 256, 0),
                                       (2, 15013, 256, 0), (25, 1231, 256, 0), (1, 28490, 256, 0)])
def test_forward_static_takes_coarser_cuts(lib, BH, N, D, dt):
    """Where the states of the finest cut exceed the scratch, a coarser one is taken: not LA_ERR_WORKSPACE."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("made-up addresses: where there is no device the call ends as it asks for the scratch's address")
    vp = ctypes.c_void_p
    f = [vp(0x10000000 + (k << 36)) for k in range(5)]
    assert lib.la_forward_static(*f, 1, BH, N, D, 1.0, 0.5, 1, dt, vp(0)) == 6


def test_argument_checks_precede_any_launch(lib):
    """Bad arguments are rejected on the host: these calls must return an error
    code without a GPU being present."""
    vp = ctypes.c_void_p
    fake = vp(0x1000)  # never dereferenced: validation fails first
    # NULL pointer
    rc = lib.la_forward(vp(0), fake, fake, fake, fake, 1, 1, 64, 16, 1.0, 0.5, 1, 0, fake, 1 << 20,
                        vp(0))
    assert rc == 1
    # bad shape
    rc = lib.la_forward(fake, fake, fake, fake, fake, 1, 1, 0, 16, 1.0, 0.5, 1, 0, fake, 1 << 20,
                        vp(0))
    assert rc == 2
    # unsupported D
    rc = lib.la_forward(fake, fake, fake, fake, fake, 1, 1, 64, 20, 1.0, 0.5, 1, 0, fake, 1 << 20,
                        vp(0))
    assert rc == 3
    # misaligned
    rc = lib.la_forward(vp(0x1004), fake, fake, fake, fake, 1, 1, 64, 16, 1.0, 0.5, 1, 0, fake,
                        1 << 20, vp(0))
    assert rc == 4
    # workspace too small
    rc = lib.la_forward(fake, fake, fake, fake, fake, 4, 16, 4096, 64, 1.0, 0.5, 1, 0, fake, 16,
                        vp(0))
    assert rc == 5
    rc = lib.la_backward(fake, fake, fake, fake, fake, fake, fake, fake, vp(0), 1, 1, 64, 16, 1.0,
                         0.5, 1, 0, fake, 1 << 20, vp(0))
    assert rc == 1
    # overlapping buffers (distinct 1 MiB-spaced fakes; O on top of Q, then dK on top of dQ)
    f = [vp(0x10000000 + k * (1 << 20)) for k in range(12)]
    rc = lib.la_forward(f[0], f[1], f[2], f[0], f[4], 1, 1, 64, 16, 1.0, 0.5, 1, 0, f[5], 1 << 20,
                        vp(0))
    assert rc == 7
    rc = lib.la_backward(f[0], f[1], f[2], f[3], f[4], f[5], f[6], f[6], f[8], 1, 1, 64, 16, 1.0,
                         0.5, 1, 0, f[9], 1 << 20, vp(0))
    assert rc == 7
    # a workspace that overlaps an input
    rc = lib.la_forward(f[0], f[1], f[2], f[3], f[4], 1, 1, 64, 16, 1.0, 0.5, 1, 0, f[1], 1 << 20,
                        vp(0))
    assert rc == 7
    rc = lib.la_backward(fake, fake, fake, fake, fake, fake, fake, fake, fake, 4, 16, 4096, 64,
                         1.0, 0.5, 1, 0, fake, 16, vp(0))
    assert rc == 5


def test_header_is_plain_c(tmp_path):
    """include/la.h is a C header: it must compile as C and as C++ on its own."""
    import shutil
    import subprocess
    hdr = os.path.join(ROOT, "include", "la.h")
    for cc, lang in (("gcc", "c"), ("g++", "c++")):
        if shutil.which(cc) is None:
            pytest.skip("%s not available" % cc)
        subprocess.run([cc, "-fsyntax-only", "-Wall", "-Werror", "-x", lang, hdr], check=True)
