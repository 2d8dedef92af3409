"""Registers and scratch memory of the kernels in the built library, read from
the metadata that the compiler leaves in its code objects (no GPU): the
occupancy that the launch shapes and the comments state."""
import struct
import subprocess

import pytest

msgpack = pytest.importorskip("msgpack")

from paper_2603_26272_amd import za


def _notes(elf):
    """The AMDGPU metadata (note type 32) of one ELF code object."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, num = struct.unpack_from("<HH", elf, 0x3A)
    for k in range(num):
        sh = shoff + k * entsize
        kind, = struct.unpack_from("<I", elf, sh + 4)
        off, size = struct.unpack_from("<QQ", elf, sh + 24)
        o = off
        while kind == 7 and o < off + size:   # SHT_NOTE
            nsz, dsz, t = struct.unpack_from("<III", elf, o)
            d = o + 12 + (nsz + 3) // 4 * 4
            if t == 32:
                yield msgpack.unpackb(elf[d:d + dsz])
            o = d + (dsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    """{demangled name: metadata}"""
    blob = open(za.LIB_PATH, "rb").read()
    found, i = {}, blob.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while i >= 0:
        n, = struct.unpack_from("<Q", blob, i + 24)
        o = i + 32
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", blob, o)
            name = blob[o + 24:o + 24 + ln]
            o += 24 + ln
            if b"gfx950" in name and size:
                for note in _notes(blob[i + off:i + off + size]):
                    found.update({k[".name"]: k for k in note["amdhsa.kernels"]})
        i = blob.find(b"__CLANG_OFFLOAD_BUNDLE__", i + 24)
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout
    out = {d: k for d, k in zip(names.splitlines(), found.values())}
    assert len(out) > 200
    return out


def _waves(k):
    """Wavefronts per SIMD that the registers (vector and accumulation
    together, in units of 8 of 512) allow."""
    return min(8, 512 // (-(-k[".vgpr_count"] // 8) * 8))


# (weights: 1 with pow(), 2 powers of 1 and 2; r)
@pytest.mark.parametrize("wv,r", [(1, 2), (1, 3), (2, 3), (2, 4)])
@pytest.mark.parametrize("d", ["x", "y"])
def test_flux_sweeps_of_general_weights_hold_two_wavefronts(kernels, d, wv, r):
    hits = [k for n, k in kernels.items() if f"k_sweep_{d}_" in n and f"<1, 4, double, 0, {wv}, {r}" in n]
    assert hits
    for k in hits:
        assert _waves(k) >= 2, k[".vgpr_count"]


@pytest.mark.parametrize("r,waves", [(2, 4), (3, 3)])
@pytest.mark.parametrize("mode", [1, 3])   # right-hand side, stage
def test_1d_euler_sweeps_of_pow_weights_keep_their_wavefronts(kernels, mode, r, waves):
    """Two registers more would cost one (a line of 4e6 cells at p = 3/2:
    12 % of a stage)."""
    hits = [k for n, k in kernels.items() if f"k_sweep_x_r<1, 3, double, {mode}, 1, {r}, " in n]
    assert hits
    for k in hits:
        assert _waves(k) >= waves and k[".private_segment_fixed_size"] == 0, k[".vgpr_count"]


def test_fp32_flux_sweep_of_pow_weights_holds_five_wavefronts(kernels):
    hits = [k for n, k in kernels.items() if "k_sweep_x_" in n and "<1, 4, float, 0, 1, 3" in n]
    assert hits and all(_waves(k) >= 5 and k[".private_segment_fixed_size"] == 0 for k in hits)


def test_scratch_memory_stays_small(kernels):
    """The runtime sets scratch aside per queue for a full device (8192
    wavefronts of 64 lanes): at most 128 bytes per lane, 64 MB, in any kernel,
    and in the fused stages none but for launches whose blocks share CUs."""
    fused = {}
    for n, k in kernels.items():
        assert k[".private_segment_fixed_size"] <= 128, (n, k[".private_segment_fixed_size"])
        if "k_fused<" in n:
            T, wv, r, mode, w = [x.strip() for x in n.split("k_fused<")[1].split(">")[0].split(",")]
            fused.setdefault((T, wv, r, mode), []).append((int(w), k[".private_segment_fixed_size"]))
    for key, variants in fused.items():
        assert min(variants)[1] == 0, (key, variants)


def test_flux_sweep_of_pow_weights_at_r2_holds_three_wavefronts(kernels):
    hits = [k for n, k in kernels.items() if "k_sweep_y_" in n and "<1, 4, double, 0, 1, 2" in n]
    assert hits and all(_waves(k) >= 3 and k[".private_segment_fixed_size"] == 0 for k in hits)
