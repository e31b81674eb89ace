"""What the compiler made of the kernels, from the metadata of the built library: memory that a kernel does not declare (arrays it
could not keep in registers) is in there, where no result shows it."""
import struct

import msgpack
import pytest


def _code_objects(blob):
    """The gfx950 images of a library's offload bundles."""
    at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        entries, = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(entries):
            offset, size, n = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + n]:
                yield blob[at + offset:at + offset + size]
            p += 24 + n
        at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__", p)


def _kernels():
    import paper_2604_03425_amd as pkg
    out = {}
    for image in _code_objects(open(pkg.library_path(), "rb").read()):
        at = image.find(b"AMDGPU\0\0")   # the name of the metadata's note, after its sizes and type
        size, = struct.unpack_from("<I", image, at - 8)
        for k in msgpack.unpackb(image[at + 8:at + 8 + size])["amdhsa.kernels"]:
            out[k[".name"]] = k
    return out


@pytest.mark.parametrize("groups", [3, 4, 6, 9, 12])
def test_wide_conversions_keep_their_arrays_in_registers(groups):
    k = _kernels()["_Z16conv_wide_kernelILi%dEEv8WideArgs" % groups]
    assert k[".group_segment_fixed_size"] == 2 * groups * 1024   # two images of the matrices, nothing else
    assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0
    assert k[".vgpr_count"] <= (128 if groups <= 9 else 168)     # two workgroups of 8 waves to a compute unit, or one


def test_profiles_name_the_two_pass_kernels_as_the_library_does():
    """The per-kernel tables join a trace's names with the library's kinds: every kind of a two-pass kernel is found under its name."""
    import subprocess
    from paper_2604_03425_amd import binding, profile_summary
    names = subprocess.run(["c++filt"], input="\n".join(_kernels()), stdout=subprocess.PIPE, text=True, check=True).stdout.splitlines()
    lib = binding._lib
    kinds = {lib.ckks_prof_kind_name(k).decode() for k in range(lib.ckks_prof_num_kinds())}
    assert {k for k in kinds if k.startswith("ntt16_")} <= {profile_summary.kind(n) for n in names}
