"""The allocation-free sampling call on a workspace full of leftovers: whatever the library's fixed array holds -- here every byte of
it set, the counts of finished slices among them -- a call gives the bits that a handle's step gives, at vocabularies on both
sides of the line from which a row is shared out, and so do the calls after it."""
import ctypes
import subprocess

import pytest
import torch

from paper_2411_00853_amd import workload as wl

pytestmark = pytest.mark.gpu


def fixed_workspace():
    """(device address, bytes) of the array: its name in the library built here leads to the address of the host's handle for it."""
    from paper_2411_00853_amd import binding as sv, build
    lib = sv.lib()
    names = {f[-1]: int(f[0], 16) for f in (l.split() for l in subprocess.check_output(["nm", build.LIB], text=True).splitlines()) if len(f) == 3}
    name, = [n for n in names if n.endswith("7scratchE")]
    handle = ctypes.cast(lib.spec_sample_step_noalloc, ctypes.c_void_p).value - names["spec_sample_step_noalloc"] + names[name]
    at, size = ctypes.c_void_p(), ctypes.c_size_t()
    assert lib.hipGetSymbolAddress(ctypes.byref(at), ctypes.c_void_p(handle)) == 0
    assert lib.hipGetSymbolSize(ctypes.byref(size), ctypes.c_void_p(handle)) == 0
    assert 1 << 18 < size.value <= 640 << 10
    return at, size


@pytest.mark.parametrize("V,B", [(16384, 5), (16385, 5), (65537, 3), (262144, 2), (128256, 40)])
@pytest.mark.parametrize("byte", [0x01, 0x7f, 0xff])
def test_leftovers_change_nothing(V, B, byte):
    from paper_2411_00853_amd import binding as sv
    lib, K = sv.lib(), 3
    at, size = fixed_workspace()
    rng = wl.Rng(V + B, "cuda")
    look = [b % (K + 1) for b in range(B)]
    tl, dl = rng.normal(1, (sum(look) + B, V), 2.0), rng.normal(2, (B, K, V), 2.0)
    toks, us = rng.randint(3, (B, K), V).to(torch.int32), rng.uniform(4, (B, K + 1))
    out = [(torch.full((B,), -9, dtype=torch.int32, device="cuda"), torch.full((B, K + 1), -9, dtype=torch.int32, device="cuda")) for _ in range(3)]
    h = sv.spec_verify_init(sv.sampler_cfg(V, B, K), None, None, None)
    sv.spec_verify_step(h, look, us, 1.0, *out[0], draft_tokens=toks, draft_logits=dl, target_logits_in=tl)
    torch.cuda.synchronize()
    assert lib.hipMemset(at, ctypes.c_int(byte), size) == 0
    torch.cuda.synchronize()
    for na, ot in out[1:]:
        sv.spec_sample_step_noalloc(V, K, look, us, 1.0, na, ot, tl, draft_tokens=toks, draft_logits=dl)
        torch.cuda.synchronize()
        assert torch.equal(na, out[0][0]) and torch.equal(ot, out[0][1])
    h.close()
