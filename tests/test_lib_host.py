"""Host-side checks of libspk that need no GPU: the library loads, exports
every symbol include/spk.h declares, presets match the workload
definitions, and parameter validation rejects bad input before any device
call."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

import inputs as I
import paper_2102_04681_amd as pkg
from paper_2102_04681_amd import spk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    src = open(os.path.join(ROOT, "include", "spk.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(spk_[a-z_0-9]+)\s*\(", src)))


def test_library_exports_every_declared_symbol():
    L = spk.lib()
    names = _declared()
    assert len(names) >= 19
    for name in names:
        assert hasattr(L, name), name
    assert sorted(names) == sorted(spk.EXPORTED)
    assert L.spk_abi_version() == spk.SPK_ABI_VERSION


@pytest.mark.parametrize("struct", [spk.spk_params, spk.spk_stats_t])
def test_struct_layout_matches_header(struct, tmp_path):
    # compile a probe against include/spk.h and compare every field offset
    # and the size with the ctypes mirror used by the binding
    name = struct.__name__
    lines = ["#include <stdio.h>", "#include <stddef.h>", '#include "spk.h"', "int main(void){",
             f'printf("%zu\\n", sizeof({name}));']
    for f, _ in struct._fields_:
        lines.append(f'printf("%zu\\n", offsetof({name}, {f}));')
    lines.append("return 0;}")
    src = tmp_path / "probe.c"
    src.write_text("\n".join(lines))
    exe = tmp_path / "probe"
    subprocess.check_call(["gcc", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)])
    out = [int(x) for x in subprocess.check_output([str(exe)]).split()]
    assert out[0] == C.sizeof(struct)
    assert out[1:] == [getattr(struct, f).offset for f, _ in struct._fields_]


_FIELDS = ["n", "neuron_kind", "conn_kind", "frac_exc", "dt_ms", "tau_m_ms", "t_ref_ms", "v_rest",
           "v_th", "v_reset", "v0_lo", "v0_hi", "i_bias", "p", "k_out", "k_in_exc", "k_in_inh",
           "w_uniform", "w_exc", "w_inh", "w_lo", "w_hi", "delay_min", "delay_max", "ext_lambda",
           "ext_w", "src_rate_hz", "acc_mode", "fixed_shift"]


@pytest.mark.parametrize("index", range(5))
@pytest.mark.parametrize("driven", [False, True])
def test_presets_match_workload_definitions(index, driven):
    got = pkg.preset(index, driven=driven, rate_hz=10.0, seed=3)
    want = I.config(index, driven=driven, seed=3, rate_hz=10.0)
    for f in _FIELDS:
        assert np.float32(got[f]) == np.float32(want[f]) or got[f] == want[f], (f, got[f], want[f])
    assert got["seed"] == 3 and got["max_steps"] == want["steps"]


def _status(cfg, **over):
    p = spk.make_params(dict(cfg, **over), max_steps=10)
    h = C.c_void_p()
    return spk.lib().spk_create(C.byref(p), None, C.byref(h))


@pytest.mark.parametrize("over", [
    dict(n=0), dict(delay_min=0), dict(delay_min=5, delay_max=4), dict(delay_max=300),
    dict(delay_min=1, delay_max=70), dict(dt_ms=0.0), dict(tau_m_ms=-1.0), dict(p=1.5),
    dict(frac_exc=2.0), dict(neuron_kind=7), dict(conn_kind=9), dict(acc_mode=4),
    dict(t_ref_ms=100.0), dict(ext_lambda=500.0), dict(acc_mode=1, fixed_shift=40),
])
def test_invalid_parameters_rejected_on_host(over):
    assert _status(I.config(0), **over) == spk.SPK_EINVAL


def test_fixed_point_weight_range_rejected_on_host():
    assert _status(I.config(0), acc_mode=1, fixed_shift=30, w_inh=-4.5) == spk.SPK_EOVERFLOW


def test_abi_version_checked():
    p = spk.make_params(I.config(0), max_steps=10)
    p.abi_version = 99
    h = C.c_void_p()
    assert spk.lib().spk_create(C.byref(p), None, C.byref(h)) == spk.SPK_EINVAL
    assert b"abi" in spk.lib().spk_last_error()


def test_null_safety():
    L = spk.lib()
    L.spk_destroy(None)
    assert L.spk_step(None, 1) == spk.SPK_EINVAL
    assert L.spk_preset(7, 0, 0.0, 1, C.byref(spk.spk_params())) == spk.SPK_EINVAL


def _host_program(tmp_path, body):
    """Output of a C++ program that includes the kernels' shared header."""
    src, exe = tmp_path / "probe.cpp", tmp_path / "probe"
    src.write_text('#include <cstdio>\n#include <cstring>\n#include "spk_internal.h"\nusing namespace spk;\n' + body)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_2102_04681_amd", "csrc"), str(src), "-o", str(exe)])
    return subprocess.check_output([str(exe)], text=True)


def test_explicit_weights_are_stored_by_their_first_class(tmp_path):
    # a table of n distinct weights whose unused entries repeat the first
    out = _host_program(tmp_path, """
int main() {
    const uint32_t w[kMaxClasses] = {0x3f800000u, 0xbf800000u, 0u, 0x80000000u};
    for (uint32_t n = 1; n <= kMaxClasses; n++) {
        uint32_t t[kMaxClasses];
        for (uint32_t k = 0; k < kMaxClasses; k++) t[k] = w[k < n ? k : 0];
        for (uint32_t k = 0; k < n; k++) printf("%u ", weight_class(t, w[k]));
    }
}""")
    assert out.split() == "0 0 1 0 1 2 0 1 2 3".split()


def test_every_spike_of_a_batch_has_one_lane(tmp_path):
    # the resident kernel's split of the tiles' spikes over waves and lanes,
    # as a wave decides it (the choice is the whole wave's): every spike of
    # every tile once, for every number of tiles; shared tiles at every count
    # up to a tile's largest batch, others at mixed counts
    out = _host_program(tmp_path, """
#include <cstdlib>
#include <vector>
static std::vector<std::vector<uint16_t>> hit;
static bool covered(uint32_t Tn, const std::vector<uint32_t> &c) {
    for (uint32_t t = 0; t < Tn; t++) hit[t].assign(c[t], 0);
    for (uint32_t w = 0; w < kRingWaves; w++) {
        RingShare h[kWave];
        bool many = false;
        for (uint32_t l = 0; l < kWave; l++) {
            h[l] = ring_share(Tn, w, l);
            if (h[l].tile >= Tn) return false;
            many |= h[l].mine && ring_many(h[l], c[h[l].tile]);
        }
        for (uint32_t l = 0; l < kWave; l++) {
            const uint32_t t = h[l].tile;
            if (!h[l].mine) continue;
            uint32_t n0 = h[l].i0, n1 = n0 + 1;
            if (many) {  // the tile's first lane stands for its range
                if (h[l].i0 % kWave) continue;
                ring_range(h[l], c[t], &n0, &n1);
            }
            for (uint32_t i = n0; i < n1 && i < c[t]; i++) hit[t][i]++;
        }
    }
    for (uint32_t t = 0; t < Tn; t++)
        for (uint16_t x : hit[t])
            if (x != 1) return false;
    return true;
}
int main() {
    hit.resize(kRingMaxT);
    for (uint32_t Tn = 1; Tn < kRingWaves; Tn++)
        for (uint32_t c = 0; c <= kMaxTileW; c += c < 1100 ? 1 : 61)
            if (!covered(Tn, std::vector<uint32_t>(Tn, c))) printf("tiles %u spikes %u\\n", Tn, c);
    for (uint32_t Tn = 1; Tn <= kRingMaxT; Tn++)
        for (uint32_t k = 0; k < 40; k++) {
            std::vector<uint32_t> c(Tn);
            for (uint32_t t = 0; t < Tn; t++) c[t] = (uint32_t)rand() % (k < 10 ? 3 : k < 25 ? 70 : 700);
            if (!covered(Tn, c)) printf("tiles %u, mixed\\n", Tn);
        }
}""")
    assert not out, out[:400]


def test_a_captured_delivery_does_not_vouch_for_the_scratch(tmp_path):
    # begin: does the call clear the zero area first; end: it left it at zero
    out = _host_program(tmp_path, """
int main() {
    ScratchFlag f;
    printf("%d", f.begin(false)); f.end(false, true);   // clean
    printf("%d", f.begin(false)); f.end(false, false);  // a launch failed, and the clear after it
    printf("%d", f.begin(true)); f.end(true, true);     // captured: clears in the graph
    printf("%d", f.begin(false)); f.end(false, true);   // eager before the graph ran: clears for itself
    printf("%d", f.begin(false)); f.end(false, true);   // clean
    printf("%d", f.begin(true));                        // captured and given up
    printf("%d", f.begin(false));                       // (returns without an end: unclean)
    printf("%d", f.begin(false));
}""")
    assert out == "00110001"


def test_kernel_reciprocal_divisions_are_exact():
    # The persistent kernel replaces two run-time divisions by multiplies
    # with precomputed reciprocals; both are exact over the operand ranges
    # the kernel uses (checked exhaustively here, in exact integers):
    #  - x / T8 as the high 32 bits of x * ceil(2^32 / T8), for x * T8 < 2^32
    #    (x: buckets < 1024, fill counters < 2048, resets < 4096; T8 <= 256);
    #  - q / spc as (q * ceil(2^16 / spc)) >> 16 for q < 256, spc <= 256.
    import numpy as np
    x = np.arange(4096, dtype=np.uint64)
    for t8 in range(2, 257):
        inv = ((1 << 32) + t8 - 1) // t8
        assert inv < (1 << 32)
        got = (x * np.uint64(inv)) >> np.uint64(32)
        assert np.array_equal(got, x // np.uint64(t8)), t8
    q = np.arange(256, dtype=np.uint64)
    for spc in range(1, 257):
        inv = (65536 + spc - 1) // spc
        got = (q * np.uint64(inv)) >> np.uint64(16)
        assert np.array_equal(got, q // np.uint64(spc)), spc
