"""The waves per CU that the rule of passes in two launches counts on: a kernel whose registers
outgrow them makes the rule wrong without any result showing it."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

KERNELS = [  # one type, several replicas; waves per CU
    ("_ZN3vbc7k_countIfLb0ELb0ELb0ELb0EEEvNS_7BuffersENS_6LaunchEiPdiNS_6OneRepIXT2_EEE", 32),
    ("_ZN3vbc7k_countIdLb0ELb0ELb0ELb0EEEvNS_7BuffersENS_6LaunchEiPdiNS_6OneRepIXT2_EEE", 32),
    ("_ZN3vbc7k_forceIfLb0ELb0ELb0ELb0EEEvNS_7BuffersENS_6LaunchEiiNS_8StepArgsEPdS4_NS_6OneRepIXT2_EEE", 24),
    ("_ZN3vbc7k_forceIdLb0ELb0ELb0ELb0EEEvNS_7BuffersENS_6LaunchEiiNS_8StepArgsEPdS4_NS_6OneRepIXT2_EEE", 20),
    ("_ZN3vbc7k_nlistENS_7BuffersENS_6LaunchEi", 24),
    ("_ZN3vbc9k_observeILb0EEEvNS_7BuffersENS_6LaunchEiPiS3_Pl", 32),
    ("_ZN3vbc10k_cc_localILb0EEEvNS_7BuffersENS_6LaunchEiNS_11ClusterWorkEPlS4_l", 32),
]


@pytest.mark.parametrize("name,waves", KERNELS)
def test_waves_per_cu(name, waves):
    from paper_2609_07842_amd import vbc
    L, n = vbc.lib(), C.c_int(0)
    handle = C.c_void_p(C.addressof(C.c_void_p.in_dll(L, name)))
    # blocks of two waves, no dynamic LDS: the registers decide
    assert L.hipOccupancyMaxActiveBlocksPerMultiprocessor(C.byref(n), handle, 128, C.c_size_t(0)) == 0
    print(f"[occupancy] {name[:24]} {n.value} blocks of two waves", flush=True)
    assert 2 * n.value >= waves
