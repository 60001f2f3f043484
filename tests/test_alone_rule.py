"""Which check passes form the profile themselves (one workgroup, sums of 32 bits) and which leave it to the finalising kernel."""
import hostcode

BODY = r"""
#include <cstdio>
#include "tao_check.hpp"
namespace tao {
thread_local int g_last_hip_error = 0;
static int finalised = 0;
void launch_profile_reduce(const CheckWorkspace&, int, unsigned long long, tao_profile*, hipStream_t) { ++finalised; }
}
int main() {
    using namespace tao;
    tao_profile out;
    const long sizes[] = {0, 1, 16384, 1L << 31, (1L << 32) - 1, 1L << 32, (1L << 32) + 1, 13L << 29, (1L << 36) - 1};
    for (int nblocks : {1, 2})
        for (long n : sizes) {
            finalised = 0;
            launch_finish(CheckWorkspace{}, nblocks, n, &out, nullptr);
            std::printf("%d %ld %d %d\n", nblocks, n, pass_out(CheckWorkspace{}, nblocks, n, &out).alone == &out, finalised);
        }
}
"""


def test_a_single_workgroup_sums_in_32_bits_only_what_fits(tmp_path):
    lines = [tuple(map(int, line.split())) for line in hostcode.run(BODY, tmp_path)]
    assert len(lines) == 18
    for nblocks, n, alone, finalised in lines:
        assert alone == (nblocks == 1 and n < 2 ** 32), (nblocks, n)
        assert finalised == 1 - alone, (nblocks, n)              # one of the two forms the profile
