"""Where a lane of the screen counts its errors of 0: in no bin, no word of the kernel's and no sum.  (What is counted there is never read, so no
profile shows a word that is another's.)"""
import hostcode

BODY = r"""
#include <cstdio>
#include "linear_screen.hpp"
namespace tao { thread_local int g_last_hip_error = 0; }
int main() {
    using namespace tao;
    for (int blocks : {1, 2, 4})
        for (int early : {0, 1})
            for (int lane = 0; lane < 64; ++lane) {
                const int cols = blocks == 1 ? 32 : 64, strip = cols + (spare_words(blocks) ? 0 : 4);
                std::printf("%d %d %d %d %d %d %d\n", blocks, lane, zero_word(lane, blocks, early, cols, strip), words_before_stages(blocks, early),
                            kHistWords, cols, strip);
            }
}
"""


def test_errors_of_0_are_counted_where_nothing_else_lies(tmp_path):
    lines = [tuple(map(int, line.split())) for line in hostcode.run(BODY, tmp_path)]
    assert len(lines) == 3 * 2 * 64
    for blocks, lane, word, stages, bins, cols, strip in lines:
        if blocks > 1:
            assert word == bins + lane < stages, (blocks, lane, word)
        else:
            row, column = divmod(word - stages, strip)
            assert 0 <= row < 32 and cols <= column < strip, (blocks, lane, word, row, column)
