// Prints the segment lengths that each_segment_rows visits for every h of argv[1] .. argv[2].
#include <cstdio>
#include <cstdlib>

#include "wv_pieces.h"

int main(int, char** argv) {
    for (int h = atoi(argv[1]); h <= atoi(argv[2]); ++h) {
        wv::each_segment_rows(h, [](int r) { printf("%d ", r); });
        printf("\n");
    }
}
