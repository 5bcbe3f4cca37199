// Walks the windows of page ids as an attention task does, over chunks and page sizes: every key once, page ids of the sequence's
// table and places in LDS alone, an end.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "etc_types.h"

using namespace etc;

static void check(bool ok, const char *what, int page_shift, int j0, int k1)
{
    if (ok) return;
    printf("%s: page shift %d, keys [%d, %d)\n", what, page_shift, j0, k1);
    exit(1);
}

int main()
{
    for (int sh = 0; sh <= 30; ++sh) {
        const long long page = 1ll << sh, win = page * kAttnPages;
        const long long ends[] = {0, 1, 5, page - 1, page, page + 1, win - 1, win, win + 1, 2 * win, 2 * win + 3, 5 * win - 1, (1ll << 31) - 2, (1ll << 31) - 1};
        for (long long start_page : {0ll, 1ll, 3ll, (long long)kAttnPages})
            for (long long n : ends) {
                const long long first = start_page * page, last = first + n;
                if (n < 0 || last >= 1ll << 31 || n / win > 100000) continue;
                const int j0 = (int)first, k1 = (int)last;
                int w0 = j0, w1 = attn_window_end(w0, k1, sh), rounds = 0;
                for (;;) {
                    check(w0 <= w1 && w1 <= k1, "a window outside the chunk", sh, j0, k1);
                    const int pages = attn_window_pages(w0, w1, sh);
                    check((w0 & (page - 1)) == 0 && pages >= 0 && pages <= kAttnPages, "more page ids than fit", sh, j0, k1);
                    check(w1 == w0 ? pages == 0 : (w0 >> sh) + pages - 1 == (w1 - 1) >> sh, "page ids that are not the window's", sh, j0, k1);
                    if (w1 >= k1) break;
                    check(w1 - w0 == win, "a window cut short", sh, j0, k1);
                    check(++rounds <= n / win, "no end", sh, j0, k1);
                    w0 = w1;
                    w1 = attn_window_end(w0, k1, sh);
                }
            }
    }
    puts("ok");
    return 0;
}
