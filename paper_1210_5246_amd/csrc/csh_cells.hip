// The pool of pinned cells the handles' kernels write their rate and flag to
// (csh_internal.h).  Pages of 64 cells in a list; nothing here throws, the callers
// being C entry points.
#include <mutex>
#include <new>

#include "csh_internal.h"

namespace csh {

namespace {

struct CellPage {
    HostCell* cells;
    uint64_t used;  // bit k: cell k is handed out
    CellPage* next;
};
std::mutex cell_mutex;
CellPage* cell_pages = nullptr;  // outlives every handle, also at process exit

CellPage* new_page()
{
    CellPage* page = new (std::nothrow) CellPage{nullptr, 0, cell_pages};
    if (!page) return nullptr;
    void* cells = nullptr;  // portable: a page serves the handles of every device
    if (hipHostMalloc(&cells, 64 * sizeof(HostCell), hipHostMallocPortable) != hipSuccess) {
        delete page;
        return nullptr;
    }
    page->cells = static_cast<HostCell*>(cells);
    return cell_pages = page;
}

}  // namespace

HostCell* acquire_cell()
{
    std::lock_guard<std::mutex> lock(cell_mutex);
    CellPage* page = cell_pages;
    while (page && ~page->used == 0) page = page->next;
    if (!page && !(page = new_page())) return nullptr;
    const int k = __builtin_ctzll(~page->used);
    page->used |= 1ull << k;
    page->cells[k] = HostCell{0.0, 0};
    return page->cells + k;
}

void release_cell(HostCell* cell)
{
    if (!cell) return;
    std::lock_guard<std::mutex> lock(cell_mutex);
    for (CellPage** at = &cell_pages; *at; at = &(*at)->next) {
        CellPage* page = *at;
        if (cell < page->cells || cell >= page->cells + 64) continue;
        page->used &= ~(1ull << (cell - page->cells));
        if (page->used == 0 && cell_pages->next) {
            *at = page->next;
            (void)hipHostFree(page->cells);
            delete page;
        }
        return;
    }
}

}  // namespace csh
